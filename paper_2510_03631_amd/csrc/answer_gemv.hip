// Single-query Answer: a[r] = sum_j D[r][j] * q[j] mod 2^32.
//
// The server's per-query response (Definition 1) is a matrix-vector product
// whose cost is streaming the database once: every byte of D is used once,
// so the kernel is bound by HBM bandwidth (the paper makes the same
// observation for its XOR variant in Section 5.2: low operational intensity,
// coalescing rather than matrix units).  Design for gfx950:
//
// * q is split into four byte limbs, q = sum_k 2^(8k) q_k, so that
//   a = sum_k 2^(8k) (D q_k).  Each D q_k is a sum of byte x byte products,
//   one v_dot4_u32_u8 per four database bytes and limb, plus a shift-add
//   per limb every 16 bytes: ~1.25 VALU lane-ops per database byte, far
//   under the ~4.9 the CUs can spend at full HBM rate.  All arithmetic
//   wraps modulo 2^32, which is all the answer needs.
// * A workgroup (WV waves) stages a slice of kSlice query words in LDS as the
//   four limb planes (split once per workgroup, not per wave).
// * Each wave owns RW database rows.  One wave-wide 16-byte load covers 1024
//   contiguous bytes of a row (fully coalesced); the RW row loads of a chunk
//   are issued back to back so RW KiB per wave are in flight, those of a
//   slice's first chunk before the slice's query words are staged.  The
//   stream is read with non-temporal loads.
// * Rows may start at any address and have any length: loads of 16 bytes
//   need no alignment on gfx950.  (20000 x 10007 unaligned bytes, the same
//   buffers on every call: 452 us byte by byte, 41.2 us so, and 33.6 us when
//   the rows are padded to an aligned pitch; with other inputs on every call
//   531 and 41.7 us.)
// * After the column loop each lane holds RW partial sums; they are
//   transposed through LDS and finished with lane shuffles, so one lane per
//   row writes the result.
// * Shapes with too few row blocks to fill the chip split the columns; the
//   per-split partial sums go to the workspace and a second kernel adds
//   them (integer addition modulo 2^32 is exact in any order).
#include <type_traits>

#include "qpir_internal.h"

namespace {

constexpr int kChunk = 1024;   // columns covered by one wave-wide 16-byte load
constexpr int kSlice = 4096;   // query words staged in LDS at a time

// Four consecutive query words -> the four limb words; limb k holds byte k
// of each word, the first word in the low byte.
__device__ inline void limbs_of4(uint32_t x0, uint32_t x1, uint32_t x2, uint32_t x3,
                                 uint32_t out[4]) {
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const int sh = 8 * k;
        out[k] = ((x0 >> sh) & 0xFFu) | (((x1 >> sh) & 0xFFu) << 8) |
                 (((x2 >> sh) & 0xFFu) << 16) | (((x3 >> sh) & 0xFFu) << 24);
    }
}

// 16 bytes at any alignment (gfx950 serves unaligned global accesses; one
// wave-wide load of 1024 consecutive bytes then touches nine lines, not
// eight).
typedef u32x4 u32x4_any __attribute__((aligned(1)));
typedef u32x4 u32x4_word __attribute__((aligned(4)));

__device__ inline u32x4 load_stream(const uint8_t* p) {
    return __builtin_nontemporal_load(reinterpret_cast<const u32x4_any*>(p));
}

// Chunk loads of RW rows of C >= 16 bytes: the 16 bytes at column c of each
// (c = chunk + 16 lane), or at C - 16 for lanes past that.
template <int RW>
__device__ inline void load_chunk(u32x4 (&d)[RW], const uint8_t* const (&rp)[RW], uint32_t c,
                                  uint32_t C) {
    const uint32_t at = min(c, C - 16u);
#pragma unroll
    for (int i = 0; i < RW; ++i) d[i] = load_stream(rp[i] + at);
}

// In a row's ragged last chunk, move the bytes of the one lane whose 16
// bytes cross the end into place.  (Lanes past the end hold anything: they
// meet zero limbs.)  Rows of whole 16-byte pieces have no such lane.
template <int RW>
__device__ inline void align_tail(u32x4 (&d)[RW], uint32_t c, uint32_t C) {
    const uint32_t sh = 8u * min(c - min(c, C - 16u), 15u);
#pragma unroll
    for (int i = 0; i < RW; ++i) {
        uint64_t lo = (uint64_t)d[i].x | ((uint64_t)d[i].y << 32);
        uint64_t hi = (uint64_t)d[i].z | ((uint64_t)d[i].w << 32);
        if (sh >= 64u) {
            lo = hi >> (sh - 64u);
        } else if (sh != 0u) {
            lo = (lo >> sh) | (hi << (64u - sh));
            hi >>= sh;
        }
        d[i] = u32x4{(uint32_t)lo, (uint32_t)(lo >> 32), (uint32_t)hi, (uint32_t)(hi >> 32)};
    }
}

// 16 database bytes times the matching 16 query words, mod 2^32: per limb k
// a chain of four dot4 products (at most 16 * 255 * 255 < 2^21, exact), then
// sum_k 2^(8k) p_k.  Combining per chunk keeps one accumulator per row.
__device__ inline uint32_t dot16(const u32x4 d, const u32x4 L[4]) {
    uint32_t p[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        uint32_t a = __builtin_amdgcn_udot4(d.x, L[k].x, 0u, false);
        a = __builtin_amdgcn_udot4(d.y, L[k].y, a, false);
        a = __builtin_amdgcn_udot4(d.z, L[k].z, a, false);
        p[k] = __builtin_amdgcn_udot4(d.w, L[k].w, a, false);
    }
    return p[0] + (p[1] << 8) + (p[2] << 16) + (p[3] << 24);
}

template <int RW, int WV>
__global__ __launch_bounds__(64 * WV) void k_answer1(const uint8_t* __restrict__ D, uint64_t pitch,
                                                     uint32_t R, uint32_t C,
                                                     const uint32_t* __restrict__ q,
                                                     uint32_t* __restrict__ out,
                                                     uint32_t cols_per_split) {
    // Loads ahead of the staging.  32 rows' loads held across it cost more
    // registers than they gain (32768 x 32768: 165 us against 158 us).
    constexpr bool kAhead = RW <= 16;
    __shared__ u32x4 s_limb[4][kSlice / 16];
    __shared__ uint32_t s_red[WV][RW][65];

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    // Wave-uniform, so the row addresses live in scalar registers.
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const uint32_t row0 = (blockIdx.x * WV + wave) * RW;
    const uint32_t cb = blockIdx.y * cols_per_split;
    const uint32_t ce = min(C, cb + cols_per_split);

    // Rows past the end re-read the last row; their sums are never stored.
    const uint8_t* rp[RW];
#pragma unroll
    for (int i = 0; i < RW; ++i) {
        const uint32_t r = min(row0 + (uint32_t)i, R - 1);
        rp[i] = D + (uint64_t)r * pitch;
    }

    uint32_t acc[RW];
#pragma unroll
    for (int i = 0; i < RW; ++i) acc[i] = 0;

    if (C < 16u) {   // shorter than a load: lane e takes column e
        if ((uint32_t)lane < C) {
#pragma unroll
            for (int i = 0; i < RW; ++i) acc[i] = (uint32_t)rp[i][lane] * q[lane];
        }
    } else for (uint32_t s0 = cb; s0 < ce; s0 += kSlice) {
        const uint32_t se = min(ce, s0 + (uint32_t)kSlice);
        u32x4 d[RW];
        if (kAhead) load_chunk<RW>(d, rp, s0 + 16u * lane, C);
        __syncthreads();   // previous slice fully consumed
        // Limbs of the slice's words, zero past its end up to a whole chunk.
        const uint32_t groups = (se - s0 + kChunk - 1) / kChunk * (kChunk / 16);
        for (int t = tid; t < kSlice / 16; t += 64 * WV) {
            if ((uint32_t)t >= groups) break;
            const uint32_t c = s0 + 16u * t;
            uint32_t x[16];
            if (c + 16 <= se) {
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const u32x4 w = *reinterpret_cast<const u32x4_word*>(q + c + 4 * v);
                    x[4 * v + 0] = w.x;
                    x[4 * v + 1] = w.y;
                    x[4 * v + 2] = w.z;
                    x[4 * v + 3] = w.w;
                }
            } else {
#pragma unroll
                for (int e = 0; e < 16; ++e) x[e] = (c + e < se) ? q[c + e] : 0u;
            }
            uint32_t l[4][4];
#pragma unroll
            for (int w = 0; w < 4; ++w) {
                uint32_t o[4];
                limbs_of4(x[4 * w], x[4 * w + 1], x[4 * w + 2], x[4 * w + 3], o);
#pragma unroll
                for (int k = 0; k < 4; ++k) l[k][w] = o[k];
            }
#pragma unroll
            for (int k = 0; k < 4; ++k) s_limb[k][t] = u32x4{l[k][0], l[k][1], l[k][2], l[k][3]};
        }
        __syncthreads();

        for (uint32_t c0 = s0; c0 < se; c0 += kChunk) {
            const uint32_t c = c0 + 16u * lane;
            u32x4 L[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) L[k] = s_limb[k][(c0 - s0) / 16 + lane];
            if (!kAhead && c0 + kChunk <= se) {
                // A whole chunk's loads and products, interleaved.
#pragma unroll
                for (int i = 0; i < RW; ++i) d[i] = load_stream(rp[i] + c);
#pragma unroll
                for (int i = 0; i < RW; ++i) acc[i] += dot16(d[i], L);
                asm volatile("");   // keep the two branches' products apart
            } else {
                if (!kAhead || c0 != s0) load_chunk<RW>(d, rp, c, C);
                if (C % 16u != 0u && c0 + kChunk > C) align_tail<RW>(d, c, C);
#pragma unroll
                for (int i = 0; i < RW; ++i) acc[i] += dot16(d[i], L);
            }
        }
    }

    // Sum the 64 lanes of each row.
#pragma unroll
    for (int i = 0; i < RW; ++i) s_red[wave][i][lane] = acc[i];
    __syncthreads();
    constexpr int kLanesPerRow = 64 / RW;
    const int i = lane / kLanesPerRow;
    const int part = lane % kLanesPerRow;
    uint32_t v = 0;
#pragma unroll
    for (int t = 0; t < RW; ++t) v += s_red[wave][i][part * RW + t];
#pragma unroll
    for (int off = 1; off < kLanesPerRow; off <<= 1) v += __shfl_xor(v, off);
    const uint32_t r = row0 + (uint32_t)i;
    if (part == 0 && r < R) out[(uint64_t)blockIdx.y * R + r] = v;
}

__global__ void k_sum_splits(const uint32_t* __restrict__ part, uint32_t R, uint32_t S,
                             uint32_t* __restrict__ out) {
    const uint32_t r = blockIdx.x * blockDim.x + threadIdx.x;
    if (r >= R) return;
    uint32_t v = 0;
    for (uint32_t s = 0; s < S; ++s) v += part[(uint64_t)s * R + r];
    out[r] = v;
}

struct SplitPlan {
    uint32_t splits;
    uint32_t cols_per_split;
};

// Split the columns into `s` pieces, of at least `min_cols` columns each and
// whole chunks (splits cost a second launch, about 2 us, and their partials).
SplitPlan plan_splits(const pir_db_t* db, uint64_t s, uint32_t min_cols) {
    s = std::min<uint64_t>(s, (db->cols + min_cols - 1) / min_cols);
    if (s < 1) s = 1;
    uint64_t cps = ((db->cols + s - 1) / s + kChunk - 1) / kChunk * kChunk;
    s = (db->cols + cps - 1) / cps;
    return SplitPlan{(uint32_t)s, (uint32_t)cps};
}

uint64_t row_blocks(const pir_db_t* db, uint32_t rows_per_block) {
    return (db->rows + rows_per_block - 1) / rows_per_block;
}

// Single query.  Blocks of 64 rows and more run long, so the splits even out
// the workgroups over the 256 CUs: the least of (rounds of workgroups) times
// (whole chunks of a piece, and half a chunk's time to start) plus a tenth per
// piece for its partials; up to 16 pieces, or one per CU for fewer than 16
// blocks.  Eight waves of 8 rows, us: 3072 x 2^18, 48 blocks: 6 splits 163,
// 16 splits 129; 12288 x 40000, 192 blocks: not split 90, 4 splits 83; 6736 x
// 21568, 106 blocks: 2 splits 31, 8 splits 28; 64 x 2^22, one block: 16
// splits 383, 128 splits 98.  Over 30 random shapes the pieces so chosen take
// 0.9% more than the best count of each.  Smaller blocks only split where
// there are fewer than four per CU (1024 x 65536, two rows per wave: 8 splits
// 16.2, not split 52; 2048 x 3001: not split 6.0, two 7.0).
SplitPlan answer1_plan(const pir_db_t* db, uint32_t rows_per_block) {
    const uint64_t blocks = row_blocks(db, rows_per_block);
    if (rows_per_block < 64) return plan_splits(db, 1024 / blocks, kSlice);
    const uint64_t chunks = (db->cols + kChunk - 1) / kChunk;
    const uint64_t most = std::min(chunks, std::max<uint64_t>(16, 256 / blocks));
    uint64_t best = chunks, best_t = ~0ull;   // chunks of a piece; time in twentieths of a chunk
    for (uint64_t s = 1; s <= most; ++s) {
        const uint64_t each = (chunks + s - 1) / s, pieces = (chunks + each - 1) / each;
        const uint64_t t = (blocks * pieces + 255) / 256 * (20 * each + 10) + 2 * pieces;
        if (t < best_t) {
            best_t = t;
            best = each;
        }
    }
    return SplitPlan{(uint32_t)((chunks + best - 1) / best), (uint32_t)(best * kChunk)};
}

size_t split_bytes(const pir_db_t* db, const SplitPlan& p) {
    return p.splits > 1 ? round_up((size_t)p.splits * db->rows * 4, kWsAlign) : 0;
}

template <int RW, int WV>
pir_status launch_answer1(const pir_db_t* db, const uint32_t* q, uint32_t* a, void* ws,
                          size_t ws_bytes, hipStream_t s) {
    constexpr uint32_t kRows = RW * WV;
    const SplitPlan p = answer1_plan(db, kRows);
    const uint32_t R = (uint32_t)db->rows, C = (uint32_t)db->cols;
    uint32_t* dst = a;
    if (p.splits > 1) {
        if (!ws || ws_bytes < split_bytes(db, p) || ((uintptr_t)ws % kWsAlign))
            return PIR_ERR_WORKSPACE;
        dst = static_cast<uint32_t*>(ws);
    }
    dim3 grid((R + kRows - 1) / kRows, p.splits);
    k_answer1<RW, WV><<<grid, 64 * WV, 0, s>>>(db->D, db->pitch, R, C, q, dst, p.cols_per_split);
    PIR_LAUNCH_CHECK();
    if (p.splits > 1) {
        k_sum_splits<<<(R + 255) / 256, 256, 0, s>>>(dst, R, p.splits, a);
        PIR_LAUNCH_CHECK();
    }
    return PIR_OK;
}

struct GemvVariant {
    const char* name;
    uint32_t rows_per_block, threads;
    pir_status (*launch)(const pir_db_t*, const uint32_t*, uint32_t*, void*, size_t, hipStream_t);
};

const GemvVariant kGemv[] = {
    {"auto", 0, 0, nullptr},
    {"rows16", 64, 256, launch_answer1<16, 4>},
    {"rows8", 32, 256, launch_answer1<8, 4>},
    {"rows32", 128, 256, launch_answer1<32, 4>},
    {"rows8w8", 64, 512, launch_answer1<8, 8>},
    {"rows4", 16, 256, launch_answer1<4, 4>},
    {"rows2", 8, 256, launch_answer1<2, 4>},
};
constexpr uint32_t kNumGemv = sizeof(kGemv) / sizeof(kGemv[0]);
constexpr uint32_t kGemvShort = 2, kGemvLong = 3, kGemvLarge = 4, kGemvMid = 5, kGemvSmall = 6;

// Built-in choice.  Few rows per wave and many short workgroups fill the chip
// evenly while the rows give whole rounds of workgroups on the 256 CUs; where
// they do not (one workgroup in four rounds for a CU, three for most), and on
// larger databases, eight waves of 8 rows with split columns come out even.
// Short rows pay a wave's start and end per row, so they take more rows a
// wave; databases of at most 512 rows only fill the chip by splitting their
// columns, where few rows a wave leave most pieces to split.  GPU us with the
// splits of answer1_plan (200 random shapes, 2^22 to 2^30 bytes: 1.3% over the
// fastest kernel of each in the geometric mean):
//                    rows16  rows32  rows8w8  rows8  rows4   rows2
//   300 x 1000000     117     194     110      78     67      64
//   2048 x 3001        9.3    16.2     8.6     6.9    5.9     5.1
//   4096 x 4096        9.2    13.7     7.8     6.7    6.6     6.1
//   8192 x 8192       16.5    18.2    15.1    16.3   14.2    14.6
//   4352 x 42752      35.1    35.5    33.5    35.1   37.5    47.2
//   6320 x 24320      28.3    27.9    27.5    28.4   31.5    32.0
//   72880 x 256       11.2    13.5    11.4    10.3   11.9    15.7
//   333824 x 512      37.4    48.4    39.6    38.3   47.1    66.9
//   20000 x 10007     46.2    48.8    45.0    47.3   41.8    45.5
//   262144 x 2048     84.5    79.7    84.4    77.0   75.9    78.7
//   8192 x 65536      87.1    88.3    87.7    86.4   86.2    95.1
//   32768 x 32768    162     158     162       -    186     178
//   131072 x 131072 2483    2408    2460       -   2524    2536
// A grid holds fewer than 2^32 threads: databases of more rows than the choice
// covers so take the tile of the most rows per thread.
constexpr uint64_t kGemvEven = 3ull << 24, kGemvBig = 3ull << 26, kGemvHuge = 1ull << 28;

uint32_t gemv_by_size(const pir_db_t* db) {
    const uint64_t R = db->rows, C = db->cols, bytes = R * C;
    if (R <= 512) return kGemvSmall;
    if (R >= 12000) {
        if (C < 1280) return kGemvShort;
        if (bytes < kGemvHuge || C <= 2048) return kGemvMid;
        return R >= 32768 && C >= 32768 ? kGemvLong : kGemvLarge;
    }
    if (bytes >= kGemvBig) return kGemvLarge;
    const uint64_t wgs = row_blocks(db, kGemv[kGemvSmall].rows_per_block) *
                         answer1_plan(db, kGemv[kGemvSmall].rows_per_block).splits;
    const uint64_t even = (wgs + 255) / 256 * 256;   // what as many rounds could hold
    return bytes >= kGemvEven && 20 * even > 21 * wgs ? kGemvLarge : kGemvSmall;
}

uint32_t gemv_auto(const pir_db_t* db) {
    const uint32_t v = gemv_by_size(db);
    return row_blocks(db, kGemv[v].rows_per_block) * kGemv[v].threads < (1ull << 32) ? v : kGemvLong;
}

// ---------------------------------------------------------------- few queries
// Batches of at most 4 queries (and the field form's single query): the same
// stream over D as k_answer1, with the limb planes of NQ queries staged in
// LDS and NQ accumulators per row, so D is read once for the whole batch.
// On the matrix cores a batch is padded to 32 queries (128 limb rows), so
// for NQ <= 4 this stream is the faster route: per 16 database bytes and
// query it costs 16 dot4 plus a combine, 1.2 VALU lane-ops per byte and
// query against the ~4.9 the CUs can spend at full HBM rate.
//
// EXACT (field form): each chunk's combined limb products are below 2^45
// (four dot4 chains of at most 16 * 255 * 255 < 2^21, shifted by 8k) and are
// added into 64-bit accumulators; D q < 2^63 for C <= 2^23, so the sum is
// the exact integer, reduced mod p once at the end.
constexpr int kFewSlice = 2048;   // query words per LDS stage

// Outputs of one workgroup row: the answer itself when one split covers all
// columns (output element (r, b) at out[r * o_ldr + b * o_ldb], reduced mod p
// in the field form), else a partial for k_few_finish.
struct FewOut {
    uint32_t* out;
    uint64_t o_ldr, o_ldb;
    uint32_t p;
    void* part;
};

template <int NQ, int RW, int WV, bool EXACT>
__global__ __launch_bounds__(64 * WV) void k_answer_few(
    const uint8_t* __restrict__ D, uint64_t pitch, uint32_t R, uint32_t C,
    const uint32_t* __restrict__ Q, uint64_t ldj, uint64_t ldb, uint32_t B,
    uint32_t cols_per_split, FewOut o) {
    typedef typename std::conditional<EXACT, uint64_t, uint32_t>::type acc_t;
    __shared__ u32x4 s_limb[NQ][4][kFewSlice / 16];
    __shared__ acc_t s_red[WV][RW][65];

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const uint32_t row0 = (blockIdx.x * WV + wave) * RW;
    const uint32_t cb = blockIdx.y * cols_per_split;
    const uint32_t ce = min(C, cb + cols_per_split);

    const uint8_t* rp[RW];
#pragma unroll
    for (int i = 0; i < RW; ++i) {
        const uint32_t r = min(row0 + (uint32_t)i, R - 1);
        rp[i] = D + (uint64_t)r * pitch;
    }
    acc_t acc[RW][NQ];
#pragma unroll
    for (int i = 0; i < RW; ++i)
#pragma unroll
        for (int b = 0; b < NQ; ++b) acc[i][b] = 0;

    if (C < 16u) {   // shorter than a load: lane e takes column e
        if ((uint32_t)lane < C) {
#pragma unroll
            for (int b = 0; b < NQ; ++b) {
                const uint32_t x = (uint32_t)b < B ? Q[(uint64_t)lane * ldj + (uint64_t)b * ldb] : 0u;
#pragma unroll
                for (int i = 0; i < RW; ++i) acc[i][b] = (acc_t)rp[i][lane] * x;
            }
        }
    } else for (uint32_t s0 = cb; s0 < ce; s0 += kFewSlice) {
        const uint32_t se = min(ce, s0 + (uint32_t)kFewSlice);
        u32x4 d[RW];
        // 16 rows' loads held across the staging would cost occupancy.
        if (RW <= 8) load_chunk<RW>(d, rp, s0 + 16u * lane, C);
        __syncthreads();   // previous slice fully consumed
        for (int t = tid; t < NQ * (kFewSlice / 16); t += 64 * WV) {
            const int b = t / (kFewSlice / 16);
            const int g = t % (kFewSlice / 16);
            const uint32_t c = s0 + 16u * g;
            uint32_t x[16];
#pragma unroll
            for (int e = 0; e < 16; ++e)
                x[e] = ((uint32_t)b < B && c + e < se) ? Q[(uint64_t)(c + e) * ldj + (uint64_t)b * ldb]
                                                       : 0u;
            uint32_t l[4][4];
#pragma unroll
            for (int w = 0; w < 4; ++w) {
                uint32_t o4[4];
                limbs_of4(x[4 * w], x[4 * w + 1], x[4 * w + 2], x[4 * w + 3], o4);
#pragma unroll
                for (int k = 0; k < 4; ++k) l[k][w] = o4[k];
            }
#pragma unroll
            for (int k = 0; k < 4; ++k) s_limb[b][k][g] = u32x4{l[k][0], l[k][1], l[k][2], l[k][3]};
        }
        __syncthreads();

        for (uint32_t c0 = s0; c0 < se; c0 += kChunk) {
            const uint32_t li = (c0 - s0) / 16 + lane;
            if (RW > 8 || c0 != s0) load_chunk<RW>(d, rp, c0 + 16u * lane, C);
            if (C % 16u != 0u && c0 + kChunk > C) align_tail<RW>(d, c0 + 16u * lane, C);
#pragma unroll
            for (int b = 0; b < NQ; ++b) {
                u32x4 L[4];
#pragma unroll
                for (int k = 0; k < 4; ++k) L[k] = s_limb[b][k][li];
#pragma unroll
                for (int i = 0; i < RW; ++i) {
                    if (EXACT) {
                        uint32_t p[4];
#pragma unroll
                        for (int k = 0; k < 4; ++k) {
                            uint32_t a = __builtin_amdgcn_udot4(d[i].x, L[k].x, 0u, false);
                            a = __builtin_amdgcn_udot4(d[i].y, L[k].y, a, false);
                            a = __builtin_amdgcn_udot4(d[i].z, L[k].z, a, false);
                            p[k] = __builtin_amdgcn_udot4(d[i].w, L[k].w, a, false);
                        }
                        acc[i][b] += (uint64_t)p[0] + ((uint64_t)p[1] << 8) +
                                     ((uint64_t)p[2] << 16) + ((uint64_t)p[3] << 24);
                    } else {
                        acc[i][b] += dot16(d[i], L);
                    }
                }
            }
        }
    }

    // Sum the 64 lanes of each (row, query); one query at a time through LDS.
    constexpr int kLanesPerRow = 64 / RW;
    const int i = lane / kLanesPerRow;
    const int prt = lane % kLanesPerRow;
    const uint32_t r = row0 + (uint32_t)i;
#pragma unroll
    for (int b = 0; b < NQ; ++b) {
        __syncthreads();
#pragma unroll
        for (int t = 0; t < RW; ++t) s_red[wave][t][lane] = acc[t][b];
        __syncthreads();
        acc_t v = 0;
#pragma unroll
        for (int t = 0; t < RW; ++t) v += s_red[wave][i][prt * RW + t];
#pragma unroll
        for (int off = 1; off < kLanesPerRow; off <<= 1) v += __shfl_xor(v, off);
        if (prt != 0 || r >= R || (uint32_t)b >= B) continue;
        if (o.part)
            static_cast<acc_t*>(o.part)[((uint64_t)blockIdx.y * B + b) * R + r] = v;
        else
            o.out[(uint64_t)r * o.o_ldr + (uint64_t)b * o.o_ldb] =
                EXACT ? (uint32_t)(v % o.p) : (uint32_t)v;
    }
}

// Sum of the column splits; the field form reduces mod p.  Output element
// (r, b) goes to out[r * o_ldr + b * o_ldb].
template <bool EXACT>
__global__ void k_few_finish(const void* __restrict__ part, uint32_t R, uint32_t B, uint32_t S,
                             uint32_t p, uint32_t* __restrict__ out, uint64_t o_ldr,
                             uint64_t o_ldb) {
    const uint64_t idx = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= (uint64_t)R * B) return;
    const uint32_t b = (uint32_t)(idx / R), r = (uint32_t)(idx % R);
    uint32_t* dst = out + (uint64_t)r * o_ldr + (uint64_t)b * o_ldb;
    if (EXACT) {
        uint64_t v = 0;
        for (uint32_t s = 0; s < S; ++s)
            v += static_cast<const uint64_t*>(part)[((uint64_t)s * B + b) * R + r];
        *dst = (uint32_t)(v % p);
    } else {
        uint32_t v = 0;
        for (uint32_t s = 0; s < S; ++s)
            v += static_cast<const uint32_t*>(part)[((uint64_t)s * B + b) * R + r];
        *dst = v;
    }
}

uint32_t few_nq(uint32_t B) { return B <= 1 ? 1u : (B <= 2 ? 2u : 4u); }

// Rows per workgroup and column splits.  The limb planes of NQ queries are
// staged for a workgroup's rows, so it takes 64 (four waves of 16) and splits
// to three workgroups per CU; 256 blocks of short rows stay whole.  Small
// databases of few rows leave too few such workgroups, and take 16 rows (four
// waves of 4), whole up to one slice of columns: a split's second launch costs
// more than the staging.  Two queries stage twice as much, so they take 64
// rows from half the size, except on a thousand rows or fewer, which would be
// cut into too many pieces.  GPU us for one / two / four queries, best splits:
//                  16 rows            64 rows
//   1024 x 1024     3.5  4.5   6.4     4.5   5.7   9.2
//   2048 x 3001     7.2  9.0  12.4    10.4  13.0  18.7
//   4096 x 4096     8.9 10.7  16.9     7.9   9.3  12.7  (four splits)
//   3072 x 8192    10.4 15.4  21.5    10.0  12.1  17.5
//   3000 x 11008   13.1 19.5  28.5    12.2  14.1  21.0
//   200 x 100000   17.0 22.3  29.4    19.9 24.0  30.3
//   16384 x 1500    8.9 13.6  19.6     8.0  10.1  15.1  (whole)
//   100000 x 160   17.1 24.4  43.4    14.2  18.7  36.9  (whole)
//   8192 x 8192    18.1 29.1  44.9    15.9  18.9  27.9
uint32_t few_rows(const pir_db_t* db, uint32_t B) {
    const uint64_t bytes = db->rows * db->cols;
    const bool small = db->rows < 16384u && (B == 1u || db->rows <= 1024u ? bytes < (1ull << 25)
                                                                          : bytes <= (1ull << 24));
    return B <= 2u && small ? 16u : 64u;
}

SplitPlan few_plan(const pir_db_t* db, uint32_t B) {
    const uint32_t rows = few_rows(db, B);
    const uint64_t blocks = row_blocks(db, rows);
    // Short rows stay whole: of one slice in blocks of 16 rows, of two chunks in
    // 256 and more blocks of 64 (17784 x 2343, two field queries: two pieces
    // 24.8 us, whole 28.2).
    if (db->cols <= (rows == 16u ? (uint64_t)kSlice : blocks >= 256u ? 2u * kChunk : 0u))
        return plan_splits(db, 1, kChunk);
    if (rows == 64u) return plan_splits(db, 768 / blocks, kChunk);
    // Up to eight pieces of half a slice for at most a block per CU, beyond only
    // of whole slices (200 x 100000, one query: 25 pieces 17 us, 49 pieces 21;
    // 6144 x 4352, 384 blocks: whole 13.4, two pieces 14.9).
    const uint64_t halves = blocks <= 256u ? std::min<uint64_t>(768 / blocks, 8) : 1;
    const SplitPlan half = plan_splits(db, halves, kSlice / 2);
    const SplitPlan whole = plan_splits(db, 512 / blocks, kSlice);
    return half.splits > whole.splits ? half : whole;
}

// Whether a call's answers and queries share memory.  An unsplit launch
// would overwrite queries that other workgroups still read.
bool few_overlap(const pir_db_t* db, const BatchIO& io, uint32_t B) {
    const uint64_t q_words = (db->cols - 1) * io.q_ldj + (uint64_t)(B - 1) * io.q_ldb + 1;
    const uint64_t o_words = (db->rows - 1) * io.o_ldr + (uint64_t)(B - 1) * io.o_ldb + 1;
    const uintptr_t q = (uintptr_t)io.Q, o = (uintptr_t)io.out;
    return q < o + 4 * o_words && o < q + 4 * q_words;
}

template <int NQ, int RW, int WV, bool EXACT>
pir_status launch_few_t(const pir_db_t* db, const BatchIO& io, uint32_t B, uint32_t modulus,
                        void* ws, hipStream_t s) {
    constexpr uint32_t kRows = RW * WV;
    const SplitPlan pl = few_plan(db, B);
    const uint32_t R = (uint32_t)db->rows, C = (uint32_t)db->cols;
    dim3 grid((R + kRows - 1) / kRows, pl.splits);
    const bool partials = pl.splits > 1 || few_overlap(db, io, B);
    const FewOut o{io.out, io.o_ldr, io.o_ldb, modulus, partials ? ws : nullptr};
    k_answer_few<NQ, RW, WV, EXACT><<<grid, 64 * WV, 0, s>>>(
        db->D, db->pitch, R, C, io.Q, io.q_ldj, io.q_ldb, B, pl.cols_per_split, o);
    PIR_LAUNCH_CHECK();
    if (!partials) return PIR_OK;
    const uint64_t n = (uint64_t)R * B;
    k_few_finish<EXACT><<<(uint32_t)((n + 255) / 256), 256, 0, s>>>(
        ws, R, B, pl.splits, modulus, io.out, io.o_ldr, io.o_ldb);
    PIR_LAUNCH_CHECK();
    return PIR_OK;
}

template <int NQ, bool EXACT>
pir_status launch_few(const pir_db_t* db, const BatchIO& io, uint32_t B, uint32_t modulus,
                      void* ws, hipStream_t s) {
    if constexpr (NQ <= 2) {
        if (few_rows(db, B) == 16u) return launch_few_t<NQ, 4, 4, EXACT>(db, io, B, modulus, ws, s);
    }
    return launch_few_t<NQ, 16, 4, EXACT>(db, io, B, modulus, ws, s);
}

}  // namespace

FewPlan few_batch_plan(const pir_db_t* db, uint32_t B) {
    return {few_rows(db, B), few_plan(db, B).splits};
}

size_t few_workspace_bytes(const pir_db_t* db, uint32_t B) {
    if (B == 0 || B > kFewMax) return 0;
    const SplitPlan pl = few_plan(db, B);
    return round_up((size_t)pl.splits * B * db->rows * 8, kWsAlign);
}

pir_status few_answer_batch(const pir_db_t* db, const BatchIO& io, uint32_t B, uint32_t modulus,
                            void* ws, size_t ws_bytes, hipStream_t s) {
    if (B == 0) return PIR_OK;
    if (B > kFewMax) return PIR_ERR_SHAPE;
    if (!ws || ws_bytes < few_workspace_bytes(db, B) || ((uintptr_t)ws % kWsAlign))
        return PIR_ERR_WORKSPACE;
    const bool exact = modulus != 0;
    switch (few_nq(B)) {
        case 1: return exact ? launch_few<1, true>(db, io, B, modulus, ws, s)
                             : launch_few<1, false>(db, io, B, modulus, ws, s);
        case 2: return exact ? launch_few<2, true>(db, io, B, modulus, ws, s)
                             : launch_few<2, false>(db, io, B, modulus, ws, s);
        default: return exact ? launch_few<4, true>(db, io, B, modulus, ws, s)
                              : launch_few<4, false>(db, io, B, modulus, ws, s);
    }
}

uint32_t gemv_variant_count() { return kNumGemv; }

const char* gemv_variant_name(uint32_t v) { return v < kNumGemv ? kGemv[v].name : nullptr; }

// Both depend on the shape only; choosing and sizing them on every call took
// up to 3 us of a call's host time.  The workspace is enough for every
// variant, so one sized once serves any tuning.
void gemv_open(pir_db_t* db) {
    db->answer_variant = gemv_auto(db);
    db->answer_ws = 0;
    for (uint32_t v = 1; v < kNumGemv; ++v)
        db->answer_ws = std::max(db->answer_ws, split_bytes(db, answer1_plan(db, kGemv[v].rows_per_block)));
}

size_t gemv_workspace_bytes(const pir_db_t* db) { return db->answer_ws; }

static uint32_t gemv_choice(const pir_db_t* db) {
    const uint32_t v = db->variant[0];
    return v == 0 || v >= kNumGemv ? db->answer_variant : v;
}

GemvPlan gemv_plan(const pir_db_t* db) {
    const uint32_t v = gemv_choice(db), rows = kGemv[v].rows_per_block;
    return {v, (uint32_t)row_blocks(db, rows), answer1_plan(db, rows).splits, kGemv[v].threads};
}

pir_status gemv_answer(const pir_db_t* db, const uint32_t* q, uint32_t* a, void* ws,
                       size_t ws_bytes, hipStream_t s) {
    return kGemv[gemv_choice(db)].launch(db, q, a, ws, ws_bytes, s);
}
