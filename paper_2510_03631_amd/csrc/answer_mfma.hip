// Batched Answer and offline hint on the int8 matrix cores.
//
//   Out[r][b] = sum_j D[r][j] * Q[j][b]   mod 2^32   (LWE form)
//   Out[r][b] = sum_j D[r][j] * Q[j][b]   mod p      (field form, p < 2^32)
//
// The LWE form is the multi-request response of Section 5.2 (Algorithm 4's
// batched product, here over Z/2^32); the hint H = D A is the same product
// with A in place of Q (Section 5.3's offline work).  The field form is the
// server product of the Goldberg / FTR instantiation (Section 5.1), the
// "mod q" of Algorithm 4.
//
// gfx950 has only signed int8 matrix instructions, so both operands are
// centred.  With q = sum_k 2^(8k) q_k (byte limbs), q_k = q'_k + 128 and
// D = D' + 128 (D' = D xor 0x80 read as int8, likewise q'_k), over the
// integers:
//
//   D q = sum_k 2^(8k) (D' q'_k)  +  128 (colsum(q) - C * 0x80808080)
//                                 +  0x80808080 rowsum(D)
//
// One int8 GEMM with M = R, K = C and N = 4 * B (the four limb planes of
// every query side by side) gives the products P_k = D' q'_k; the epilogue
// adds P_0 + 2^8 P_1 + 2^16 P_2 + 2^24 P_3 and the two terms (column sums
// from the ingest kernel, row sums from the database handle).
// * Modulo 2^32 the int32 accumulators wrap freely: only residues are used.
// * The field form rebuilds D q exactly, modulo 2^64 (D q < 2^64 for
//   C <= 2^23), and reduces it mod p.  A product P_k over K <= 2^17 columns
//   lies in [-16256 K, 16384 K]: the int32 accumulator holds it exactly
//   except for +2^31 (all products (-128)(-128) with K = 2^17), which reads
//   back as -2^31, a value the true sum cannot take, and is mapped back.  So
//   every accumulation in the field form covers at most 2^17 columns; longer
//   rows are split along K (below).
//
// Split-K.  When the output tiles cannot fill the chip (few rows: the
// incremental hint, short databases), or the field form needs it, the K
// range is cut into S pieces; each workgroup writes its piece's limb
// combination as a partial (4 bytes mod 2^32, or 8 bytes exact) and a
// finishing kernel adds the S partials and the centring terms.
//
// Kernels
//   k_zero_words  clear the column sums, where the ingest sums
//   k_ingest      Q -> QL (N x Cp centred int8, K-contiguous) and, unless
//                 the tiles sum for themselves (tile_sums), exact 64-bit
//                 colsum[b] = sum_j Q[j][b]
//   k_gemm_ring   int8 MFMA 32x32x32; global tiles go straight to LDS
//                 (global_load_lds_dwordx4) into a ring of stages; fused
//                 epilogue, optional row gather, optional split-K
//   k_gemm_roles  the same with separate loader waves for D and QL
//   k_gemm        register-staged LDS tiles, two buffers, for databases the
//                 ring cannot serve (rows not 16-byte aligned)
//   k_finish      sums split-K partials and adds the centring terms
//                 (k_finish4, k_finish_rows: four outputs a thread)
//
// QL row index of (query b, limb k): n = (b / 32) * 128 + k * 32 + (b % 32),
// so the four limbs of a query land in the same lane of four adjacent 32x32
// output tiles and the epilogue combines them in registers.  Batches of at
// most 16 queries may use the narrow layout n = (b / 8) * 32 + k * 8 + b % 8
// instead: one 32-column tile holds all four limbs of 8 queries, so a batch
// of 8 is not padded to 32 queries; the epilogue then combines the limbs
// of a query across lanes c, c+8, c+16, c+24 with two shuffles.  QL is stored in
// 4 KiB tiles of 32 rows x 128 bytes (tile (n/32, k/128) at
// ((n/32) * Cp/128 + k/128) * 4096, row n%32 at 128 (n%32) within it): the
// ingest writes whole tiles and a 1 KiB block of a GEMM k-tile is contiguous.
#include <algorithm>
#include <cmath>
#include <iterator>
#include <type_traits>

#include "qpir_internal.h"

namespace {

typedef int i32x4 __attribute__((ext_vector_type(4)));
typedef int i32x16 __attribute__((ext_vector_type(16)));
typedef __attribute__((address_space(3))) void lds_void_t;
typedef __attribute__((address_space(1))) void glb_void_t;
typedef unsigned long long u64;

constexpr uint32_t kCentreWord = 0x80808080u;
constexpr int kCpolNT = 2;   // cache-policy operand of a load: nt (non-temporal) on gfx950
constexpr int kKPad = 256;                    // QL rows are zero-padded to a multiple of this
constexpr uint32_t kExactSpan = 1u << 17;     // columns one exact int32 accumulation may cover
constexpr uint32_t kMaxExactCols = 1u << 23;  // D q < 2^64 and exact row sums
constexpr uint32_t kMaxSplits = 64;           // split-K pieces chosen for occupancy


// Epilogue modes.
enum : int {
    kFinal32 = 0,     // Out mod 2^32
    kPart32 = 1,      // split partial sum_k 2^(8k) P_k mod 2^32 (no centring terms)
    kFinalModP = 2,   // Out mod p
    kPart64 = 3,      // split partial sum_k 2^(8k) P_k, exact (mod 2^64)
    // By rows: answers and partials contiguous along rows, four rows per
    // store.  Modes of their own: a branch at every store, or one around two copies of
    // the epilogue (which spilled), cost 0.7 us a tile.
    kFinal32Rows = 4,
    kPart32Rows = 5,
    kClientQuery = 6,    // kFinal32Rows, then the client's query epilogue
    kClientDecode = 7,   // kFinal32Rows, then the client's decode
};

__global__ void k_zero_words(uint32_t* __restrict__ p, uint32_t n) {
    const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = 0;
}

// Block: 128 query coordinates j x 64 queries b.  Element (j, b) of the
// query matrix is Q[j * ldj + b * ldb].  Loads are coalesced along b for the
// row-major layout (ldb == 1: a wave reads 64 consecutive words of one row)
// and along j for the query-major one (QMAJOR, ldj == 1).  The tile goes
// through LDS with rows padded to 129 words, so that the stores hit 64
// distinct banks.  The block's QL rows 4*b0 .. 4*b0+255 (either layout)
// are consecutive 128-byte runs of the tiled layout; in the write phase lane l of a wave
// packs and stores 16-byte chunk l % 8 of row l / 8, so one store covers
// eight whole rows (1 KiB).  (Storing a thread's whole row as eight 16-byte
// pieces made every store touch 64 lines: 1.6 TB/s at 128 queries.)  The
// rows of limb 0 also sum their words (colsum set): three lane shuffles
// combine the eight chunks of a row, and one lane adds the exact column sum.
constexpr int kIngJ = 128;
constexpr int kIngB = 64;

// VEC: 16-byte loads (4 consecutive queries of a row, or 4 consecutive
// coordinates of a query) at any word address, where the contiguous extent
// (B, or C for QMAJOR) is at least 4; the last group of a ragged extent is
// loaded four words before its end, and words that two lanes then hold are
// stored twice.  Each thread has its whole share of the tile (8 loads, 128
// bytes) in flight at once; with a word per load, 8 of 32 in flight, a
// call of 37 queries on 20000 x 10007 took 100.8 us, 88.9 so.
typedef u32x4 word_u32x4 __attribute__((aligned(4)));
template <bool QMAJOR, bool VEC>
__global__ __launch_bounds__(256) void k_ingest(const uint32_t* __restrict__ Q, uint64_t ldj,
                                                uint64_t ldb, uint32_t C, uint32_t B, uint32_t Bp,
                                                uint32_t Cp, int8_t* __restrict__ QL,
                                                u64* __restrict__ colsum, bool narrow) {
    __shared__ uint32_t s[kIngB][kIngJ + 1];
    const int t = threadIdx.x;
    // Query blocks vary fastest across the grid, so the blocks that read one
    // row of a row-major Q (64 queries each) are dispatched together.
    const uint32_t b0 = blockIdx.x * (uint32_t)kIngB;
    const uint32_t j0 = blockIdx.y * (uint32_t)kIngJ;
    if (VEC && QMAJOR) {
        const int j4 = t & 31, br = t >> 5;
        const uint32_t j = j0 + 4u * j4;
        u32x4 v[8];
#pragma unroll
        for (int p = 0; p < 8; ++p) {
            const uint32_t b = b0 + br + 8 * p;
            v[p] = (j < C && b < B)
                       ? *reinterpret_cast<const word_u32x4*>(Q + (uint64_t)b * ldb + min(j, C - 4u))
                       : u32x4{0, 0, 0, 0};
        }
        const int at = (int)(j < C ? min(j, C - 4u) : j) - (int)j0;
        const int past = (int)min(C - j0, (uint32_t)kIngJ);   // coordinates the block holds
#pragma unroll
        for (int p = 0; p < 8; ++p) {
            const int bl = br + 8 * p;
#pragma unroll
            for (int x = 0; x < 4; ++x) {
                if (C % 4u == 0) {              // uniform: whole groups only
                    s[bl][4 * j4 + x] = v[p][x];
                } else {
                    if (at + x >= 0) s[bl][at + x] = v[p][x];
                    if (at < 4 * j4 && 4 * j4 + x >= past) s[bl][4 * j4 + x] = 0u;
                }
            }
        }
    } else if (VEC) {
        const int q4 = t & 15, jr = t >> 4;
        const uint32_t b = b0 + 4u * q4;
        u32x4 v[8];
#pragma unroll
        for (int p = 0; p < 8; ++p) {
            const uint32_t j = j0 + jr + 16 * p;
            v[p] = (j < C && b < B)
                       ? *reinterpret_cast<const word_u32x4*>(Q + (uint64_t)j * ldj + min(b, B - 4u))
                       : u32x4{0, 0, 0, 0};
        }
        const int at = (int)(b < B ? min(b, B - 4u) : b) - (int)b0;
#pragma unroll
        for (int p = 0; p < 8; ++p) {
            const int jl = jr + 16 * p;
#pragma unroll
            for (int x = 0; x < 4; ++x) {
                if (B % 4u == 0) s[4 * q4 + x][jl] = v[p][x];
                else if (at + x >= 0) s[at + x][jl] = v[p][x];
            }
        }
    } else if (QMAJOR) {
        const int jl = t & (kIngJ - 1);
        const uint32_t j = j0 + jl;
#pragma unroll 8
        for (int p = 0; p < kIngB / 2; ++p) {
            const int bl = (t >> 7) + 2 * p;
            const uint32_t b = b0 + bl;
            s[bl][jl] = (j < C && b < B) ? Q[(uint64_t)j * ldj + (uint64_t)b * ldb] : 0u;
        }
    } else {
        const int bl = t & (kIngB - 1);
        const uint32_t b = b0 + bl;
#pragma unroll 8
        for (int p = 0; p < kIngJ / 4; ++p) {
            const int jl = (t >> 6) + 4 * p;
            const uint32_t j = j0 + jl;
            s[bl][jl] = (j < C && b < B) ? Q[(uint64_t)j * ldj + (uint64_t)b * ldb] : 0u;
        }
    }
    __syncthreads();
    const int e = t & 7;                       // 16-byte chunk of the row
    const uint32_t n0 = 4u * b0;               // first QL row of the block, either layout
#pragma unroll 2
    for (int rnd = 0; rnd < 8; ++rnd) {
        const int R = rnd * 32 + (t >> 3);     // row of the block, 0..255
        // Wide: R = 128 g + 32 limb + b % 32; narrow: R = 32 g + 8 limb + b % 8.
        // Either way limb and the 8-query group of b are uniform per wave.
        const int limb = narrow ? (R & 31) >> 3 : (R & 127) >> 5;
        const int bl = narrow ? (R >> 5) * 8 + (R & 7) : (R >> 7) * 32 + (R & 31);
        const uint32_t b = b0 + bl;
        if (b >= Bp) continue;                 // uniform per wave (Bp % 8 == 0): no QL row
        const bool live = b < B;
        uint32_t w[4];
        u64 sum = 0;
#pragma unroll
        for (int x = 0; x < 4; ++x) {
            uint32_t word = 0;
#pragma unroll
            for (int y = 0; y < 4; ++y) {
                const int jl = 16 * e + 4 * x + y;
                const uint32_t v = s[bl][jl];
                if (limb == 0 && colsum) sum += v;
                const uint32_t byte =
                    (live && j0 + jl < C) ? (((v >> (8 * limb)) & 0xFFu) ^ 0x80u) : 0u;
                word |= byte << (8 * y);
            }
            w[x] = word;
        }
        *reinterpret_cast<u32x4*>(QL + ql_row(n0 + R, Cp) + ql_col(j0) + 16 * e) =
            u32x4{w[0], w[1], w[2], w[3]};
        if (limb == 0 && colsum) {
            sum += __shfl_xor(sum, 1);
            sum += __shfl_xor(sum, 2);
            sum += __shfl_xor(sum, 4);
            if (e == 0 && live) atomicAdd(&colsum[b], sum);
        }
    }
}

// ---------------------------------------------------------------- epilogue
struct Epi {
    uint32_t M;                 // output rows (gathered rows, or R)
    uint32_t B, R, C;
    const uint32_t* rows;       // database row of output row i, or null
    const u64* colsum;          // exact column sums, B words, or null (see SUMS)
    const uint32_t* rowsum;     // row metadata: exact row sums, or row terms (see row_scale)
    uint32_t row_scale;         // factor of rowsum mod 2^32
    uint32_t* out;
    uint64_t o_ldr, o_ldb;
    void* part;                 // split-K partials [split][M][B], or [split][B][M] with by_rows
    uint32_t p;                 // modulus of the field form
    bool by_rows;               // answers contiguous along rows: four rows per 16-byte access
    ClientEpi client;           // client modes
};

// Column terms; zero where the product added them itself (k_gemm_ring, SUMS).
__device__ inline uint32_t colterm32(const Epi& e, uint32_t b) {
    if (!e.colsum) return 0u;
    return 128u * ((uint32_t)e.colsum[b] - e.C * kCentreWord);
}

__device__ inline u64 colterm64(const Epi& e, uint32_t b) {
    if (!e.colsum) return 0ull;
    return 128ull * (e.colsum[b] - (u64)e.C * kCentreWord);
}

// Exact value of a limb product read from its int32 accumulator (K <= 2^17).
__device__ inline u64 limb64(int32_t v) {
    return v == INT32_MIN ? (1ull << 31) : (u64)(int64_t)v;
}

template <int MODE>
constexpr bool partial_mode() {
    return MODE == kPart32 || MODE == kPart32Rows || MODE == kPart64;
}

template <int MODE>
constexpr bool by_rows_mode() {
    return MODE >= kFinal32Rows;
}

template <int MODE>
constexpr bool mod32_mode() {
    return MODE != kFinalModP && MODE != kPart64;
}

// What is added to every limb combination of query b before it is stored:
// its bias, and in the final modes the column term.
template <int MODE>
__device__ inline u64 query_term(const Epi& e, uint32_t b, u64 bias) {
    if (partial_mode<MODE>() || b >= e.B) return bias;
    return bias + (MODE == kFinalModP ? colterm64(e, b) : (u64)colterm32(e, b));
}

using gu32 = __attribute__((address_space(1))) uint32_t;
using gu32x4 = __attribute__((address_space(1))) u32x4;

// What the stores of a wave's rows need of the database: the row sums of its
// lane's 16 TM rows (register v of tile a holds row m_base + 32 a + 8 (v/4)
// + 4 (lane/32) + v%4) and, gathered, the rows themselves.  All are loaded
// before the first store: a load between stores waits for every store before
// it, 64 times a tile (1024 queries on 32768 x 32768: 3900 -> 3860 us).
template <int MODE, bool GATHER, int TM>
struct RowTerms {
    static constexpr bool kUsed = !partial_mode<MODE>();
    uint32_t sum[kUsed ? TM : 1][16], row[kUsed && GATHER ? TM : 1][16];

    __device__ RowTerms(const Epi& e, uint32_t m_base, int lane) {
        if constexpr (kUsed) {
#pragma unroll
            for (int a = 0; a < TM; ++a) {
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    uint32_t i = m_base + a * 32 + 8 * (v / 4) + 4 * (lane >> 5) + v % 4;
                    if constexpr (GATHER) {
                        i = e.rows[i < e.M ? i : e.M - 1u];
                        row[a][v] = i;
                    }
                    sum[a][v] = e.rowsum[i < e.R ? i : e.R - 1u];
                }
            }
        }
    }
    __device__ u32x4 sum4(int a, int v4) const {
        return u32x4{sum[a][4 * v4], sum[a][4 * v4 + 1], sum[a][4 * v4 + 2], sum[a][4 * v4 + 3]};
    }
};

// Output element (local row i, query b; register v of tile a) from its limb
// combination x = sum_k 2^(8k) P_k plus the query's term (exact; only x mod
// 2^32 matters in the 32-bit modes).
template <int MODE, bool GATHER, int TM>
__device__ inline void epi_put(const Epi& e, uint32_t split, uint32_t i, uint32_t b, u64 x,
                               const RowTerms<MODE, GATHER, TM>& t, int a, int v) {
    if (i >= e.M || b >= e.B) return;
    if constexpr (MODE == kFinal32 || MODE == kFinalModP) {
        uint32_t r = i;
        if constexpr (GATHER) r = t.row[a][v];
        if (r >= e.R) return;
        gu32* dst = (gu32*)e.out + (uint64_t)r * e.o_ldr + (uint64_t)b * e.o_ldb;
        if constexpr (MODE == kFinal32)
            *dst = (uint32_t)x + e.row_scale * t.sum[a][v];
        else
            *dst = (uint32_t)((x + (u64)kCentreWord * t.sum[a][v]) % e.p);
    } else {
        const uint64_t at = ((uint64_t)split * e.M + i) * e.B + b;
        if constexpr (MODE == kPart32)
            static_cast<uint32_t*>(e.part)[at] = (uint32_t)x;
        else
            static_cast<u64*>(e.part)[at] = x;
    }
}

// The client step's operand for query b at rows i .. i+3, and the queried column.
template <int MODE>
__device__ inline u32x4 client_add(const Epi& e, uint32_t i, uint32_t b) {
    if constexpr (MODE != kClientQuery && MODE != kClientDecode) return u32x4{0u, 0u, 0u, 0u};
    if (i >= e.M || b >= e.B) return u32x4{0u, 0u, 0u, 0u};
    return *reinterpret_cast<const u32x4*>(e.client.add + (uint64_t)b * e.o_ldb + i);
}

template <int MODE>
__device__ inline uint32_t client_col(const Epi& e, uint32_t b) {
    if constexpr (MODE != kClientQuery) return 0u;
    return b < e.B ? e.client.cols[b] : 0u;
}

// Answers of query b at rows i .. i+3 (i % 4 == 0, e.M % 4 == 0; the query's
// and the rows' terms are in x) stored; kClientQuery and kClientDecode add
// the client step's epilogue.
template <int MODE>
__device__ inline void rows4_store(const Epi& e, uint32_t i, uint32_t b, u32x4 x, u32x4 add,
                                   uint32_t col) {
    const uint64_t at = (uint64_t)b * e.o_ldb + i;
    if constexpr (MODE == kClientQuery) {
        x += add;
        const uint32_t d = col - i;      // the queried column, if among the four
        x.x += d == 0u ? kClientDelta : 0u;
        x.y += d == 1u ? kClientDelta : 0u;
        x.z += d == 2u ? kClientDelta : 0u;
        x.w += d == 3u ? kClientDelta : 0u;
    }
    if constexpr (MODE == kClientDecode) {
        const u32x4 y = add - x + kClientDelta / 2u;
        *(gu32*)(e.client.bytes + at) =
            (y.x >> 24) | ((y.y >> 24) << 8) | ((y.z >> 24) << 16) | (y.w & 0xFF000000u);
    } else {
        *(gu32x4*)((gu32*)e.out + at) = x;
    }
}

template <int MODE>
__device__ inline void epi_put_rows4(const Epi& e, uint32_t split, uint32_t i, uint32_t b,
                                     u32x4 x, u32x4 rowsum, u32x4 add, uint32_t col) {
    if (i >= e.M || b >= e.B) return;
    if constexpr (MODE == kPart32Rows)
        *reinterpret_cast<u32x4*>(static_cast<uint32_t*>(e.part) +
                                  ((uint64_t)split * e.B + b) * e.M + i) = x;
    else
        rows4_store<MODE>(e, i, b, x + e.row_scale * rowsum, add, col);
}

// Write a wave's accumulators through the epilogue: the four limb tiles of
// query group g sit in acc[a][4g .. 4g+3] (C layout of the 32x32 MFMA: lane
// holds column lane % 32, register v holds row 8 (v/4) + 4 (lane/32) + v%4,
// so four consecutive registers are four consecutive rows).
// bias[t] is added to every product of limb tile t (the lane's column).
// BY_TILE: the row terms of one 32-row tile at a time, where all of them
// would not fit the registers.
template <int MODE, bool GATHER, int TM, int TN,
          bool BY_TILE = TM == 4 && (GATHER || MODE == kFinalModP)>
__device__ inline void epi_wave(const Epi& e, uint32_t split, const i32x16 (&acc)[TM][TN],
                                const int64_t (&bias)[TN], uint32_t m_base, uint32_t n_base,
                                int lane) {
    constexpr bool kMod32 = mod32_mode<MODE>();
    using Rows = RowTerms<MODE, GATHER, BY_TILE ? 1 : TM>;
    Rows rt(e, m_base, lane);
    auto row4 = [&](int a, int v4) { return m_base + a * 32 + 8 * v4 + 4 * (lane >> 5); };
#pragma unroll
    for (int g = 0; g < TN / 4; ++g) {
        const uint32_t bq = n_base / 4u + 32u * g + (uint32_t)(lane & 31);
        const u64 qterm = query_term<MODE>(
            e, bq, (u64)bias[4 * g] + ((u64)bias[4 * g + 1] << 8) + ((u64)bias[4 * g + 2] << 16) +
                       ((u64)bias[4 * g + 3] << 24));
        const uint32_t col = client_col<MODE>(e, bq);
        u32x4 add[TM][4];
#pragma unroll
        for (int k = 0; k < 4 * TM; ++k) add[k / 4][k % 4] = client_add<MODE>(e, row4(k / 4, k % 4), bq);
#pragma unroll
        for (int a = 0; a < TM; ++a) {
            if (BY_TILE && (g || a)) rt = Rows(e, m_base + a * 32, lane);
            const int ta = BY_TILE ? 0 : a;
#pragma unroll
            for (int v4 = 0; v4 < 4; ++v4) {
                u64 x[4];
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const int v = 4 * v4 + j;
                    const int32_t p0 = acc[a][4 * g][v], p1 = acc[a][4 * g + 1][v],
                                  p2 = acc[a][4 * g + 2][v], p3 = acc[a][4 * g + 3][v];
                    x[j] = kMod32 ? (u64)((uint32_t)p0 + ((uint32_t)p1 << 8) +
                                          ((uint32_t)p2 << 16) + ((uint32_t)p3 << 24) +
                                          (uint32_t)qterm)
                                  : limb64(p0) + (limb64(p1) << 8) + (limb64(p2) << 16) +
                                        (limb64(p3) << 24) + qterm;
                }
                const uint32_t i = row4(a, v4);
                if constexpr (by_rows_mode<MODE>()) {
                    const u32x4 x4 = {(uint32_t)x[0], (uint32_t)x[1], (uint32_t)x[2],
                                      (uint32_t)x[3]};
                    u32x4 rs = {0u, 0u, 0u, 0u};
                    if constexpr (Rows::kUsed) rs = rt.sum4(ta, v4);
                    epi_put_rows4<MODE>(e, split, i, bq, x4, rs, add[a][v4], col);
                } else {
#pragma unroll
                    for (int j = 0; j < 4; ++j)
                        epi_put(e, split, i + j, bq, x[j], rt, ta, 4 * v4 + j);
                }
            }
        }
    }
}

// Narrow layout: in 32-column tile t of a wave, lane column c holds limb
// c / 8 of query n_base / 4 + 8 t + c % 8 (C layout as above).  The four
// limbs of a query sit in lanes c, c ^ 8, c ^ 16, c ^ 24 of the same half
// wave; two xor shuffles add the shifted products.  Then the lanes with c < 8
// store, or, along rows, the lanes of limb l store the four rows of register
// group l.
template <int MODE, bool GATHER, int TM, int TN>
__device__ inline void epi_wave_narrow(const Epi& e, uint32_t split, const i32x16 (&acc)[TM][TN],
                                       const int64_t (&bias)[TN], uint32_t m_base, uint32_t n_base,
                                       int lane) {
    const int c = lane & 31;
    const int limb = c >> 3;
    constexpr bool kMod32 = mod32_mode<MODE>();
    const RowTerms<MODE, GATHER, TM> rt(e, m_base, lane);
#pragma unroll
    for (int t = 0; t < TN; ++t) {
        const uint32_t bq = n_base / 4u + 8u * t + (uint32_t)(c & 7);
        const u64 qterm = query_term<MODE>(e, bq, 0);
#pragma unroll
        for (int a = 0; a < TM; ++a) {
            const uint32_t i0 = m_base + a * 32 + 4 * (lane >> 5);
            if constexpr (kMod32) {
                u32x4 x4[4];
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    uint32_t y = ((uint32_t)acc[a][t][v] + (uint32_t)bias[t]) << (8 * limb);
                    y += __shfl_xor(y, 8);
                    y += __shfl_xor(y, 16);
                    x4[v / 4][v % 4] = y + (uint32_t)qterm;
                }
                if constexpr (by_rows_mode<MODE>()) {
                    auto of_limb = [&](u32x4 y0, u32x4 y1, u32x4 y2, u32x4 y3) {
                        return limb == 0 ? y0 : (limb == 1 ? y1 : (limb == 2 ? y2 : y3));
                    };
                    u32x4 rs = {0u, 0u, 0u, 0u};
                    if constexpr (rt.kUsed)
                        rs = of_limb(rt.sum4(a, 0), rt.sum4(a, 1), rt.sum4(a, 2), rt.sum4(a, 3));
                    epi_put_rows4<MODE>(e, split, i0 + 8 * limb, bq,
                                                    of_limb(x4[0], x4[1], x4[2], x4[3]), rs, rs, 0u);
                } else if (limb == 0) {
#pragma unroll
                    for (int v = 0; v < 16; ++v)
                        epi_put(e, split, i0 + 8 * (v / 4) + v % 4, bq, (u64)x4[v / 4][v % 4], rt, a, v);
                }
            } else {
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    u64 x = (limb64(acc[a][t][v]) + (u64)bias[t]) << (8 * limb);
                    x += __shfl_xor(x, 8);
                    x += __shfl_xor(x, 16);
                    if (limb == 0)
                        epi_put(e, split, i0 + 8 * (v / 4) + v % 4, bq, x + qterm, rt, a, v);
                }
            }
        }
    }
}

// Sum of the split partials plus the centring terms, one output per thread.
template <bool EXACT>
__global__ __launch_bounds__(256) void k_finish(Epi e, uint32_t splits) {
    const uint64_t idx = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= (uint64_t)e.M * e.B) return;
    const uint32_t i = (uint32_t)(idx / e.B), b = (uint32_t)(idx % e.B);
    const uint32_t r = e.rows ? e.rows[i] : i;
    if (r >= e.R) return;
    const uint64_t plane = (uint64_t)e.M * e.B;
    uint32_t* dst = e.out + (uint64_t)r * e.o_ldr + (uint64_t)b * e.o_ldb;
    const uint32_t rowsum = e.rowsum[r];
    if (EXACT) {
        const u64 ct = colterm64(e, b);
        const u64* part = static_cast<const u64*>(e.part) + idx;
        u64 v = part[0];
#pragma unroll 4
        for (uint32_t s = 1; s < splits; ++s) v += part[s * plane];
        *dst = (uint32_t)((v + ct + (u64)kCentreWord * rowsum) % e.p);
    } else {
        const uint32_t ct = colterm32(e, b);
        const uint32_t* part = static_cast<const uint32_t*>(e.part) + idx;
        uint32_t v = part[0];
#pragma unroll 4
        for (uint32_t s = 1; s < splits; ++s) v += part[s * plane];
        *dst = v + ct + e.row_scale * rowsum;
    }
}

// The same for the mod 2^32 form, four queries per thread with 16-byte
// partial loads and output stores (B % 4 == 0, queries contiguous and the
// output rows 16-byte aligned): a quarter of the threads and address
// arithmetic for a pass that only streams the partials.
__global__ __launch_bounds__(256) void k_finish4(Epi e, uint32_t splits) {
    const uint64_t g = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;   // group of 4 outputs
    const uint32_t B4 = e.B / 4u;
    if (g >= (uint64_t)e.M * B4) return;
    const uint32_t i = (uint32_t)(g / B4), b = 4u * (uint32_t)(g % B4);
    const uint32_t r = e.rows ? e.rows[i] : i;
    if (r >= e.R) return;
    const uint64_t plane4 = (uint64_t)e.M * B4;
    const u32x4* part = static_cast<const u32x4*>(e.part) + g;
    const uint32_t rowsum = e.rowsum[r];
    u32x4 ct = {0u, 0u, 0u, 0u};
    if (e.colsum)
        ct = u32x4{colterm32(e, b), colterm32(e, b + 1), colterm32(e, b + 2), colterm32(e, b + 3)};
    u32x4 v = part[0];
#pragma unroll 4
    for (uint32_t s = 1; s < splits; ++s) v += part[s * plane4];
    *reinterpret_cast<u32x4*>(e.out + (uint64_t)r * e.o_ldr + b) = v + ct + e.row_scale * rowsum;
}

// The same for answers and partials contiguous along rows (query-major
// answers, M % 4 == 0): four rows of a query per thread.
template <int MODE>
__global__ __launch_bounds__(256) void k_finish_rows(Epi e, uint32_t splits) {
    const uint64_t g = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const uint32_t M4 = e.M / 4u;
    if (g >= (uint64_t)M4 * e.B) return;
    const uint32_t b = (uint32_t)(g / M4), i = 4u * (uint32_t)(g % M4);
    const u32x4* part = static_cast<const u32x4*>(e.part) + g;
    const u32x4 rowsum = *reinterpret_cast<const u32x4*>(e.rowsum + i);
    const u32x4 add = client_add<MODE>(e, i, b);
    const uint32_t col = client_col<MODE>(e, b), ct = colterm32(e, b);
    u32x4 v = part[0];
#pragma unroll 4
    for (uint32_t s = 1; s < splits; ++s) v += part[(uint64_t)s * M4 * e.B];
    rows4_store<MODE>(e, i, b, v + ct + e.row_scale * rowsum, add, col);
}

// Workgroups are dealt round-robin to the 8 XCDs; give each XCD a
// contiguous range of workgroup indices, so the tiles it runs at once are
// neighbours (shared D rows and query tiles stay in its own L2).
__device__ inline uint32_t xcd_remap(uint32_t bid, uint32_t nblk) {
    const uint32_t per = nblk / 8u;
    return bid < per * 8u ? (bid % 8u) * per + bid / 8u : bid;
}

// Tile of a (remapped) workgroup index, split-major: within a split, tiles
// go in groups of `group` row tiles (8 over a whole database) so the ~32
// workgroups an XCD runs at once share D and QL tiles in its L2.  Gathered
// rows take every row tile of a column tile as one group: their few row
// tiles then read each limb-plane tile together.
struct TileId {
    uint32_t m, n, split;
};

__device__ inline TileId tile_of(uint32_t bid, uint32_t n_tiles, uint32_t m_tiles,
                                 uint32_t kGroup = 8) {
    const uint32_t tiles = n_tiles * m_tiles;
    TileId t;
    t.split = bid / tiles;
    bid %= tiles;
    const uint32_t first_m = (bid / (kGroup * n_tiles)) * kGroup;
    const uint32_t gsize = min(m_tiles - first_m, kGroup);
    const uint32_t in_group = bid % (kGroup * n_tiles);
    t.m = first_m + in_group % gsize;
    t.n = in_group / gsize;
    return t;
}

// ---------------------------------------------------------------- LDS ring helpers
// 16-byte slot of (row, segment) in an LDS row.  A fragment read has 32
// lanes on 32 consecutive rows at one segment; gfx950's LDS serves a
// 16-byte read 16 lanes at a time across 64 four-byte banks, so the 16 rows
// of a pass must land on 16 distinct 16-byte bank groups.  A 64-byte row
// spans 16 banks (row % 4 picks the quarter of the bank space), a 128-byte
// row 32 banks (row % 2); XORing the segment with the next row bits fills
// the remaining choices.  (Measured: a swizzle that is conflict-free for
// 8 lanes over 32 banks spent half of the LDS cycles in bank conflicts.)
template <int BK>
__device__ inline int swz(int row, int seg) {
    return BK == 64 ? (seg ^ ((row >> 2) & 3)) : (seg ^ ((row >> 1) & 7));
}

// s_waitcnt with only vmcnt constrained (gfx9 encoding: vmcnt low bits
// [3:0], high bits [15:14]; expcnt and lgkmcnt left at their maximum).
template <int N>
__device__ inline void wait_vmcnt() {
    static_assert(N >= 0 && N < 64, "vmcnt range");
    __builtin_amdgcn_s_waitcnt((N & 0xF) | ((N >> 4) << 14) | (0x7 << 4) | (0xF << 8));
}

// Workgroup barrier without the memory fence of __syncthreads(): the fence
// would drain every outstanding load (vmcnt(0)) and empty the ring.  Each
// wave has already waited for its own tile loads (wait_vmcnt), and LDS
// reads are not moved across the asm statements.
__device__ inline void ring_barrier() {
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

// ---------------------------------------------------------------- GEMM, register-staged
// 16 bytes at any alignment.
typedef u32x4 u32x4_any __attribute__((aligned(1)));

template <int WM_, int WN_, int TM_, int TN_>
struct Tile {
    static constexpr int WM = WM_, WN = WN_, TM = TM_, TN = TN_, BK = 128;
    static constexpr int NW = WM * WN;
    static constexpr int THREADS = 64 * NW;
    static constexpr int BM = WM * TM * 32;
    static constexpr int BN = WN * TN * 32;
    static constexpr int A_LOADS = BM / 8 / NW;      // 1 KiB blocks of 8 rows per wave
    static constexpr int B_LOADS = BN / 8 / NW;
    static constexpr int LOADS = A_LOADS + B_LOADS;
    static constexpr int BUF_BYTES = (BM + BN) * BK;
    static constexpr int LDS_BYTES = 2 * BUF_BYTES;
    static_assert(NW == 4 || NW == 8, "four or eight waves");
    static_assert(TN % 4 == 0, "a wave covers whole groups of four limbs");
    static_assert(A_LOADS >= 1 && B_LOADS >= 1, "tile too small for the waves");
    static_assert(LDS_BYTES <= 160 * 1024, "LDS");
};

// The product for databases the ring cannot serve: direct-to-LDS loads need
// 16-byte aligned rows, so here the tiles pass through registers.  D rows are
// read in 16-byte pieces at any address; in a row's ragged last tile the
// piece that crosses the end is the row's last 16 bytes, shifted, and pieces
// past it meet zero limbs.  LWE form.
//
// Two LDS buffers (the ring's swizzle) and one barrier per 128-byte tile: the
// loads of tile u+1 are issued one after each of the first MFMAs of tile u
// and written to the other buffer after its last.  Bound by that staging: the
// loads have one tile's MFMAs to land, and every byte passes the register
// file.  37 and 200 queries on 20000 rows of 10007 bytes, whole calls on the
// same buffers: byte loads, no split-K 698 and 1887 us; 16-byte loads and
// split-K, one buffer and two barriers 115 and 417 us; now 88 and 282 us (37
// queries with other inputs on every call: 900 and 90 us).
template <class T, bool GATHER, int MODE>
__global__ __launch_bounds__(T::THREADS) void k_gemm(const uint8_t* __restrict__ D, uint64_t pitch,
                                                     const int8_t* __restrict__ QL, uint32_t Cp,
                                                     uint32_t n_tiles, uint32_t m_tiles,
                                                     uint32_t kts, Epi e) {
    extern __shared__ __attribute__((aligned(16))) uint8_t smem[];
    const uint32_t R = e.R, C = e.C, M = e.M;
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave / T::WN;
    const int wn = wave % T::WN;

    const TileId tl = tile_of(xcd_remap(blockIdx.x, gridDim.x), n_tiles, m_tiles,
                              GATHER ? m_tiles : 8u);
    const uint32_t m0 = tl.m * T::BM;
    const uint32_t n0 = tl.n * T::BN;
    const uint32_t ktiles_all = (C + T::BK - 1) / T::BK;
    const uint32_t kt0 = tl.split * kts;
    const uint32_t ktiles = kt0 < ktiles_all ? min(kts, ktiles_all - kt0) : 0u;

    // Block i of this wave: rows 8 (wave + NW i) .. + 7, lane: row lane / 8,
    // 16-byte segment lane % 8.
    const int lrow = lane >> 3;
    const uint32_t kseg = 16u * (lane & 7);
    const uint8_t* arow[T::A_LOADS];
    const int8_t* brow[T::B_LOADS];
#pragma unroll
    for (int i = 0; i < T::A_LOADS; ++i) {
        uint32_t mi = m0 + 8 * (wave + T::NW * i) + lrow;
        mi = mi < M ? mi : M - 1;
        const uint32_t r = GATHER ? e.rows[mi] : mi;
        arow[i] = D + (uint64_t)(r < R ? r : R - 1) * pitch;
    }
#pragma unroll
    for (int i = 0; i < T::B_LOADS; ++i)
        brow[i] = QL + ql_row(n0 + 8 * (wave + T::NW * i) + lrow, Cp) + kseg;

    u32x4 ra[T::A_LOADS], rb[T::B_LOADS];
    // Load i of the tile at column k0 (C >= 16), D first.
    auto load_one = [&](uint32_t k0, int i) {
        if (i < T::A_LOADS)
            ra[i < T::A_LOADS ? i : 0] = *reinterpret_cast<const u32x4_any*>(
                arow[i < T::A_LOADS ? i : 0] + min(k0 + kseg, C - 16u));
        else
            rb[i - T::A_LOADS] = *reinterpret_cast<const u32x4*>(brow[i - T::A_LOADS] + ql_col(k0));
    };
    auto store = [&](uint32_t k0, uint8_t* buf) {
        if (k0 + T::BK > C && C % 16u != 0u) {   // the row's ragged last tile
            const uint32_t k = k0 + kseg;
            const uint32_t sh = 8u * min(k - min(k, C - 16u), 15u);
#pragma unroll
            for (int i = 0; i < T::A_LOADS; ++i) {
                u64 lo = (u64)ra[i].x | ((u64)ra[i].y << 32), hi = (u64)ra[i].z | ((u64)ra[i].w << 32);
                if (sh >= 64u) {
                    lo = hi >> (sh - 64u);
                } else if (sh != 0u) {
                    lo = (lo >> sh) | (hi << (64u - sh));
                    hi >>= sh;
                }
                ra[i] = u32x4{(uint32_t)lo, (uint32_t)(lo >> 32), (uint32_t)hi, (uint32_t)(hi >> 32)};
            }
        }
#pragma unroll
        for (int i = 0; i < T::A_LOADS; ++i) {
            const int r = 8 * (wave + T::NW * i) + lrow;
            *reinterpret_cast<u32x4*>(buf + r * T::BK + 16 * swz<128>(r, lane & 7)) =
                ra[i] ^ u32x4{kCentreWord, kCentreWord, kCentreWord, kCentreWord};
        }
#pragma unroll
        for (int i = 0; i < T::B_LOADS; ++i) {
            const int r = 8 * (wave + T::NW * i) + lrow;
            *reinterpret_cast<u32x4*>(buf + T::BM * T::BK + r * T::BK +
                                      16 * swz<128>(r, lane & 7)) = rb[i];
        }
    };

    i32x16 acc[T::TM][T::TN];
#pragma unroll
    for (int a = 0; a < T::TM; ++a)
#pragma unroll
        for (int b = 0; b < T::TN; ++b)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[a][b][v] = 0;

    const int frow = lane & 31;
    const int fseg = lane >> 5;
    i32x4 fa[2][T::TM], fb[2][T::TN];
    auto read_frags = [&](const uint8_t* buf, int ks, int f) {
        const int seg = 2 * ks + fseg;
#pragma unroll
        for (int a = 0; a < T::TM; ++a) {
            const int r = wm * T::TM * 32 + a * 32 + frow;
            fa[f][a] = *reinterpret_cast<const i32x4*>(buf + r * T::BK + 16 * swz<128>(r, seg));
        }
#pragma unroll
        for (int b = 0; b < T::TN; ++b) {
            const int r = wn * T::TN * 32 + b * 32 + frow;
            fb[f][b] = *reinterpret_cast<const i32x4*>(buf + T::BM * T::BK + r * T::BK +
                                                       16 * swz<128>(r, seg));
        }
    };

    if (ktiles > 0) {
        if (C >= 16u) {
#pragma unroll
            for (int i = 0; i < T::LOADS; ++i) load_one(kt0 * T::BK, i);
        } else {   // rows shorter than a load: one tile, byte by byte
#pragma unroll
            for (int i = 0; i < T::A_LOADS; ++i) {
                uint32_t w[4] = {0, 0, 0, 0};
                for (uint32_t x = 0; kseg + x < C; ++x)
                    w[x >> 2] |= (uint32_t)arow[i][kseg + x] << (8 * (x & 3));
                ra[i] = u32x4{w[0], w[1], w[2], w[3]};
            }
#pragma unroll
            for (int i = T::A_LOADS; i < T::LOADS; ++i) load_one(0, i);
        }
        store(C >= 16u ? kt0 * T::BK : 0u, smem);
    }
    __syncthreads();
    for (uint32_t u = 0; u < ktiles; ++u) {
        const uint8_t* buf = smem + (u & 1u) * T::BUF_BYTES;
        // Past the last tile the loads repeat it, into a buffer nobody reads.
        const uint32_t k1 = (kt0 + min(u + 1u, ktiles - 1u)) * T::BK;
        read_frags(buf, 0, 0);
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) {
            if (ks < 3) read_frags(buf, ks + 1, (ks + 1) & 1);
            __builtin_amdgcn_sched_barrier(0);
            constexpr int kMfma = T::TM * T::TN;
            const int lo = ks * kMfma < T::LOADS ? ks * kMfma : T::LOADS;
            const int hi = (ks + 1) * kMfma < T::LOADS ? (ks + 1) * kMfma : T::LOADS;
#pragma unroll
            for (int a = 0; a < T::TM; ++a)
#pragma unroll
                for (int b = 0; b < T::TN; ++b)
                    acc[a][b] = __builtin_amdgcn_mfma_i32_32x32x32_i8(fa[ks & 1][a], fb[ks & 1][b],
                                                                      acc[a][b], 0, 0, 0);
            if (C >= 16u) {
#pragma unroll
                for (int i = lo; i < hi; ++i) load_one(k1, i);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        if (C >= 16u) store(k1, smem + ((u + 1u) & 1u) * T::BUF_BYTES);
        __syncthreads();
    }
    const int64_t bias[T::TN] = {};
    epi_wave<MODE, GATHER, T::TM, T::TN>(e, tl.split, acc, bias, m0 + wm * T::TM * 32,
                                          n0 + wn * T::TN * 32, lane);
}

// ---------------------------------------------------------------- GEMM, LDS ring
// The main kernel for databases with 16-byte aligned rows.  Global tiles go straight to LDS with global_load_lds_dwordx4 (no register
// staging), into a ring of STAGES k-tiles of BK bytes, so STAGES-1 tiles are
// in flight while one is consumed.  Centring of D (xor 0x80) is applied to
// the A fragments in registers.
// DX_ > 0 gives D DX_ more ring slots than the limb planes (SA = STAGES +
// DX_ D tiles against SB = STAGES QL tiles), QX_ > 0 the limb planes QX_
// more than D: the deeper operand's tiles are issued that many stages
// earlier than the tiles of the other they meet.
template <int WM_, int WN_, int TM_, int TN_, int STAGES_, int BK_ = 64, bool NARROW_ = false,
          int DX_ = 0, int QX_ = 0>
struct Ring {
    static constexpr int WM = WM_, WN = WN_, TM = TM_, TN = TN_, STAGES = STAGES_;
    static constexpr int DX = DX_, QX = QX_;
    static constexpr int SA = STAGES + DX, SB = STAGES + QX;   // D and QL ring slots
    static constexpr int SMAX = SA > SB ? SA : SB;
    static_assert(DX == 0 || QX == 0, "one operand runs deeper");
    static constexpr bool NARROW = NARROW_;              // narrow QL layout (8 queries per tile)
    static constexpr int NW = WM * WN;                   // waves per workgroup
    static constexpr int THREADS = 64 * NW;
    static constexpr int BK = BK_;                       // k bytes per stage: 64 or 128
    static constexpr int SEGS = BK / 16;                 // 16-byte slots per LDS row
    static constexpr int RPB = 1024 / BK;                // rows per 1 KiB block
    static constexpr int BM = WM * TM * 32;
    static constexpr int BN = WN * TN * 32;
    static constexpr int A_BYTES = BM * BK;
    static constexpr int B_BYTES = BN * BK;
    static constexpr int STAGE_BYTES = (BM + BN) * BK;
    static constexpr int A_BLOCKS = BM / RPB;            // 1 KiB blocks
    static constexpr int BLOCKS = (BM + BN) / RPB;
    static constexpr int LOADS = BLOCKS / NW;            // per wave per tile
    static constexpr int LDS_BYTES = SA * A_BYTES + SB * B_BYTES;
    static_assert(BK == 64 || BK == 128, "64- or 128-byte stages");
    static_assert(NW == 4 || NW == 8, "four or eight waves");
    static_assert(NARROW || TN % 4 == 0, "a wave covers whole groups of four limbs");
    static_assert(BLOCKS % NW == 0, "blocks split evenly over waves");
    static_assert(A_BLOCKS % NW == 0, "a wave's first A_LOADS loads carry D rows");
    static constexpr int A_LOADS = A_BLOCKS / NW;
    static constexpr int B_LOADS = LOADS - A_LOADS;
    // Per stage a wave issues LOADS loads, one list: D first then QL (DX
    // == 0), or QL first then D (DX > 0): the deeper operand goes last, so
    // its tile issued after the other's may stay in flight while that one
    // is consumed.  Loads complete in order; at the start of stage u at most
    // QL_WAIT of this wave's loads may still be outstanding for tiles u (D
    // and QL) to have landed: the deeper operand's loads of the stage that
    // issued the other operand's tile u, plus the stages after it.
    static constexpr int QL_WAIT =
        (DX > 0 ? A_LOADS : 0) + (QX > 0 ? LOADS - A_LOADS : 0) + (STAGES - 2) * LOADS;
    // The loads of the tile that refills a freed slot are spread over all
    // KS k-steps of a stage when another tile is in flight (three or more
    // stages, or a D ring one tile deeper, whose D tile then has two stages
    // to land), else over the fewest k-steps that fit (one load per MFMA),
    // so the tile has the rest of the stage to land.  (Deeper D ring, 64
    // queries at 32768^2: 380-384 us with the loads in the first k-step,
    // 347-357 us spread; the two-stage ring and a deeper QL ring gained
    // nothing from spreading.)
    static constexpr int KS = BK / 32;
    static constexpr int FIT = (LOADS + TM * TN - 1) / (TM * TN);
    static constexpr int ISSUE_STEPS = (STAGES > 2 || DX > 0) ? KS : (FIT < KS ? FIT : KS);
    static_assert(QL_WAIT < 64, "vmcnt range");
    static_assert(STAGES >= 2, "one tile in flight while one is consumed");
    static_assert(LDS_BYTES <= 160 * 1024, "LDS");
};

// Workgroup w covers tile tile_of(w) and, with split-K, the k-tiles
// [split * kts, split * kts + kts) of its piece.
// PLANES (the client's products): column block i of e.client.n columns holds
// byte plane i of a word matrix, and limbs below i are zero in the limb planes
// there (both by value and as stored), so only the limb tiles from i up are
// loaded, read and multiplied: 10 of 16 products.  A k-tile counts for the
// block its first column lies in; what it holds of the next is zero for limb
// i.  These products are bound by the loads into LDS (about 11 TB/s over the
// chip); 64 secrets on 32768 x 1024 words, whole query call with its epilogue
// and the operand kernel: 54 us with every limb and separate epilogues, 41.6
// with the products left out and the epilogue fused (128 x 128 tile), 35.8
// with the loads left out too (128 x 256).
// SUMS: the kernel sums the limb planes' entries q' of its columns beside the
// products (four dot instructions per fragment) and adds 128 sum(q') to every
// product, which is the column term, so the ingest neither clears nor sums:
// one launch and the atomics less (see tile_sums).
template <class T, bool GATHER, int MODE, bool NTD, bool SUMS, bool PLANES = false>
__global__ __launch_bounds__(T::THREADS) void k_gemm_ring(const uint8_t* __restrict__ D,
                                                          uint64_t pitch,
                                                          const int8_t* __restrict__ QL,
                                                          uint32_t Cp, uint32_t n_tiles,
                                                          uint32_t m_tiles, uint32_t kts, Epi e) {
    extern __shared__ __attribute__((aligned(16))) uint8_t smem[];
    const uint32_t R = e.R, C = e.C, M = e.M;
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave / T::WN;
    const int wn = wave % T::WN;

    const TileId tl = tile_of(xcd_remap(blockIdx.x, gridDim.x), n_tiles, m_tiles,
                              GATHER ? m_tiles : 8u);
    const uint32_t m0 = tl.m * T::BM;
    const uint32_t n0 = tl.n * T::BN;
    const uint32_t ktiles_all = (C + T::BK - 1) / T::BK;
    const uint32_t kt0 = tl.split * kts;
    const uint32_t ktiles = kt0 < ktiles_all ? min(kts, ktiles_all - kt0) : 0u;

    // Per-lane source of each of this wave's LOADS block loads: lane l of a
    // load fills slot l % SEGS of row l / SEGS of a 1 KiB block.  Loads
    // i < A_LOADS carry D rows, the rest QL rows.
    const int lrow = lane / T::SEGS;
    const uint8_t* src[T::LOADS];
    // Load i of a stage's list: a D load (is_a) and its block index within
    // the D or QL part of the tile.
    auto is_a = [](int i) { return T::DX > 0 ? i >= T::B_LOADS : i < T::A_LOADS; };
    auto blk = [](int i) {
        return T::DX > 0 ? (i >= T::B_LOADS ? i - T::B_LOADS : i)
                         : (i < T::A_LOADS ? i : i - T::A_LOADS);
    };
    // 1 KiB block of the D or QL part of a tile that load i of the list
    // fills.  PLANES orders the QL loads by limb (a limb's rows are 4 blocks
    // of every 16), the same number of each for every wave.
    constexpr int kPerLimb = PLANES ? T::B_LOADS / 4 : 1;
    static_assert(!PLANES || (T::DX == 0 && T::QX == 0 && T::B_LOADS % 4 == 0),
                  "whole limbs per wave, one list order");
    auto block_of = [&](int i) {
        if (!PLANES || is_a(i)) return wave + T::NW * blk(i);
        const int j = blk(i);
        const int idx = wave + T::NW * (j % kPerLimb);
        constexpr int kBlocks = 32 / T::RPB;     // blocks of one limb of 32 queries
        return idx / kBlocks * 4 * kBlocks + j / kPerLimb * kBlocks + idx % kBlocks;
    };
    // A wave's blocks are whole swizzle periods apart (at least 32 rows, or
    // limbs), so a lane has the same segment in all of them.
    const uint32_t seg_off = 16u * swz<T::BK>(wave * T::RPB + lrow, lane % T::SEGS);
#pragma unroll
    for (int i = 0; i < T::LOADS; ++i) {
        const bool a = is_a(i);
        const int r = block_of(i) * T::RPB + lrow;
        if (a) {
            uint32_t mi = m0 + r;
            mi = mi < M ? mi : M - 1;
            uint32_t dr = GATHER ? e.rows[mi] : mi;
            dr = dr < R ? dr : R - 1;
            src[i] = D + (uint64_t)dr * pitch;
        } else {
            src[i] = reinterpret_cast<const uint8_t*>(QL) + ql_row(n0 + r, Cp) + seg_off;
        }
    }

    // Load i of k-tile t into its ring slot.  Every load is issued, so each
    // wave has the same count in flight per tile:
    // * a D segment past column C reads the row's last 16-byte segment
    //   instead; those bytes, and any of the row's padding in that segment,
    //   meet zero-padded query bytes;
    // * t past the piece's last tile is clamped to it: such a load refills a
    //   slot no later iteration reads.
    const uint32_t t_last = ktiles ? ktiles - 1 : 0;
    const uint32_t c_last = (C - 1u) & ~15u;
    uint8_t* const ringA = smem;                          // SA D tiles
    uint8_t* const ringB = smem + T::SA * T::A_BYTES;     // SB QL tiles
    // Load i of the list issued at stage u: D tile u + SA - 1 or QL tile
    // u + SB - 1 (DX == 0: the same tile u + STAGES - 1).
    auto issue_tile = [&](uint32_t t, int i) {
        const bool a = is_a(i);
        const uint32_t tt = min(t, t_last);
        const uint32_t k0 = (kt0 + tt) * T::BK;
        uint8_t* dst = (a ? ringA + (t % T::SA) * T::A_BYTES : ringB + (t % T::SB) * T::B_BYTES) +
                       block_of(i) * 1024;
        const uint8_t* p = a ? src[i] + min(k0 + seg_off, c_last)
                             : src[i] + ql_col(k0);   // BK divides 128
        if (NTD && a)   // D read once: non-temporal
            __builtin_amdgcn_global_load_lds((glb_void_t*)p, (lds_void_t*)dst, 16, 0, kCpolNT);
        else
            __builtin_amdgcn_global_load_lds((glb_void_t*)p, (lds_void_t*)dst, 16, 0, 0);
    };
    auto issue_one = [&](uint32_t u, int i) {
        issue_tile(u + (is_a(i) ? T::SA : T::SB) - 1, i);
    };

    i32x16 acc[T::TM][T::TN];
#pragma unroll
    for (int a = 0; a < T::TM; ++a)
#pragma unroll
        for (int b = 0; b < T::TN; ++b)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[a][b][v] = 0;

    const int frow = lane & 31;
    const int fseg = lane >> 5;
    const u32x4 centre = u32x4{kCentreWord, kCentreWord, kCentreWord, kCentreWord};
    constexpr int KS = T::KS;

    int32_t qsum[T::TN] = {};

    // Fragments of one k-step of tile u (buffer buf).
    u32x4 fa[2][T::TM];
    i32x4 fb[2][T::TN];
    auto read_frags = [&](uint32_t u, int ks, int buf, int limb0) {
        const uint8_t* sa = ringA + (u % T::SA) * T::A_BYTES;
        const uint8_t* sb = ringB + (u % T::SB) * T::B_BYTES;
        const int seg = 2 * ks + fseg;
#pragma unroll
        for (int a = 0; a < T::TM; ++a) {
            const int r = wm * T::TM * 32 + a * 32 + frow;
            fa[buf][a] = *reinterpret_cast<const u32x4*>(sa + r * T::BK + 16 * swz<T::BK>(r, seg));
        }
#pragma unroll
        for (int b = 0; b < T::TN; ++b) {
            if (PLANES && b % 4 < limb0) continue;
            const int r = wn * T::TN * 32 + b * 32 + frow;
            fb[buf][b] = *reinterpret_cast<const i32x4*>(sb + r * T::BK + 16 * swz<T::BK>(r, seg));
        }
    };
    // One k-step of MFMAs (centred A fragments ac, B buffer buf) with loads
    // lo .. hi-1 of stage u's list placed between them, one after each MFMA
    // (VMEM and MFMA scheduling groups); narrow tiles, with more loads than
    // MFMAs, issue the rest after the last MFMA.
    auto mfma_step = [&](const i32x4 (&ac)[T::TM], int buf, uint32_t u, int lo, int hi, auto limb0) {
        constexpr int kLimb0 = decltype(limb0)::value;
        constexpr int kMfma = T::TM * T::TN / 4 * (4 - kLimb0);
#pragma unroll
        for (int a = 0; a < T::TM; ++a)
#pragma unroll
            for (int b = 0; b < T::TN; ++b)
                if (!PLANES || b % 4 >= kLimb0)
                    acc[a][b] = __builtin_amdgcn_mfma_i32_32x32x32_i8(ac[a], fb[buf][b], acc[a][b], 0, 0, 0);
        if constexpr (SUMS) {
#pragma unroll
            for (int b = 0; b < T::TN; ++b) {
                if (PLANES && b % 4 < kLimb0) continue;
#pragma unroll
                for (int w = 0; w < 4; ++w)
                    qsum[b] = __builtin_amdgcn_sdot4(fb[buf][b][w], 0x01010101, qsum[b], false);
            }
        }
        constexpr int kSkip = PLANES ? kLimb0 * kPerLimb : 0;   // QL loads left out
#pragma unroll
        for (int i = lo; i < hi; ++i) issue_one(u, i < T::A_LOADS ? i : i + kSkip);
        const int paired = hi - lo < kMfma ? hi - lo : kMfma;
#pragma unroll
        for (int j = 0; j < paired; ++j) {
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
            __builtin_amdgcn_sched_group_barrier(0x010, 1, 0);
        }
#pragma unroll
        for (int j = paired; j < kMfma; ++j) __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
#pragma unroll
        for (int j = paired; j < hi - lo; ++j) __builtin_amdgcn_sched_group_barrier(0x010, 1, 0);
        __builtin_amdgcn_sched_barrier(0);
    };
    // First load of tile t_next issued in k-step j, of `loads`.
    auto first_load = [](int j, int loads) {
        return j < T::ISSUE_STEPS ? j * loads / T::ISSUE_STEPS : loads;
    };

    // The lists of the stages before the first, in the same order: stage v
    // (v = -(max(SA, SB)-1) .. -1) issues the tiles of its list that exist.
    if (ktiles > 0) {
#pragma unroll
        for (int v = -(T::SMAX - 1); v < 0; ++v)
#pragma unroll
            for (int i = 0; i < T::LOADS; ++i) {
                const int t = v + (is_a(i) ? T::SA : T::SB) - 1;
                if (t >= 0) issue_tile((uint32_t)t, i);
            }
    }

    auto stage = [&](uint32_t u, auto limb0) {
        // The loads issued after tile u's (see QL_WAIT) may still be in
        // flight; loads complete in order, so tile u has landed once at most
        // that many of this wave's loads are outstanding.  The barrier then
        // makes every wave's part visible and frees the slots of tile u-1
        // (every wave's reads of it have returned: the last MFMAs of tile
        // u-1 waited for them), which are refilled with D tile u+SA-1 and
        // QL tile u+SB-1 while tile u is consumed.
        // A stage of column block i issues the loads of limbs i and up, which
        // the tile it loads (of block i or later) reads, and never fewer than
        // the stages after it: its own count bounds what may be outstanding.
        constexpr int kLoads = T::LOADS - (PLANES ? decltype(limb0)::value * kPerLimb : 0);
        wait_vmcnt<PLANES ? (T::STAGES - 2) * kLoads : T::QL_WAIT>();
        ring_barrier();

        // Per k-step: centre the A fragments, read the fragments of the next
        // step, then the MFMAs with this step's share of the next tile's
        // loads between them (ISSUE_STEPS).  A wave issuing a tile's loads
        // back to back waits on the address unit with no MFMA to run
        // (measured: about 40% of the loop); between MFMAs the waits overlap
        // them.  The scheduling barriers keep this order.
        read_frags(u, 0, 0, decltype(limb0)::value);
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            i32x4 a_c[T::TM];
#pragma unroll
            for (int a = 0; a < T::TM; ++a) a_c[a] = __builtin_bit_cast(i32x4, fa[ks & 1][a] ^ centre);
            __builtin_amdgcn_sched_barrier(0);
            if (ks + 1 < KS) read_frags(u, ks + 1, (ks + 1) & 1, decltype(limb0)::value);
            __builtin_amdgcn_sched_barrier(0);
            mfma_step(a_c, ks & 1, u, first_load(ks, kLoads), first_load(ks + 1, kLoads), limb0);
        }
    };
    uint32_t u = 0;
    if constexpr (PLANES) {
        // First k-tile of this piece past column block i.
        auto last = [&](uint32_t i) {
            const uint32_t t = ((i + 1u) * e.client.n + T::BK - 1u) / T::BK;
            return min(ktiles, t > kt0 ? t - kt0 : 0u);
        };
        for (const uint32_t e0 = last(0); u < e0; ++u) stage(u, std::integral_constant<int, 0>{});
        for (const uint32_t e1 = last(1); u < e1; ++u) stage(u, std::integral_constant<int, 1>{});
        for (const uint32_t e2 = last(2); u < e2; ++u) stage(u, std::integral_constant<int, 2>{});
        for (; u < ktiles; ++u) stage(u, std::integral_constant<int, 3>{});
    } else {
        for (; u < ktiles; ++u) stage(u, std::integral_constant<int, 0>{});
    }
    // Loads past the last tile may still be landing in LDS.
    wait_vmcnt<0>();

    int64_t bias[T::TN] = {};
    if constexpr (SUMS) {
        // The lane's column: its half's entries and the other half's.
#pragma unroll
        for (int b = 0; b < T::TN; ++b)
            bias[b] = 128 * (int64_t)(qsum[b] + __shfl_xor(qsum[b], 32));
    }
    if constexpr (T::NARROW)
        epi_wave_narrow<MODE, GATHER, T::TM, T::TN>(e, tl.split, acc, bias, m0 + wm * T::TM * 32,
                                                     n0 + wn * T::TN * 32, lane);
    else
        epi_wave<MODE, GATHER, T::TM, T::TN>(e, tl.split, acc, bias, m0 + wm * T::TM * 32,
                                              n0 + wn * T::TN * 32, lane);
}

// ---------------------------------------------------------------- GEMM, split load roles
// Vector-memory loads of one wave complete in order, so a wave that feeds
// both the D stream (HBM, long latency) and the query stream (L2, short
// latency) can only run as far ahead as the shorter ring allows.  Here waves
// 0-1 load only D tiles into a deep ring of SA stages and waves 2-3 load only
// query tiles into a ring of SB stages; each wave waits on its own counter,
// then all four meet at the barrier and compute.  LWE form, no split.
template <int WM_, int WN_, int TM_, int TN_, int SA_, int SB_>
struct Roles {
    static constexpr int WM = WM_, WN = WN_, TM = TM_, TN = TN_, SA = SA_, SB = SB_;
    static constexpr int BK = 64;
    static constexpr int BM = WM * TM * 32;
    static constexpr int BN = WN * TN * 32;
    static constexpr int A_BYTES = BM * BK;
    static constexpr int B_BYTES = BN * BK;
    static constexpr int A_LOADS = BM / 16 / 2;          // per loader wave per tile
    static constexpr int B_LOADS = BN / 16 / 2;
    static constexpr int LDS_BYTES = SA * A_BYTES + SB * B_BYTES;
    static_assert(WM * WN == 4, "four waves");
    static_assert(TN % 4 == 0, "a wave covers whole groups of four limbs");
    static_assert(SA >= 2 && SB >= 2, "at least double buffering");
    static_assert((SA - 2) * A_LOADS < 64 && (SB - 2) * B_LOADS < 64, "vmcnt range");
    static_assert(LDS_BYTES <= 160 * 1024, "LDS");
};

template <class T, bool GATHER>
__global__ __launch_bounds__(256) void k_gemm_roles(const uint8_t* __restrict__ D, uint64_t pitch,
                                                    const int8_t* __restrict__ QL, uint32_t Cp,
                                                    uint32_t n_tiles, uint32_t m_tiles, Epi e) {
    extern __shared__ __attribute__((aligned(16))) uint8_t smem[];
    const uint32_t R = e.R, C = e.C, M = e.M;
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave / T::WN;
    const int wn = wave % T::WN;
    const bool loads_d = wave < 2;
    const int lw = wave & 1;                               // index among the loader pair

    const TileId tl = tile_of(xcd_remap(blockIdx.x, gridDim.x), n_tiles, m_tiles);
    const uint32_t m0 = tl.m * T::BM;
    const uint32_t n0 = tl.n * T::BN;

    constexpr int NL = T::A_LOADS > T::B_LOADS ? T::A_LOADS : T::B_LOADS;
    const uint8_t* src[NL];
    uint32_t seg_off[NL];
    const int lrow = lane >> 2;
#pragma unroll
    for (int i = 0; i < NL; ++i) {
        const int kb = lw + 2 * i;                         // 1 KiB block within the tile
        const int r = kb * 16 + lrow;
        const int seg = swz<64>(r, lane & 3);
        seg_off[i] = 16u * seg;
        if (loads_d) {
            uint32_t mi = m0 + (uint32_t)min(r, T::BM - 1);
            mi = mi < M ? mi : M - 1;
            uint32_t dr = GATHER ? e.rows[mi] : mi;
            dr = dr < R ? dr : R - 1;
            src[i] = D + (uint64_t)dr * pitch + seg_off[i];
        } else {
            src[i] = reinterpret_cast<const uint8_t*>(QL) +
                     ql_row(n0 + (uint32_t)min(r, T::BN - 1), Cp) + seg_off[i];
        }
    }
    const uint32_t ktiles = (C + T::BK - 1) / T::BK;
    uint8_t* ringA = smem;
    uint8_t* ringB = smem + T::SA * T::A_BYTES;

    auto issue = [&](uint32_t t) {
        const uint32_t k0 = t * T::BK;
        if (loads_d) {
            uint8_t* stage = ringA + (t % T::SA) * T::A_BYTES;
#pragma unroll
            for (int i = 0; i < T::A_LOADS; ++i) {
                uint8_t* dst = stage + (lw + 2 * i) * 1024;
                if (k0 + seg_off[i] + 16 <= C)
                    __builtin_amdgcn_global_load_lds((glb_void_t*)(src[i] + k0), (lds_void_t*)dst,
                                                     16, 0, 0);
            }
        } else {
            uint8_t* stage = ringB + (t % T::SB) * T::B_BYTES;
            const uint32_t kq = ql_col(k0);
#pragma unroll
            for (int i = 0; i < T::B_LOADS; ++i) {
                uint8_t* dst = stage + (lw + 2 * i) * 1024;
                __builtin_amdgcn_global_load_lds((glb_void_t*)(src[i] + kq), (lds_void_t*)dst,
                                                 16, 0, 0);
            }
        }
    };

    i32x16 acc[T::TM][T::TN];
#pragma unroll
    for (int a = 0; a < T::TM; ++a)
#pragma unroll
        for (int b = 0; b < T::TN; ++b)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[a][b][v] = 0;

    const int frow = lane & 31;
    const int fseg = lane >> 5;
    const u32x4 centre = u32x4{kCentreWord, kCentreWord, kCentreWord, kCentreWord};

    const int depth = loads_d ? T::SA : T::SB;
    for (int p = 0; p < depth - 1; ++p)
        if ((uint32_t)p < ktiles) issue(p);

    for (uint32_t t = 0; t < ktiles; ++t) {
        // Each loader wave waits for its own part of tile t (counting as in
        // k_gemm_ring; only D loads of the last tile can be skipped).
        if (loads_d) {
            if (t + T::SA - 1 < ktiles) wait_vmcnt<(T::SA - 2) * T::A_LOADS>();
            else wait_vmcnt<0>();
        } else {
            if (t + T::SB - 1 < ktiles) wait_vmcnt<(T::SB - 2) * T::B_LOADS>();
            else wait_vmcnt<0>();
        }
        ring_barrier();
        if (t + depth - 1 < ktiles) issue(t + depth - 1);

        const uint8_t* sa = ringA + (t % T::SA) * T::A_BYTES;
        const uint8_t* sb = ringB + (t % T::SB) * T::B_BYTES;
#pragma unroll
        for (int ks = 0; ks < T::BK / 32; ++ks) {
            const int seg = 2 * ks + fseg;
            i32x4 fa[T::TM], fb[T::TN];
#pragma unroll
            for (int a = 0; a < T::TM; ++a) {
                const int r = wm * T::TM * 32 + a * 32 + frow;
                u32x4 v = *reinterpret_cast<const u32x4*>(sa + r * T::BK + 16 * swz<64>(r, seg));
                v ^= centre;
                fa[a] = __builtin_bit_cast(i32x4, v);
            }
#pragma unroll
            for (int b = 0; b < T::TN; ++b) {
                const int r = wn * T::TN * 32 + b * 32 + frow;
                fb[b] = *reinterpret_cast<const i32x4*>(sb + r * T::BK + 16 * swz<64>(r, seg));
            }
#pragma unroll
            for (int a = 0; a < T::TM; ++a)
#pragma unroll
                for (int b = 0; b < T::TN; ++b)
                    acc[a][b] = __builtin_amdgcn_mfma_i32_32x32x32_i8(fa[a], fb[b], acc[a][b], 0, 0, 0);
        }
    }
    const int64_t bias[T::TN] = {};
    epi_wave<kFinal32, GATHER, T::TM, T::TN, T::TM == 4>(e, 0, acc, bias, m0 + wm * T::TM * 32,
                                              n0 + wn * T::TN * 32, lane);
}

// ---------------------------------------------------------------- dispatch
struct Gemm {
    const pir_db_t* db;
    const int8_t* QL;
    uint32_t Cp, N;
    Epi e;
    uint32_t splits, kts;   // split-K pieces and k-tiles per piece
    bool exact;             // field form
};

uint32_t g_cus = 256;       // compute units of the device (set at init)
uint64_t g_max_grid_y = 65535;   // largest grid y extent of the device (set at init)

uint32_t ceil_div(uint64_t a, uint64_t b) { return (uint32_t)((a + b - 1) / b); }

// With one column tile (a batch no wider than the tile), each byte of D is
// read by one workgroup only, so D's loads are marked non-temporal and do
// not evict the limb planes every workgroup re-reads.
template <class T, bool GATHER, int MODE, bool SUMS>
pir_status launch_ring_sums(const Gemm& g, uint32_t n_tiles, uint32_t m_tiles, hipStream_t s) {
    const uint64_t blocks = (uint64_t)n_tiles * m_tiles * g.splits;
    if (blocks > 0x7FFFFFFFull) return PIR_ERR_SHAPE;
    bool nt = false;
    if constexpr (!GATHER) {
        if (n_tiles == 1) {
            nt = true;
            k_gemm_ring<T, false, MODE, true, SUMS>
                <<<(uint32_t)blocks, T::THREADS, T::LDS_BYTES, s>>>(
                    g.db->D, g.db->pitch, g.QL, g.Cp, n_tiles, m_tiles, g.kts, g.e);
        }
    }
    if (!nt)
        k_gemm_ring<T, GATHER, MODE, false, SUMS><<<(uint32_t)blocks, T::THREADS, T::LDS_BYTES, s>>>(
            g.db->D, g.db->pitch, g.QL, g.Cp, n_tiles, m_tiles, g.kts, g.e);
    PIR_LAUNCH_CHECK();
    return PIR_OK;
}

// Whether a tile has the summing kernel: at most 128 limb rows.
template <class T>
constexpr bool can_sum() {
    return T::BN <= 128;
}

template <class T, bool GATHER, int MODE>
pir_status launch_ring_mode(const Gemm& g, uint32_t n_tiles, uint32_t m_tiles, hipStream_t s) {
    if constexpr (can_sum<T>() && !GATHER) {
        if (!g.e.colsum) return launch_ring_sums<T, GATHER, MODE, true>(g, n_tiles, m_tiles, s);
    }
    if constexpr (T::BN < 128 && !GATHER) return PIR_ERR_UNSUPPORTED;   // always summed (tile_sums)
    else return launch_ring_sums<T, GATHER, MODE, false>(g, n_tiles, m_tiles, s);
}

template <class T>
pir_status launch_ring(const Gemm& g, hipStream_t s) {
    const uint32_t n_tiles = ceil_div(g.N, T::BN);
    const uint32_t m_tiles = ceil_div(g.e.M, T::BM);
    const bool gather = g.e.rows != nullptr;
    if (g.exact) {
        if (gather) return PIR_ERR_UNSUPPORTED;
        if (g.splits > 1) return launch_ring_mode<T, false, kPart64>(g, n_tiles, m_tiles, s);
        return launch_ring_mode<T, false, kFinalModP>(g, n_tiles, m_tiles, s);
    }
    if (g.splits > 1) {
        if (gather) return launch_ring_mode<T, true, kPart32>(g, n_tiles, m_tiles, s);
        if (g.e.by_rows) return launch_ring_mode<T, false, kPart32Rows>(g, n_tiles, m_tiles, s);
        return launch_ring_mode<T, false, kPart32>(g, n_tiles, m_tiles, s);
    }
    if (gather) return launch_ring_mode<T, true, kFinal32>(g, n_tiles, m_tiles, s);
    if (g.e.by_rows) return launch_ring_mode<T, false, kFinal32Rows>(g, n_tiles, m_tiles, s);
    return launch_ring_mode<T, false, kFinal32>(g, n_tiles, m_tiles, s);
}

// The client's products (limb planes with zeroed limbs, see k_gemm_ring).
// One column tile covers the batch where the tile is wide enough.
template <class T>
pir_status launch_client(const Gemm& g, int mode, hipStream_t s) {
    const uint32_t n_tiles = ceil_div(g.N, T::BN);
    const uint32_t m_tiles = ceil_div(g.e.M, T::BM);
    const uint64_t blocks = (uint64_t)n_tiles * m_tiles * g.splits;
    if (blocks > 0x7FFFFFFFull) return PIR_ERR_SHAPE;
#define PIR_CLIENT(MODE)                                                                       \
    k_gemm_ring<T, false, MODE, false, (T::BN <= 128), true>                                  \
        <<<(uint32_t)blocks, T::THREADS, T::LDS_BYTES, s>>>(                                   \
        g.db->D, g.db->pitch, g.QL, g.Cp, n_tiles, m_tiles, g.kts, g.e)
    if (mode == kPart32Rows) PIR_CLIENT(kPart32Rows);
    else if (mode == kClientQuery) PIR_CLIENT(kClientQuery);
    else PIR_CLIENT(kClientDecode);
#undef PIR_CLIENT
    PIR_LAUNCH_CHECK();
    return PIR_OK;
}

template <class T>
pir_status set_client_lds() {
    const void* fns[] = {
        (const void*)k_gemm_ring<T, false, kPart32Rows, false, (T::BN <= 128), true>,
        (const void*)k_gemm_ring<T, false, kClientQuery, false, (T::BN <= 128), true>,
        (const void*)k_gemm_ring<T, false, kClientDecode, false, (T::BN <= 128), true>,
    };
    for (const void* f : fns)
        if (hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, T::LDS_BYTES) !=
            hipSuccess)
            return PIR_ERR_DEVICE;
    return PIR_OK;
}

template <class T, bool SUMS>
pir_status set_ring_lds_sums() {
    const void* fns[] = {
        (const void*)k_gemm_ring<T, false, kFinal32, false, SUMS>,
        (const void*)k_gemm_ring<T, false, kPart32, false, SUMS>,
        (const void*)k_gemm_ring<T, false, kFinal32Rows, false, SUMS>,
        (const void*)k_gemm_ring<T, false, kPart32Rows, false, SUMS>,
        (const void*)k_gemm_ring<T, false, kPart64, false, SUMS>,
        (const void*)k_gemm_ring<T, false, kFinalModP, false, SUMS>,
        (const void*)k_gemm_ring<T, false, kFinal32, true, SUMS>,
        (const void*)k_gemm_ring<T, false, kPart32, true, SUMS>,
        (const void*)k_gemm_ring<T, false, kFinal32Rows, true, SUMS>,
        (const void*)k_gemm_ring<T, false, kPart32Rows, true, SUMS>,
        (const void*)k_gemm_ring<T, false, kPart64, true, SUMS>,
        (const void*)k_gemm_ring<T, false, kFinalModP, true, SUMS>,
    };
    for (const void* f : fns)
        if (hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, T::LDS_BYTES) !=
            hipSuccess)
            return PIR_ERR_DEVICE;
    return PIR_OK;
}

template <class T>
pir_status set_ring_lds() {
    if constexpr (can_sum<T>()) {
        const pir_status st = set_ring_lds_sums<T, true>();
        if (st != PIR_OK) return st;
    }
    if constexpr (T::BN >= 128) {
        const pir_status st = set_ring_lds_sums<T, false>();
        if (st != PIR_OK) return st;
    }
    const void* fns[] = {
        (const void*)k_gemm_ring<T, true, kFinal32, false, false>,
        (const void*)k_gemm_ring<T, true, kPart32, false, false>,
    };
    for (const void* f : fns)
        if (hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, T::LDS_BYTES) !=
            hipSuccess)
            return PIR_ERR_DEVICE;
    return PIR_OK;
}

template <class T>
pir_status launch_roles(const Gemm& g, hipStream_t s) {
    if (g.exact || g.splits != 1) return PIR_ERR_UNSUPPORTED;
    const uint32_t n_tiles = ceil_div(g.N, T::BN);
    const uint32_t m_tiles = ceil_div(g.e.M, T::BM);
    const uint64_t blocks = (uint64_t)n_tiles * m_tiles;
    if (blocks > 0x7FFFFFFFull) return PIR_ERR_SHAPE;
    if (g.e.rows)
        k_gemm_roles<T, true><<<(uint32_t)blocks, 256, T::LDS_BYTES, s>>>(
            g.db->D, g.db->pitch, g.QL, g.Cp, n_tiles, m_tiles, g.e);
    else
        k_gemm_roles<T, false><<<(uint32_t)blocks, 256, T::LDS_BYTES, s>>>(
            g.db->D, g.db->pitch, g.QL, g.Cp, n_tiles, m_tiles, g.e);
    PIR_LAUNCH_CHECK();
    return PIR_OK;
}

template <class T>
pir_status set_roles_lds() {
    if (hipFuncSetAttribute((const void*)k_gemm_roles<T, false>,
                            hipFuncAttributeMaxDynamicSharedMemorySize, T::LDS_BYTES) != hipSuccess ||
        hipFuncSetAttribute((const void*)k_gemm_roles<T, true>,
                            hipFuncAttributeMaxDynamicSharedMemorySize, T::LDS_BYTES) != hipSuccess)
        return PIR_ERR_DEVICE;
    return PIR_OK;
}

template <class T>
pir_status launch_reg(const Gemm& g, hipStream_t s) {
    if (g.exact) return PIR_ERR_UNSUPPORTED;
    const uint32_t n_tiles = ceil_div(g.N, T::BN);
    const uint32_t m_tiles = ceil_div(g.e.M, T::BM);
    const uint64_t blocks = (uint64_t)n_tiles * m_tiles * g.splits;
    if (blocks > 0x7FFFFFFFull) return PIR_ERR_SHAPE;
    const pir_db_t* db = g.db;
#define PIR_GEMM(GATHER, MODE)                                                              \
    k_gemm<T, GATHER, MODE><<<(uint32_t)blocks, T::THREADS, T::LDS_BYTES, s>>>(             \
        db->D, db->pitch, g.QL, g.Cp, n_tiles, m_tiles, g.kts, g.e)
    if (g.splits > 1) {
        if (g.e.rows) PIR_GEMM(true, kPart32);
        else if (g.e.by_rows) PIR_GEMM(false, kPart32Rows);
        else PIR_GEMM(false, kPart32);
    } else {
        if (g.e.rows) PIR_GEMM(true, kFinal32);
        else if (g.e.by_rows) PIR_GEMM(false, kFinal32Rows);
        else PIR_GEMM(false, kFinal32);
    }
#undef PIR_GEMM
    PIR_LAUNCH_CHECK();
    return PIR_OK;
}

template <class T>
pir_status set_reg_lds() {
    const void* fns[] = {
        (const void*)k_gemm<T, false, kFinal32>, (const void*)k_gemm<T, true, kFinal32>,
        (const void*)k_gemm<T, false, kPart32>, (const void*)k_gemm<T, true, kPart32>,
        (const void*)k_gemm<T, false, kFinal32Rows>, (const void*)k_gemm<T, false, kPart32Rows>,
    };
    for (const void* f : fns)
        if (hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, T::LDS_BYTES) !=
            hipSuccess)
            return PIR_ERR_DEVICE;
    return PIR_OK;
}

// Kernel variants of the batched product.  Ring and roles variants may be
// pinned on a 16-byte aligned database with C a multiple of 16; 256-wide tiles
// need N a multiple of 256 (batches above 32 queries, padded to 64).  Ring
// variants split K (and so serve the field form), register-staged ones on the
// databases the ring does not serve.
using Ring128x128S8 = Ring<4, 1, 1, 4, 8>;              // 128 KiB LDS
using Ring128x128K128S4 = Ring<4, 1, 1, 4, 4, 128>;     // 128 KiB, 128-byte stages
using Ring128x256S6 = Ring<2, 2, 2, 4, 6>;              // 144 KiB
using Ring8w128x256K128S3 = Ring<4, 2, 1, 4, 3, 128>;   // 8 waves, 144 KiB
using Ring8w256x256S4 = Ring<4, 2, 2, 4, 4>;            // 8 waves, 128 KiB
using Ring8w256x256K128S2 = Ring<4, 2, 2, 4, 2, 128>;   // 8 waves, 128 KiB
// The same with a third D slot (D two tiles ahead, QL one): 160 KiB.
using Ring8w256x256K128D3 = Ring<4, 2, 2, 4, 2, 128, false, 1>;
// 128 x 256 with four D slots and three QL slots: 160 KiB.
using Ring8w128x256K128D4 = Ring<4, 2, 1, 4, 3, 128, false, 1>;
// 128 x 256 with five D slots (D four tiles ahead) and two QL slots: 144 KiB.
using Ring8w128x256K128D5 = Ring<4, 2, 1, 4, 2, 128, false, 3>;
// 256 x 256 with a third QL slot (limb planes two tiles ahead): 160 KiB.
using Ring8w256x256K128Q3 = Ring<4, 2, 2, 4, 2, 128, false, 0, 1>;
// Narrow tiles with deeper D rings: 256 x 32 with 4 D / 3 QL slots (140 KiB),
// 128 x 32 with 8 D / 6 QL slots (152 KiB).
using Narrow256x32K128D4 = Ring<4, 1, 2, 1, 3, 128, true, 1>;
using Narrow128x32K128D8 = Ring<4, 1, 1, 1, 6, 128, true, 2>;
using Ring256x256K128S2 = Ring<2, 2, 4, 4, 2, 128>;     // 4 waves of 128 x 128, 128 KiB
// The same with the D or the limb-plane ring one tile deeper (160 KiB): a
// 128 x 128 wave tile reads 0.5 KiB of LDS fragments per MFMA against 0.75
// for the 8-wave tile's 64 x 128.
using Ring256x256K128D3 = Ring<2, 2, 4, 4, 2, 128, false, 1>;
using Ring256x256K128Q3 = Ring<2, 2, 4, 4, 2, 128, false, 0, 1>;
// Two workgroups per CU (64 KiB each): the waves sharing a SIMD belong to
// different workgroups, so one's barrier does not idle the other.
using Ring128x128K128S2 = Ring<4, 1, 1, 4, 2, 128>;
// Narrow layout (8 queries per 32-column tile), one column tile per batch.
using Narrow256x32K128S4 = Ring<4, 1, 2, 1, 4, 128, true>;    // <= 8 queries, 144 KiB
using Narrow256x64K128S4 = Ring<8, 1, 1, 2, 4, 128, true>;    // <= 16 queries, 160 KiB
using Narrow128x32K128S6 = Ring<4, 1, 1, 1, 6, 128, true>;    // <= 8 queries, 120 KiB
using Roles256x256A5B4 = Roles<2, 2, 4, 4, 5, 4>;       // 80 + 64 KiB
using Roles128x256A10B4 = Roles<2, 2, 2, 4, 10, 4>;     // 80 + 64 KiB
using Reg128x256 = Tile<4, 2, 1, 4>;                     // 8 waves, 96 KiB
using Reg128x128 = Tile<4, 1, 1, 4>;                     // 4 waves, 64 KiB: two per CU
using Reg256x256 = Tile<4, 2, 2, 4>;                     // 8 waves, 128 KiB

enum Kind : uint8_t { kAuto, kRing, kRoles, kReg, kFew };

struct VariantInfo {
    const char* name;
    Kind kind;
    uint32_t bm, bn, bk;
    pir_status (*launch)(const Gemm&, hipStream_t);
    uint32_t per_cu;        // workgroups resident per CU (LDS-limited ring variants)
    bool narrow;            // narrow QL layout: all queries in one column tile
    pir_status (*client)(const Gemm&, int mode, hipStream_t);   // client's products, or null
};

constexpr VariantInfo kVariants[] = {
    {"auto", kAuto, 0, 0, 0, nullptr},
    {"ring_128x128_s8", kRing, 128, 128, 64, launch_ring<Ring128x128S8>},
    {"ring_128x128_k128_s4", kRing, 128, 128, 128, launch_ring<Ring128x128K128S4>},
    {"ring_128x256_s6", kRing, 128, 256, 64, launch_ring<Ring128x256S6>},
    {"ring8w_128x256_k128_s3", kRing, 128, 256, 128, launch_ring<Ring8w128x256K128S3>, 1, false,
     launch_client<Ring8w128x256K128S3>},
    {"ring8w_256x256_s4", kRing, 256, 256, 64, launch_ring<Ring8w256x256S4>},
    {"ring8w_256x256_k128_s2", kRing, 256, 256, 128, launch_ring<Ring8w256x256K128S2>, 1, false,
     launch_client<Ring8w256x256K128S2>},
    {"ring_256x256_k128_s2", kRing, 256, 256, 128, launch_ring<Ring256x256K128S2>},
    {"roles_256x256_a5b4", kRoles, 256, 256, 64, launch_roles<Roles256x256A5B4>},
    {"roles_128x256_a10b4", kRoles, 128, 256, 64, launch_roles<Roles128x256A10B4>},
    {"reg_128x256", kReg, 128, 256, 128, launch_reg<Reg128x256>},
    {"reg_128x128", kReg, 128, 128, 128, launch_reg<Reg128x128>, 2},
    {"few", kFew, 0, 0, 0, nullptr},   // dot4 stream, batches of at most kFewMax
    {"ring_128x128_k128_s2", kRing, 128, 128, 128, launch_ring<Ring128x128K128S2>, 2, false,
     launch_client<Ring128x128K128S2>},
    {"narrow_256x32_k128_s4", kRing, 256, 32, 128, launch_ring<Narrow256x32K128S4>, 1, true},
    {"narrow_256x64_k128_s4", kRing, 256, 64, 128, launch_ring<Narrow256x64K128S4>, 1, true},
    {"narrow_128x32_k128_s6", kRing, 128, 32, 128, launch_ring<Narrow128x32K128S6>, 1, true},
    {"ring8w_256x256_k128_d3q2", kRing, 256, 256, 128, launch_ring<Ring8w256x256K128D3>},
    {"ring8w_128x256_k128_d4q3", kRing, 128, 256, 128, launch_ring<Ring8w128x256K128D4>},
    {"ring8w_128x256_k128_d5q2", kRing, 128, 256, 128, launch_ring<Ring8w128x256K128D5>},
    {"ring8w_256x256_k128_d2q3", kRing, 256, 256, 128, launch_ring<Ring8w256x256K128Q3>},
    {"narrow_256x32_k128_d4q3", kRing, 256, 32, 128, launch_ring<Narrow256x32K128D4>, 1, true},
    {"narrow_128x32_k128_d8q6", kRing, 128, 32, 128, launch_ring<Narrow128x32K128D8>, 1, true},
    {"ring_256x256_k128_d3q2", kRing, 256, 256, 128, launch_ring<Ring256x256K128D3>},
    {"ring_256x256_k128_d2q3", kRing, 256, 256, 128, launch_ring<Ring256x256K128Q3>},
    {"reg_256x256", kReg, 256, 256, 128, launch_reg<Reg256x256>},
};
constexpr uint32_t kNumVariants = sizeof(kVariants) / sizeof(kVariants[0]);
constexpr uint32_t kVarRing128 = 2, kVarRing256 = 4, kVarReg128x256 = 10, kVarReg128 = 11,
                   kVarFew = 12, kVarRing128x2 = 13, kVarNarrow256 = 15, kVarNarrow128 = 16,
                   kVarRing4wD3 = 23, kVarReg256 = 25;
constexpr bool same_name(const char* a, const char* b) {
    return *a == *b && (*a == '\0' || same_name(a + 1, b + 1));
}
// The built-in choices name table rows by index: keep them on their rows.
static_assert(same_name(kVariants[kVarRing128].name, "ring_128x128_k128_s4") &&
                  same_name(kVariants[kVarRing256].name, "ring8w_128x256_k128_s3") &&
                  same_name(kVariants[kVarReg256].name, "reg_256x256") &&
                  same_name(kVariants[kVarReg128].name, "reg_128x128") &&
                  same_name(kVariants[kVarReg128x256].name, "reg_128x256") &&
                  same_name(kVariants[kVarRing128x2].name, "ring_128x128_k128_s2") &&
                  same_name(kVariants[kVarNarrow256].name, "narrow_256x64_k128_s4") &&
                  same_name(kVariants[kVarNarrow128].name, "narrow_128x32_k128_s6") &&
                  same_name(kVariants[kVarFew].name, "few") &&
                  same_name(kVariants[kVarRing4wD3].name, "ring_256x256_k128_d3q2"),
              "default variant indices");

// Databases the ring kernels may be pinned for and the field form runs on.
bool ring_ok(const pir_db_t* db) { return db->aligned && (db->cols % 16 == 0); }

// Databases the ring serves: aligned rows of any length (a row's last 16-byte
// segment lies inside its pitch).  37 and 200 queries on 20000 rows of 10007
// bytes, pitch 10240: 75 and 225 us, against 166 and 454 us while rows whose
// length is not a multiple of 16 went through registers.
bool ring_serves(const pir_db_t* db) { return db->aligned; }

uint32_t padded_batch(uint32_t B) { return B <= 32u ? 32u : (B + 63u) / 64u * 64u; }

// Queries a variant's QL layout holds for batch B: narrow variants hold one
// column tile (BN / 4 queries), the others B padded to 32 or to 64.
uint32_t layout_batch(const VariantInfo& vi, uint32_t B) {
    return vi.narrow ? vi.bn / 4u : padded_batch(B);
}

bool variant_valid(const pir_db_t* db, uint32_t B, uint32_t v) {
    if (v == 0) return true;
    if (v >= kNumVariants) return false;
    const VariantInfo& vi = kVariants[v];
    if (vi.kind == kFew) return B <= kFewMax;
    if (vi.kind != kReg && !ring_ok(db)) return false;
    if (vi.narrow) return 4u * B <= vi.bn;
    return (4u * padded_batch(B)) % vi.bn == 0;
}

struct SplitPlan {
    uint32_t splits, kts;
    double us;              // estimated time of the product and its finish
};

// Time of one k-tile of a workgroup with the chip full, microseconds: what a
// CU's share of the memory (6.7 TB/s of database bytes), of the loads into
// LDS (both operands, 10.8 TB/s) or of the matrix cores (2.2 POP/s) takes;
// workgroups on one CU share them, and register-staged tiles pay their LDS
// stores on top (15%; 128 x 256, whose eight waves each wait for few loads,
// 60%: 64 queries on unaligned 20000 x 10007 bytes 113 us, 256 x 256 85).  Against whole calls: 128 x 32 0.63 (60000 x 12000 0.61,
// 32768 x 32768 0.73), 128 x 128 0.78 (0.76-0.83), 128 x 256 1.17 (1.05-1.3),
// 256 x 256 1.95 (1.9-2.1).
double ktile_us(const VariantInfo& vi) {
    const double bytes = vi.bm / 26e3, lds = (vi.bm + vi.bn) / 42e3;
    const double ops = 2.0 * vi.bm * vi.bn / 8.6e6;
    const double us = vi.bk * std::max({bytes, lds, ops}) * std::max(1u, vi.per_cu);
    return vi.kind == kReg ? (vi.bm < vi.bn ? 1.6 : 1.15) * us : us;
}

// Split-K plan for a ring variant.  LDS lets one or two ring workgroups
// (per_cu) reside on a CU, so a launch runs in ceil(tiles * S / slots)
// rounds of 1/S of the K range each, slots = CUs * per_cu, and each round
// also fills and drains the ring (about kFillTiles k-tiles); splitting adds
// the finish launch, a pass of it per piece, and one write and one read of S
// partials.  The plan is
// the S (up to kMaxSplits, at least two k-tiles per piece) of the least sum,
// looked for below two rounds of tiles; for a number of rounds the best S is
// the most that fits in them or, if less, where the partials' growth meets
// the product's gain.  With the partials at a flat 0.5% of the product per
// piece, a few ten thousand rows were split far too often: 60000 x 12000, 64
// queries in 13 pieces, 390 us, whole 243.  The field form also caps each
// piece at kExactSpan columns.
// `reg`: register-staged tiles split too (on databases the ring does not
// serve; elsewhere they are only run when pinned, whole).
constexpr double kFillTiles = 3, kFinishUs = 3, kPieceUs = 0.3, kPartialBytesPerUs = 5e6;

// Rounds of tiles a plan may split into: tiles that fill more than half the
// chip gain by pieces in up to four (1024 field queries on 3072 x 2^18, 192
// tiles: four pieces in three rounds 3.4 ms, two in two 4.2), fewer tiles
// fill one or two well.
constexpr uint64_t max_rounds(uint64_t tiles, uint64_t slots) { return 2 * tiles > slots ? 4 : 2; }

// Writing and reading the partials of one piece of `rows` rows and N limb rows.
double part_us(uint32_t rows, uint32_t N, bool exact) {
    return 2.0 * (exact ? 8 : 4) * (double)rows * (N / 4) / kPartialBytesPerUs;
}

SplitPlan plan_splits(uint32_t M, uint32_t N, uint32_t C, const VariantInfo& vi, bool exact,
                      bool reg) {
    const uint32_t ktiles = ceil_div(C, vi.bk);
    const uint64_t mt = ceil_div(M, vi.bm), tiles = mt * ceil_div(N, vi.bn);
    const uint64_t slots = (uint64_t)g_cus * std::max(1u, vi.per_cu);
    const double tk = ktile_us(vi);
    // Per piece, from whole tiles: one bound for every M of as many tiles.
    const double part = kPieceUs + (double)mt * part_us(vi.bm, N, exact);
    SplitPlan best{1u, ktiles, 1e30};
    auto consider = [&](uint64_t want) {
        const uint32_t kts = ceil_div(ktiles, (uint32_t)want);
        const uint32_t sp = ceil_div(ktiles, kts);
        const double us = (double)ceil_div(tiles * sp, slots) * (kts + kFillTiles) * tk +
                          (sp > 1 ? kFinishUs + sp * part : 0.0);
        if (us < best.us) best = {sp, kts, us};
    };
    const bool can_split = (vi.kind == kRing || (reg && vi.kind == kReg)) && ktiles != 0 && tiles != 0;
    if (!can_split) {
        best.us = (double)ceil_div(tiles, slots) * (ktiles + kFillTiles) * tk;
        return best;
    }
    const uint64_t lo = exact ? ceil_div(ktiles, kExactSpan / vi.bk) : 1u;
    consider(lo);
    if (tiles < 2ull * slots) {
        const uint64_t hi = std::max<uint64_t>(lo, std::min(kMaxSplits, ktiles / 2));
        for (uint64_t r = 1; r <= max_rounds(tiles, slots); ++r) {
            const uint64_t fit = r * slots / tiles;
            const uint64_t gain = (uint64_t)std::sqrt(r * ktiles * tk / part);
            consider(std::max(lo, std::min({hi, fit, gain})));
        }
    }
    return best;
}

// Matrix-core choice (any batch size, gathered rows allowed): of the tiles
// that led the autotuner somewhere, the one whose plan takes least time.
// Large databases get the tiles that a rule on the batch alone gave (128 x
// 128 up to 32 queries, 256 x 256 above); small ones, whose tiles leave
// CUs idle, smaller tiles, and up to 8 and 16 queries the narrow tiles,
// which stage a quarter and half of the query bytes.  Whole calls, microseconds, with the rule
// on the batch alone (and its split plan) and with this one:
//                     8 queries      48           128          256
//   2000 x 5000      18.8   17.7   30.0  21.0   34.6  24.5   38.6  32.7
//   1500 x 30000     30.4   23.9   53.0  41.7   60.0  51.8   76.3  77.9
//   20000 x 10007    67.9   46.6   76.4  72.4    160   132    246   244
//   60000 x 12000     186    119    288   195    489   371    732   718
// `wide`: the limb planes are laid out already, or rows gathered: no narrow
// tile.
uint32_t priced_gemm(const pir_db_t* db, uint32_t B, uint32_t M, bool exact, bool wide) {
    static constexpr uint32_t ring[] = {kVarNarrow128, kVarNarrow256, kVarRing128,
                                        kVarRing128x2, kVarRing256,   kVarRing4wD3};
    static constexpr uint32_t reg[] = {kVarReg128, kVarReg128x256, kVarReg256};
    const bool staged = !ring_serves(db);
    const uint32_t* list = staged ? reg : ring;
    const size_t n = staged ? std::size(reg) : std::size(ring);
    uint32_t best = staged ? kVarReg128 : kVarRing128;
    double best_us = 1e30;
    for (size_t i = 0; i < n; ++i) {
        const VariantInfo& vi = kVariants[list[i]];
        if (vi.narrow ? wide || 4u * B > vi.bn : (4u * padded_batch(B)) % vi.bn != 0) continue;
        const uint32_t N = 4u * layout_batch(vi, B);
        const double us = plan_splits(M, N, (uint32_t)db->cols, vi, exact, staged).us;
        if (us < best_us) {
            best_us = us;
            best = list[i];
        }
    }
    return best;
}

// Pricing takes up to 0.3 us; the choice for whole-database products is kept
// in the handle (racing writers store the same value).
uint32_t default_gemm(const pir_db_t* db, uint32_t B, uint32_t M, bool exact, bool wide) {
    if (wide || M != db->rows) return priced_gemm(db, B, M, exact, wide);
    std::atomic<uint32_t>& slot = db->tile[exact][batch_bucket(B)];
    const uint32_t kept = slot.load(std::memory_order_relaxed);
    if (kept >> 8 == B) return kept & 0xFFu;
    const uint32_t v = priced_gemm(db, B, M, exact, false);
    slot.store((B << 8) | v, std::memory_order_relaxed);
    return v;
}

// The dot4 stream beats the padded matrix-core tile up to two queries; at
// four it is bound by VALU issue (measured at 32768 x 32768: 173 vs 254 us
// for one query, 194 vs 236 us for two, 400 vs 224 us for four), which
// databases of up to kFewSmall bytes, bound by launches, do not notice (one
// launch or two instead of three; four queries: 1024 x 1024 12-14 vs 16-18
// us, 5000 x 2001 16 vs 17-21, 4096 x 4096 16 vs 17; 30000 x 3000 38 vs 31).
// Rows shorter than a wave's load leave its lanes idle and count as whole
// ones: few of them still run best in the stream (3277 x 1017 11.9 vs 21 us,
// 13312 x 72 11.5 vs 14.7), many in the tile (GPU time 65536 x 256 22.8 vs 14.2,
// 2^18 x 64 81 vs 33, 2^20 x 16 320 vs 112), where the stream's partials would
// also outgrow a fixed scratch.
constexpr uint32_t kFewDefault = 2;
constexpr uint64_t kFewSmall = 1ull << 24;
constexpr uint64_t kFewCols = 1024;

bool few_default(const pir_db_t* db, uint32_t B) {
    return B <= kFewDefault ||
           (B <= kFewMax && db->rows * std::max(db->cols, kFewCols) <= kFewSmall);
}

// Gathered rows (the incremental hint): scattered row addresses add
// address-translation latency, which the three-stage 128 x 256 ring hides
// best.  Whole call, 1311 scattered rows of the 131072 x 131072 database,
// n = 1024, on two machines: 1001-1019 us, against 1007-1294 us for the
// two-stage 256 x 256 tile that is fastest over the whole database (that
// one took 1146 us for the same rows sorted, 980 us for consecutive rows).
uint32_t default_rows(const pir_db_t* db, uint32_t B, uint32_t m) {
    return ring_serves(db) && padded_batch(B) >= 64u ? kVarRing256
                                                     : default_gemm(db, B, m, false, true);
}

struct BatchLayout {
    uint32_t Bp, N, Cp;     // queries in the QL layout, its limb rows, padded columns
    size_t colsum_off, part_off, total;
};

// At least the partial words of a query, splits x output rows, of any plan
// that cuts `vi`'s tiles into pieces for occupancy, on up to R rows (gathered
// calls have fewer rows, and so may split more).  The loops follow
// plan_splits: S pieces of mt row tiles in `r` rounds are only chosen where
// they take less time than whole tiles in u rounds, which bounds mt.
// What fills those rounds bounds them all, and the search ends near it, or
// where it cannot pass `least`.
uint64_t worst_pieces(uint64_t R, uint32_t C, const VariantInfo& vi, uint32_t nt, bool exact,
                      uint64_t least) {
    const uint32_t ktiles = ceil_div(C, vi.bk);
    const uint64_t slots = (uint64_t)g_cus * std::max(1u, vi.per_cu);
    const uint64_t mt_all = ceil_div(R, vi.bm), hi = std::min(kMaxSplits, ktiles / 2);
    const uint64_t most = std::min(hi * R, max_rounds(mt_all * nt, slots) * slots / nt * vi.bm);
    if (hi < 2 || most <= least) return least;
    const double tk = ktile_us(vi);
    const double part_mt = part_us(vi.bm, nt * vi.bn, exact);   // per piece and row tile
    uint64_t worst = least;
    uint32_t kts_before = 0;
    for (uint64_t S = 2; S <= hi; ++S) {
        const uint32_t kts = ceil_div(ktiles, (uint32_t)S);
        if (kts == kts_before) continue;   // fewer pieces than S: the same plan
        kts_before = kts;
        const double gain1 = (ktiles + kFillTiles) * tk, piece = (kts + kFillTiles) * tk;
        const double fixed = kFinishUs + S * kPieceUs - 1e-3;
        for (uint64_t u = 1; u <= 2; ++u) {
            for (uint64_t r = 1; r <= 4; ++r) {
                const double room = u * gain1 - r * piece - fixed;
                if (room <= 0) break;
                const uint64_t mt = std::min({mt_all, r * slots / (S * nt), u * slots / nt,
                                              (uint64_t)std::min(room / (S * part_mt), 1e9)});
                if (mt == 0 || (u == 2 && mt * nt <= slots)) continue;
                if (r > max_rounds(mt * nt, slots)) continue;
                worst = std::max(worst, S * std::min<uint64_t>(R, mt * vi.bm));
            }
        }
        if (worst + worst / 32 >= most) return most;
    }
    return worst;
}

// At least the partial words of a query of any split-K plan for the batches
// whose wide layout has N limb columns (exact partials count two words): every
// ring variant valid for them (narrow variants, one column tile, for N = 128:
// batches of at most 32), and the exact form's fewest pieces.  On a database
// the ring does not serve, every register-staged variant instead.
uint64_t worst_split_words(const pir_db_t* db, uint32_t N_wide) {
    const uint64_t R = db->rows;
    const uint32_t C = (uint32_t)db->cols;
    const bool exact_ok = C <= kMaxExactCols && ring_ok(db);
    const bool reg = !ring_serves(db);
    uint64_t worst = 0;
    for (uint32_t v = 1; v < kNumVariants; ++v) {
        const VariantInfo& vi = kVariants[v];
        if (vi.kind != (reg ? kReg : kRing)) continue;
        if (vi.narrow ? N_wide != 128u : N_wide % vi.bn != 0) continue;
        bool seen = false;   // the same tile under another pipeline
        for (uint32_t w = 1; w < v && !seen; ++w) {
            const VariantInfo& o = kVariants[w];
            seen = o.kind == vi.kind && o.bm == vi.bm && o.bn == vi.bn && o.bk == vi.bk &&
                   std::max(1u, o.per_cu) == std::max(1u, vi.per_cu);
        }
        if (seen) continue;
        const uint32_t nt = vi.narrow ? 1u : N_wide / vi.bn;
        worst = worst_pieces(R, C, vi, nt, false, worst);
        if (!exact_ok) continue;
        const uint32_t ktiles = ceil_div(C, vi.bk);
        const uint64_t lo = ceil_div(ktiles, kExactSpan / vi.bk);
        if (lo <= 1) {
            worst = std::max(worst, 2 * worst_pieces(R, C, vi, nt, true, worst / 2));
        } else {   // the pieces fill at most max_rounds rounds, or are the fewest
            const uint64_t slots = (uint64_t)g_cus * std::max(1u, vi.per_cu);
            const uint64_t rounds = max_rounds((uint64_t)nt * ceil_div(R, vi.bm), slots);
            const uint64_t hi = std::min(kMaxSplits, ktiles / 2);
            worst = std::max({worst, 2 * lo * R, 2 * std::min(hi * R, rounds * slots / nt * vi.bm)});
        }
    }
    return worst;
}

// Split-K partial bytes the workspace reserves for batch B.  The bound takes
// some microseconds and is kept in the handle per padded-batch bucket (racing
// writers store the same value).
size_t partial_bound(const pir_db_t* db, uint32_t B, uint32_t N) {
    std::atomic<uint64_t>& slot = db->split_words[batch_bucket(N / 4)];
    uint64_t cached = slot.load(std::memory_order_relaxed);
    uint64_t worst;
    if (cached != 0 && (cached >> 40) == N) {
        worst = cached & ((1ull << 40) - 1);
    } else {
        worst = worst_split_words(db, N);
        slot.store(((uint64_t)N << 40) | worst, std::memory_order_relaxed);
    }
    return worst ? round_up((size_t)worst * B * 4, kWsAlign) : 0;
}

// Workspace: limb planes, exact column sums, split-K partials.  The
// partial bound covers every variant (it depends on the wide layout only),
// and the wide layout's limb planes are the larger, so mfma_workspace_bytes
// uses the wide layout.
BatchLayout batch_layout(const pir_db_t* db, uint32_t B, const VariantInfo& vi) {
    BatchLayout L;
    L.Bp = layout_batch(vi, B);
    L.N = 4u * L.Bp;
    L.Cp = (uint32_t)round_up(db->cols, kKPad);
    L.colsum_off = round_up((size_t)L.N * L.Cp, kWsAlign);
    L.part_off = L.colsum_off + round_up((size_t)L.Bp * 8, kWsAlign);
    L.total = L.part_off + partial_bound(db, B, 4u * padded_batch(B));
    return L;
}

}  // namespace

pir_status mfma_init() {
    int dev = 0, cus = 0;
    if (hipGetDevice(&dev) == hipSuccess &&
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess &&
        cus > 0)
        g_cus = (uint32_t)cus;
    int gy = 0;
    if (hipDeviceGetAttribute(&gy, hipDeviceAttributeMaxGridDimY, dev) == hipSuccess && gy > 0)
        g_max_grid_y = (uint64_t)gy;
    pir_status st;
    if ((st = set_ring_lds<Ring128x128S8>()) != PIR_OK) return st;
    if ((st = set_ring_lds<Ring128x128K128S4>()) != PIR_OK) return st;
    if ((st = set_ring_lds<Ring128x256S6>()) != PIR_OK) return st;
    if ((st = set_ring_lds<Ring8w128x256K128S3>()) != PIR_OK) return st;
    if ((st = set_ring_lds<Ring8w256x256S4>()) != PIR_OK) return st;
    if ((st = set_ring_lds<Ring8w256x256K128S2>()) != PIR_OK) return st;
    if ((st = set_ring_lds<Ring256x256K128S2>()) != PIR_OK) return st;
    if ((st = set_ring_lds<Ring128x128K128S2>()) != PIR_OK) return st;
    if ((st = set_ring_lds<Narrow256x32K128S4>()) != PIR_OK) return st;
    if ((st = set_ring_lds<Narrow256x64K128S4>()) != PIR_OK) return st;
    if ((st = set_ring_lds<Narrow128x32K128S6>()) != PIR_OK) return st;
    if ((st = set_ring_lds<Ring8w256x256K128D3>()) != PIR_OK) return st;
    if ((st = set_ring_lds<Ring8w128x256K128D4>()) != PIR_OK) return st;
    if ((st = set_ring_lds<Ring8w128x256K128D5>()) != PIR_OK) return st;
    if ((st = set_ring_lds<Ring8w256x256K128Q3>()) != PIR_OK) return st;
    if ((st = set_ring_lds<Narrow256x32K128D4>()) != PIR_OK) return st;
    if ((st = set_ring_lds<Narrow128x32K128D8>()) != PIR_OK) return st;
    if ((st = set_ring_lds<Ring256x256K128D3>()) != PIR_OK) return st;
    if ((st = set_ring_lds<Ring256x256K128Q3>()) != PIR_OK) return st;
    if ((st = set_client_lds<Ring128x128K128S2>()) != PIR_OK) return st;
    if ((st = set_client_lds<Ring8w128x256K128S3>()) != PIR_OK) return st;
    if ((st = set_client_lds<Ring8w256x256K128S2>()) != PIR_OK) return st;
    if ((st = set_reg_lds<Reg128x256>()) != PIR_OK) return st;
    if ((st = set_reg_lds<Reg128x128>()) != PIR_OK) return st;
    if ((st = set_reg_lds<Reg256x256>()) != PIR_OK) return st;
    if ((st = set_roles_lds<Roles256x256A5B4>()) != PIR_OK) return st;
    return set_roles_lds<Roles128x256A10B4>();
}

uint32_t mfma_variant_count() { return kNumVariants; }

const char* mfma_variant_name(uint32_t v) { return v < kNumVariants ? kVariants[v].name : nullptr; }

bool mfma_variant_valid(const pir_db_t* db, uint32_t B, uint32_t v, bool gathered) {
    if (gathered && v != 0 && v < kNumVariants && kVariants[v].kind == kFew) return false;
    return variant_valid(db, B, v);
}

size_t mfma_workspace_bytes(const pir_db_t* db, uint32_t B) {
    if (B == 0) return 0;
    return std::max(batch_layout(db, B, kVariants[kVarRing128]).total, few_workspace_bytes(db, B));
}

// Every choice and every check of a batched call, before anything is
// enqueued: variant, layout, split plan, grid limits and the workspace bytes
// the call touches.
pir_status mfma_plan_batch(const pir_db_t* db, uint32_t B, const uint32_t* rows, uint32_t m,
                           uint32_t modulus, bool planes, BatchPlan* plan) {
    const uint32_t C = (uint32_t)db->cols;
    const bool exact = modulus != 0;
    if (exact && rows) return PIR_ERR_UNSUPPORTED;   // no gathered field form
    if (exact && C > kMaxExactCols) return PIR_ERR_SHAPE;
    if (exact && planes) return PIR_ERR_UNSUPPORTED;

    uint32_t v = (rows ? db->variant_rows : db->variant)[batch_bucket(B)];
    const uint32_t M = rows ? m : (uint32_t)db->rows;
    if (v == 0 || !variant_valid(db, B, v))
        v = rows                               ? default_rows(db, B, m)
            : !planes && few_default(db, B)    ? kVarFew
                                               : default_gemm(db, B, M, exact, planes);
    if (rows && kVariants[v].kind == kFew) v = default_gemm(db, B, m, false, true);
    // Pre-ingested planes are in the wide layout: matrix-core variants that read it.
    if (planes && (kVariants[v].kind == kFew || kVariants[v].narrow))
        v = default_gemm(db, B, M, exact, true);
    // The field form runs on ring tiles, over rows of whole 16-byte pieces, and
    // on the dot4 stream, which takes any rows.
    if (exact && kVariants[v].kind != kFew && (kVariants[v].kind != kRing || !ring_ok(db)))
        v = (few_default(db, B) || (B <= kFewMax && !ring_ok(db)))
                ? kVarFew
                : default_gemm(db, B, M, true, false);
    if (exact && (kVariants[v].kind == kReg || kVariants[v].kind == kRoles ||
                  (kVariants[v].kind == kRing && !ring_ok(db))))
        return PIR_ERR_UNSUPPORTED;   // field form beyond kFewMax queries needs the ring kernels

    BatchPlan P{};
    P.variant = v;
    if (kVariants[v].kind == kFew) {
        P.few = true;
        P.need = few_workspace_bytes(db, B);
        *plan = P;
        return PIR_OK;
    }
    const VariantInfo& vi = kVariants[v];
    const BatchLayout L = batch_layout(db, B, vi);
    P.Bp = L.Bp;
    P.N = L.N;
    P.Cp = L.Cp;
    P.colsum_off = L.colsum_off;
    P.part_off = L.part_off;
    if ((uint64_t)L.Cp / kIngJ > g_max_grid_y) return PIR_ERR_SHAPE;   // ingest grid
    P.M = M;
    P.exact = exact;
    const SplitPlan sp = plan_splits(P.M, L.N, C, vi, exact, !ring_serves(db));
    P.splits = sp.splits;
    P.kts = sp.kts;
    const uint64_t blocks = (uint64_t)ceil_div(L.N, vi.bn) * ceil_div(P.M, vi.bm) * sp.splits;
    if (blocks > 0x7FFFFFFFull) return PIR_ERR_SHAPE;
    P.need = L.part_off;
    if (sp.splits > 1) {
        const uint64_t n = (uint64_t)P.M * B;
        if ((n + 255) / 256 > 0x7FFFFFFFull) return PIR_ERR_SHAPE;   // k_finish grid
        P.need += (size_t)sp.splits * P.M * B * (exact ? 8 : 4);
        if (P.need > L.total) return PIR_ERR_WORKSPACE;   // cannot happen: the layout bounds every plan
    }
    *plan = P;
    return PIR_OK;
}

// Fewer pieces, or one, where a fixed scratch cannot hold the partials of
// the plan: the allocation-free entry point serves every batch whose limb planes
// fit.  The field form's pieces also keep its sums exact and are left alone.
void mfma_plan_fit(const pir_db_t* db, uint32_t B, size_t scratch_bytes, BatchPlan* plan) {
    if (plan->few || plan->exact || plan->splits <= 1 || plan->need <= scratch_bytes) return;
    const uint32_t ktiles = ceil_div(db->cols, kVariants[plan->variant].bk);
    const size_t piece = (size_t)plan->M * B * 4;
    const size_t room = scratch_bytes > plan->part_off ? (scratch_bytes - plan->part_off) / piece : 0;
    plan->kts = ceil_div(ktiles, std::max<size_t>(room, 1));
    plan->splits = ceil_div(ktiles, plan->kts);
    plan->need = plan->part_off + (plan->splits > 1 ? plan->splits * piece : 0);
}

// Write the limb planes and (sums) the column sums, cleared first, of the
// queries into `base` (the layout of `P`).
static pir_status ingest(const pir_db_t* db, const BatchIO& io, uint32_t B, const BatchPlan& P,
                  bool narrow, bool sums, uint8_t* base, hipStream_t s) {
    const uint32_t C = (uint32_t)db->cols;
    int8_t* QL = reinterpret_cast<int8_t*>(base);
    u64* colsum = sums ? reinterpret_cast<u64*>(base + P.colsum_off) : nullptr;
    if (sums) {
        k_zero_words<<<(2 * P.Bp + 255) / 256, 256, 0, s>>>(reinterpret_cast<uint32_t*>(colsum),
                                                             2 * P.Bp);
        PIR_LAUNCH_CHECK();
    }
    dim3 ig((P.Bp + kIngB - 1) / kIngB, P.Cp / kIngJ);
    const bool qmajor = io.q_ldj == 1;
    const bool vec = (qmajor ? C : B) >= 4u;
#define PIR_INGEST(QM, V)                                                                  \
    k_ingest<QM, V><<<ig, 256, 0, s>>>(io.Q, io.q_ldj, io.q_ldb, C, B, P.Bp, P.Cp, QL, colsum, \
                                       narrow)
    if (qmajor) {
        if (vec) PIR_INGEST(true, true); else PIR_INGEST(true, false);
    } else {
        if (vec) PIR_INGEST(false, true); else PIR_INGEST(false, false);
    }
#undef PIR_INGEST
    PIR_LAUNCH_CHECK();
    return PIR_OK;
}

// Whether the product sums the limb planes itself (SUMS).  Narrow tiles have
// the issue slots to spare (8 queries on 8192 x 8192 22.8 -> 20.6 us); 128 x
// 128 tiles do for one column tile and while the launch and the atomics weigh
// more than the dot instructions (32 queries: 4096 x 4096 20.9 -> 19.1 us,
// 16384 x 16384 74.7 -> 73.7, 65536 x 32768 408 -> 462; 64 queries, two
// column tiles: 8192 x 8192 34.8 -> 39.4, 16384 x 8192 49.9 -> 61.7).
static bool tile_sums(const pir_db_t* db, const VariantInfo& vi, const BatchPlan& P,
                      const uint32_t* rows, bool client) {
    if (vi.kind != kRing || vi.bn > 128u || rows) return false;
    return vi.bn < 128u || client ||
           (P.N <= 128u && db->rows * db->cols <= (1ull << 28));
}

// Answers contiguous along rows, in whole aligned groups of four: 16-byte
// stores along rows instead of one word per lane and row (128 queries' worth
// of lines per store instruction).
static bool mfma_by_rows(const BatchIO& io, const BatchPlan& P, const uint32_t* rows, bool exact) {
    return !exact && !rows && P.M % 4 == 0 && io.o_ldr == 1 && io.o_ldb % 4 == 0 &&
           (uintptr_t)io.out % 16 == 0;
}

// Enqueue a planned batched call; `ws` holds at least plan.need bytes.  With
// `planes` (the wide-layout limb planes and column sums of these queries,
// written by mfma_ingest_planes) the ingest is skipped.
pir_status mfma_run_batch(const pir_db_t* db, const BatchIO& io, uint32_t B,
                          const uint32_t* rows, uint32_t modulus, const BatchPlan& P, void* ws,
                          const void* planes, const ClientEpi* client, hipStream_t s) {
    if (P.few) return few_answer_batch(db, io, B, modulus, ws, P.need, s);
    const uint32_t C = (uint32_t)db->cols;
    const bool exact = modulus != 0;
    const VariantInfo& vi = kVariants[P.variant];
    uint8_t* base = static_cast<uint8_t*>(ws);
    const uint8_t* qbase = planes ? static_cast<const uint8_t*>(planes) : base;
    const int8_t* QL = reinterpret_cast<const int8_t*>(qbase);
    const bool sums = !tile_sums(db, vi, P, rows, client != nullptr);
    const u64* colsum = sums ? reinterpret_cast<const u64*>(qbase + P.colsum_off) : nullptr;
    if (!planes) {
        const pir_status st = ingest(db, io, B, P, vi.narrow, sums, base, s);
        if (st != PIR_OK) return st;
    }
    if (P.M == 0) return PIR_OK;

    Gemm g;
    g.db = db;
    g.QL = QL;
    g.Cp = P.Cp;
    g.N = P.N;
    g.exact = exact;
    g.splits = P.splits;
    g.kts = P.kts;
    g.e = Epi{P.M,       B,        (uint32_t)db->rows,   C,       rows,  colsum, db->rowterm,
              db->row_scale, io.out, io.o_ldr, io.o_ldb, base + P.part_off, modulus,
              mfma_by_rows(io, P, rows, exact), client ? *client : ClientEpi{}};
    const uint64_t n = (uint64_t)P.M * B;
    if (client) {
        const int mode = client->bytes ? kClientDecode : kClientQuery;
        const pir_status st = vi.client(g, P.splits > 1 ? kPart32Rows : mode, s);
        if (st != PIR_OK || P.splits <= 1) return st;
        if (mode == kClientDecode)
            k_finish_rows<kClientDecode><<<(uint32_t)((n / 4 + 255) / 256), 256, 0, s>>>(g.e, P.splits);
        else
            k_finish_rows<kClientQuery><<<(uint32_t)((n / 4 + 255) / 256), 256, 0, s>>>(g.e, P.splits);
        PIR_LAUNCH_CHECK();
        return PIR_OK;
    }
    const pir_status st = vi.launch(g, s);
    if (st != PIR_OK || P.splits <= 1) return st;
    if (n == 0) return PIR_OK;
    const bool vec4 = !exact && B % 4 == 0 && io.o_ldb == 1 && io.o_ldr % 4 == 0 &&
                      (uintptr_t)io.out % 16 == 0;
    if (exact)
        k_finish<true><<<(uint32_t)((n + 255) / 256), 256, 0, s>>>(g.e, P.splits);
    else if (g.e.by_rows)
        k_finish_rows<kFinal32Rows><<<(uint32_t)((n / 4 + 255) / 256), 256, 0, s>>>(g.e, P.splits);
    else if (vec4)
        k_finish4<<<(uint32_t)((n / 4 + 255) / 256), 256, 0, s>>>(g.e, P.splits);
    else
        k_finish<false><<<(uint32_t)((n + 255) / 256), 256, 0, s>>>(g.e, P.splits);
    PIR_LAUNCH_CHECK();
    return PIR_OK;
}

// Whether a planned product can end in the client's epilogue.
bool mfma_client_fused(const BatchPlan& P, const BatchIO& io, const ClientEpi& client) {
    return kVariants[P.variant].client && mfma_by_rows(io, P, nullptr, false) &&
           (uintptr_t)client.add % 16 == 0 && (uintptr_t)client.bytes % 4 == 0;
}

pir_status mfma_answer_batch(const pir_db_t* db, const BatchIO& io, uint32_t B,
                             const uint32_t* rows, uint32_t m, uint32_t modulus, void* ws,
                             size_t ws_bytes, const void* planes, size_t planes_bytes,
                             hipStream_t s) {
    BatchPlan plan;
    const pir_status st = mfma_plan_batch(db, B, rows, m, modulus, planes != nullptr, &plan);
    if (st != PIR_OK) return st;
    // The reported size is the contract for every kernel path.
    if (!ws || ws_bytes < mfma_workspace_bytes(db, B) || ((uintptr_t)ws % kWsAlign))
        return PIR_ERR_WORKSPACE;
    if (planes && (planes_bytes < mfma_planes_bytes(db, B) || ((uintptr_t)planes % kWsAlign)))
        return PIR_ERR_WORKSPACE;
    return mfma_run_batch(db, io, B, rows, modulus, plan, ws, planes, nullptr, s);
}

size_t mfma_planes_bytes(const pir_db_t* db, uint32_t n) {
    if (n == 0) return 0;
    return batch_layout(db, n, kVariants[kVarRing128]).part_off;
}

pir_status mfma_ingest_planes(const pir_db_t* db, const uint32_t* A, uint32_t n, void* planes,
                              size_t planes_bytes, hipStream_t s) {
    BatchLayout L = batch_layout(db, n, kVariants[kVarRing128]);
    if (!planes || planes_bytes < L.part_off || ((uintptr_t)planes % kWsAlign))
        return PIR_ERR_WORKSPACE;
    if ((uint64_t)L.Cp / kIngJ > g_max_grid_y) return PIR_ERR_SHAPE;
    BatchPlan P{};
    P.Bp = L.Bp;
    P.N = L.N;
    P.Cp = L.Cp;
    P.colsum_off = L.colsum_off;
    const BatchIO io{A, n, 1, nullptr, n, 1};
    return ingest(db, io, n, P, false, true, static_cast<uint8_t*>(planes), s);
}
