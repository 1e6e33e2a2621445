// Chor XOR PIR response (the ENS instantiation, Section 5.1; server step of
// Algorithm 3): for each query bit vector q_b over the r database rows,
//
//     out[b] = XOR over rows i with bit i of q_b set of DB[i]
//
// DB rows are b-bit blocks stored as W 32-bit words (row pitch in words);
// query b is packed 32 rows per word, little-endian (bit j of word k selects
// row 32k + j); bits past the last row are ignored.
//
// * One query (k_chor_stream) reads only the rows it selects, about half of
//   the database, and is bound by HBM: the selector words of a whole slab are
//   fetched up front, set bits are taken with a wave-uniform bit scan, and up
//   to 32 rows per wave are in flight (non-temporal loads).
// * Two or more queries (k_chor_parity) run on the matrix cores.  XOR is
//   addition modulo 2, so every output bit is the parity of an integer count,
//
//       out[b] bit c of word n = (sum_r sel[b][r] * bit_c(DB[r][n])) mod 2,
//
//   a matrix product of 0/1 entries: M = queries, N = bits, K = rows.  The
//   entries are exact in the 4-bit float format, whose matrix instruction
//   has twice the int8 rate, and the counts (at most 2^18 per workgroup,
//   scaled by 1/2, 1 or 2) are exact in its fp32 accumulators.
// * Slabs of rows combine into the output with atomicXor (the result does
//   not depend on the order); the output is cleared first by a fill kernel,
//   except where one slab covers all rows.
#include <string.h>

#include <type_traits>

#include "qpir_internal.h"

namespace {

constexpr int kThreads = 256;
constexpr uint32_t kChunkWords = 4 * kThreads;

typedef int i32x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

// Output before accumulation: zero, or a copy of `init` (the OOP response
// starts from its precomputed value A).
__global__ void k_chor_init(uint32_t* __restrict__ p, const uint32_t* __restrict__ init,
                            uint64_t n) {
    const uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = init ? init[i] : 0u;
}

template <bool VEC>
__device__ inline u32x4 load_words_nt(const uint32_t* row, uint32_t w, uint32_t W) {
    if (VEC)   // W % 4 == 0, aligned
        return __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(row + w));
    return u32x4{w < W ? row[w] : 0u, w + 1 < W ? row[w + 1] : 0u,
                 w + 2 < W ? row[w + 2] : 0u, w + 3 < W ? row[w + 3] : 0u};
}

__device__ inline uint32_t xcd_remap(uint32_t bid, uint32_t nblk) {
    const uint32_t per = nblk / 8u;
    return bid < per * 8u ? (bid % 8u) * per + bid / 8u : bid;
}

// One query.  Workgroup = one slab of rows [r0, r1), all columns in chunks
// of 1024 words (lane t: words 4t..4t+3).  One load per lane fetches the
// selector words of 64 consecutive 32-row blocks, taken in pairs: the 64-bit
// mask names the rows to read, up to kDepth of them in flight per wave.
constexpr int kDepth = 32;

template <bool VEC>
__global__ __launch_bounds__(kThreads) void k_chor_stream(const uint32_t* __restrict__ DB,
                                                          uint64_t pitch, uint32_t rows,
                                                          uint32_t W,
                                                          const uint32_t* __restrict__ Q,
                                                          uint32_t slab_rows,
                                                          uint32_t* __restrict__ out) {
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint32_t slab = xcd_remap(blockIdx.x, gridDim.x);
    const uint32_t r0 = slab * slab_rows;
    const uint32_t r1 = min(rows, r0 + slab_rows);

    for (uint32_t c0 = 0; c0 < W; c0 += kChunkWords) {
        if (c0 + 256u * (uint32_t)wave >= W) continue;   // no lane of this wave has words here
        const uint32_t w = c0 + 4u * threadIdx.x;
        const bool active = w < W;
        u32x4 acc = u32x4{0, 0, 0, 0};
        for (uint32_t base = r0; base < r1; base += 32u * 64u) {
            uint32_t qv = 0;
            const uint32_t rb = base + 32u * (uint32_t)lane;
            if (rb < r1) {
                qv = Q[rb / 32u];
                const uint32_t nrow = min(32u, r1 - rb);
                if (nrow < 32u) qv &= (1u << nrow) - 1u;
            }
            for (int jb = 0; jb < 64; jb += 2) {
                const uint32_t rblk = base + 32u * (uint32_t)jb;
                if (rblk >= r1) break;                    // uniform
                const uint32_t lo = __builtin_amdgcn_readlane(qv, jb);
                const uint32_t hi = __builtin_amdgcn_readlane(qv, jb + 1);
                uint64_t any = (uint64_t)lo | ((uint64_t)hi << 32);
                while (any) {
                    u32x4 d[kDepth];
#pragma unroll
                    for (int k = 0; k < kDepth; ++k) {
                        d[k] = u32x4{0, 0, 0, 0};
                        if (any) {                        // uniform
                            const uint32_t idx = (uint32_t)__builtin_ctzll(any);
                            any &= any - 1u;
                            if (active)
                                d[k] = load_words_nt<VEC>(DB + (uint64_t)(rblk + idx) * pitch, w,
                                                          W);
                        }
                    }
#pragma unroll
                    for (int k = 0; k < kDepth; ++k) acc ^= d[k];
                }
            }
        }
        if (active) {
            uint32_t* o = out + w;
            if (acc.x) atomicXor(o, acc.x);
            if (w + 1 < W && acc.y) atomicXor(o + 1, acc.y);
            if (w + 2 < W && acc.z) atomicXor(o + 2, acc.z);
            if (w + 3 < W && acc.w) atomicXor(o + 3, acc.w);
        }
    }
}

// ---------------------------------------------------------------- matrix cores
// A workgroup (four waves, or NH = 2 groups of four side by side in columns)
// covers a slab of rows, 32 words per group of four waves and 32 TM queries.
// It walks the rows in chunks of 128 = two k-steps of 64 rows.  Lane half h
// of a k-step s covers the 32 rows of block 2h + s of the chunk.
//
// Operands (32x32x64 instruction, lane l: row or column l % 32, entries of
// half l / 32; the order of a half's 32 entries is free as long as both
// operands share it: register j, nibble i holds row 4i + j of the block).
// * Queries: a lane's 32 entries are one selector word v; register j is
//   (v >> j) & 0x11111111, moved to bit 1 (value 1.0): seven instructions.
// * Database: each thread loads 16 words of one column (rows 4i + j of a
//   block, j two consecutive values), transposes them by nibbles in
//   registers (two passes of and/or, then byte permutes) and stores them to
//   LDS, so that nibble position p of 32 rows becomes one 16-byte read; a
//   wave reads positions p and p + 4 (p = wave) and masks bit c of every
//   nibble: the mask's place is the entry's value (0.5, 1.0, 2.0; bit 3 is
//   shifted to 2.0), one instruction per register for three of four bits.
//   The scale is constant per accumulator tile and undone at the end.
//
// A wave's 8 TM accumulator tiles (2 nibbles x 4 bits x TM) use 128 TM
// registers: one wave per SIMD for TM = 2, two for TM = 1 (NH = 2 puts both
// in one workgroup, whose rows are then read in 256-byte pieces).
//
// Software pipeline, per chunk ch: 16 slices of TM matrix instructions, with
// the vector work of other chunks between them: the next slice's masks, the
// transpose and LDS store of chunk ch + 2, the loads of chunk ch + 4.  Three
// LDS buffers, one barrier per chunk.
//
// Bound: up to 32 queries by HBM; above, by the matrix cores with the vector
// instructions beside them (about six per matrix instruction; a loop of bare
// 0/1 matrix instructions reaches 7.6 POP/s in the power budget, 7.3 with
// four vector instructions beside each).  Against lookups in 16-entry XOR
// tables in LDS, which this replaces, whole calls on 2^18 blocks of 3 KB: 8
// queries 230 -> 137 us (5.9 TB/s), 32 252 -> 143 us, 64 350 -> 205 us, 128
// 617 -> 372 us, 1024 2.88 -> 2.55 ms (5.2 POP/s); on 2^13 blocks: 16 queries
// 52 -> 15 us, 128 148 -> 23 us, 1024 249 -> 105 us.
constexpr int kParBufs = 3;
constexpr uint32_t kParChunk = 128;              // rows per chunk
constexpr uint32_t kParMaxSlab = 1u << 18;       // rows counted in one accumulator
constexpr uint32_t kParWords = 32;               // words per group of four waves

__device__ inline f32x16 mfma_f4(const u32x4 a, const u32x4 b, const f32x16 c) {
    const i32x8 aa = {(int)a.x, (int)a.y, (int)a.z, (int)a.w, 0, 0, 0, 0};
    const i32x8 bb = {(int)b.x, (int)b.y, (int)b.z, (int)b.w, 0, 0, 0, 0};
    return __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(aa, bb, c, 4, 4, 0, 0, 0, 0);
}

__device__ inline u32x4 expand_selectors(uint32_t v) {
    constexpr uint32_t m = 0x22222222u;          // 1.0 in every nibble
    return u32x4{(v << 1) & m, v & m, (v >> 1) & m, (v >> 2) & m};
}

__device__ inline u32x4 bit_plane(const u32x4 t, int c) {
    return c < 3 ? (t & (0x11111111u << c)) : ((t >> 1) & 0x44444444u);
}

// Barrier that waits for LDS operations only: row loads stay in flight.
__device__ inline void lds_barrier() {
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt((0x3F & 0xF) | ((0x3F >> 4) << 14) | (0x7 << 4) | (0x0 << 8));
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

// 8 x 8 nibble transpose in two parts: rows 2k and 2k + 1 exchange nibbles
// (part 1, for k = 0..3), then the even (o = 0) or odd (o = 1) nibbles' bytes
// move: afterwards x[p] nibble i is nibble p of the original x[i].
__device__ inline void transpose_nibbles(uint32_t (&x)[8], int k) {
    const uint32_t a = x[2 * k], b = x[2 * k + 1];
    x[2 * k] = (a & 0x0F0F0F0Fu) | ((b << 4) & 0xF0F0F0F0u);
    x[2 * k + 1] = ((a >> 4) & 0x0F0F0F0Fu) | (b & 0xF0F0F0F0u);
}

__device__ inline void transpose_bytes(uint32_t (&x)[8], int o) {
    const uint32_t v0 = x[o], v1 = x[o + 2], v2 = x[o + 4], v3 = x[o + 6];
    const uint32_t p = __builtin_amdgcn_perm(v1, v0, 0x05010400u);
    const uint32_t q = __builtin_amdgcn_perm(v1, v0, 0x07030602u);
    const uint32_t r = __builtin_amdgcn_perm(v3, v2, 0x05010400u);
    const uint32_t s = __builtin_amdgcn_perm(v3, v2, 0x07030602u);
    x[o] = __builtin_amdgcn_perm(r, p, 0x05040100u);
    x[o + 2] = __builtin_amdgcn_perm(r, p, 0x07060302u);
    x[o + 4] = __builtin_amdgcn_perm(s, q, 0x05040100u);
    x[o + 6] = __builtin_amdgcn_perm(s, q, 0x07060302u);
}

// NT: non-temporal row loads.  `first`: this launch writes the output (init
// or zero, xor the product) instead of adding to it with atomics.
template <int TM, int NH, bool NT>
__global__ __launch_bounds__(256 * NH, TM == 1 ? 2 : 1) void k_chor_parity(
    const uint32_t* __restrict__ DB, uint64_t pitch, uint32_t rows, uint32_t W,
    const uint32_t* __restrict__ Q, uint32_t qwords, uint32_t B, uint32_t slab_rows,
    uint32_t n_qg, uint32_t n_cs, bool first, const uint32_t* init, uint32_t* out) {
    constexpr int NW = kParWords;
    constexpr int kWgWords = NW * NH;
    __shared__ u32x4 s_t[NH][kParBufs][4][8][NW];     // [block][nibble position][word]
    __shared__ uint32_t s_out[32 * TM][kWgWords];
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave_wg = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wave = wave_wg & 3, half = wave_wg >> 2;
    // The query groups of a column slice are consecutive and slabs outermost:
    // groups that read the same rows run on one XCD and share its L2.
    const uint32_t bid = xcd_remap(blockIdx.x, gridDim.x);
    const uint32_t qg = bid % n_qg;
    const uint32_t cs = (bid / n_qg) % n_cs;
    const uint32_t slab = bid / (n_qg * n_cs);
    const uint32_t r0 = slab * slab_rows;
    const uint32_t r1 = min(rows, r0 + slab_rows);
    const uint32_t nch = (r1 - r0 + kParChunk - 1) / kParChunk;

    // Row loads: the wave's block of the chunk, lane: word lane % 32, rows
    // 4i + j0 and 4i + j0 + 1.  Fast: the chunk lies inside the rows; else
    // the chunk index and the rows are clamped (the selector bits of rows
    // past the end are cleared, and a clamped chunk is not counted).
    typedef std::integral_constant<bool, true> Fast;
    typedef std::integral_constant<bool, false> Slow;
    const int jn = lane & (NW - 1), j0 = 2 * (lane >> 5);
    const uint32_t* dcol = DB + min((cs * NH + half) * NW + jn, W - 1);
    auto load_d = [&](auto fast, uint32_t ch, uint32_t (&x)[2][8], int k0, int n) {
        if constexpr (decltype(fast)::value) {
            const uint32_t* p = dcol + (uint64_t)(r0 + kParChunk * ch + 32u * wave) * pitch +
                                (uint64_t)j0 * pitch;
#pragma unroll
            for (int k = k0; k < k0 + n; ++k) {
                const uint32_t* a = p + (uint64_t)(4 * (k % 8) + k / 8) * pitch;
                x[k / 8][k % 8] = NT ? __builtin_nontemporal_load(a) : *a;
            }
        } else {
            const uint32_t rb = r0 + kParChunk * min(ch, nch - 1) + 32u * wave + j0;
#pragma unroll
            for (int k = k0; k < k0 + n; ++k)
                x[k / 8][k % 8] =
                    dcol[(uint64_t)min(rb + 4 * (k % 8) + k / 8, rows - 1) * pitch];
        }
    };
    // Selector words of the lane's query and half, both k-steps.  Queries
    // past B repeat the last one; their outputs are not stored.
    const int h = lane >> 5;
    const uint32_t* qrow[TM];
#pragma unroll
    for (int a = 0; a < TM; ++a)
        qrow[a] = Q + (uint64_t)min((qg * TM + a) * 32u + (lane & 31), B - 1) * qwords;
    auto load_q = [&](auto fast, uint32_t ch, uint32_t (&v)[TM][2]) {
        if constexpr (decltype(fast)::value) {
            const uint32_t w = (r0 + kParChunk * ch) / 32u + 2u * h;
#pragma unroll
            for (int a = 0; a < TM; ++a) {
                v[a][0] = qrow[a][w];
                v[a][1] = qrow[a][w + 1];
            }
        } else {
            const uint32_t w = (r0 + kParChunk * min(ch, nch - 1)) / 32u + 2u * h;
#pragma unroll
            for (int s = 0; s < 2; ++s) {
                const uint32_t row = 32u * (w + s);       // rows of the word
                const uint32_t n = row < rows ? min(32u, rows - row) : 0u;
                const uint32_t mask = n == 32u ? 0xFFFFFFFFu : (1u << n) - 1u;
#pragma unroll
                for (int a = 0; a < TM; ++a) v[a][s] = qrow[a][min(w + s, qwords - 1)] & mask;
            }
        }
    };
    auto put = [&](uint32_t ch, const uint32_t (&x)[2][8], int o) {   // nibbles o, o + 2, ..
        uint32_t* dst = reinterpret_cast<uint32_t*>(&s_t[half][ch % kParBufs][wave][0][jn]) + j0;
#pragma unroll
        for (int p = o; p < 8; p += 2)
            *reinterpret_cast<uint64_t*>(dst + p * NW * 4) =
                (uint64_t)x[0][p] | ((uint64_t)x[1][p] << 32);
    };
    auto get = [&](uint32_t ch, u32x4 (&t)[2][2]) {
#pragma unroll
        for (int s = 0; s < 2; ++s)
#pragma unroll
            for (int g = 0; g < 2; ++g)
                t[s][g] = s_t[half][ch % kParBufs][2 * h + s][wave + 4 * g][jn];
    };

    f32x16 acc[TM][2][4];
#pragma unroll
    for (int a = 0; a < TM; ++a)
#pragma unroll
        for (int g = 0; g < 2; ++g)
#pragma unroll
            for (int c = 0; c < 4; ++c)
#pragma unroll
                for (int v = 0; v < 16; ++v) acc[a][g][c][v] = 0.f;

    uint32_t x[2][2][8];        // rows of chunks ch + 2, ch + 3
    uint32_t qv[2][TM][2];      // selector words of chunks ch, ch + 1
    u32x4 t[2][2][2];           // database operands of chunks ch, ch + 1
    u32x4 fa[2][TM], fb[2];     // expanded operands: k-step, slice
    {
        uint32_t x0[2][8], x1[2][8];
        load_d(Slow{}, 0, x0, 0, 16);
        load_d(Slow{}, 1, x1, 0, 16);
        load_q(Slow{}, 0, qv[0]);
        load_q(Slow{}, 1, qv[1]);
        load_d(Slow{}, 2, x[0], 0, 16);
        load_d(Slow{}, 3, x[1], 0, 16);
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            uint32_t (&y)[2][8] = u ? x1 : x0;
#pragma unroll
            for (int g = 0; g < 2; ++g) {
#pragma unroll
                for (int k = 0; k < 4; ++k) transpose_nibbles(y[g], k);
                transpose_bytes(y[g], 0);
                transpose_bytes(y[g], 1);
            }
            put(u, y, 0);
            put(u, y, 1);
        }
        lds_barrier();
        get(0, t[0]);
#pragma unroll
        for (int a = 0; a < TM; ++a) fa[0][a] = expand_selectors(qv[0][a][0]);
        fb[0] = bit_plane(t[0][0][0], 0);
    }
    // Chunk ch: buffer (ch + 2) % 3, which it fills, was last read by get()
    // in chunk ch - 2, before two barriers.
    auto body = [&](auto fast, uint32_t ch, int cur) {
        get(ch + 1, t[cur ^ 1]);
        uint32_t q1[TM];
#pragma unroll
        for (int a = 0; a < TM; ++a) q1[a] = qv[cur][a][1];
#pragma unroll
        for (int sl = 0; sl < 16; ++sl) {
            const int s = sl / 8, l = sl % 8, g = l / 4, c = l % 4;
            // Two waves per SIMD fill each other's gaps best when every
            // slice keeps its place; one wave is left to the scheduler
            // (32 queries 151 -> 142 us with the barriers, 128 queries 362
            // -> 372 us).
            if constexpr (TM == 1) __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int a = 0; a < TM; ++a) acc[a][g][c] = mfma_f4(fa[s][a], fb[sl & 1], acc[a][g][c]);
            fb[(sl + 1) & 1] = sl + 1 < 16 ? bit_plane(t[cur][(sl + 1) / 8][(sl + 1) / 4 % 2], (sl + 1) % 4)
                                           : bit_plane(t[cur ^ 1][0][0], 0);
            if (l < TM) fa[s ^ 1][l] = expand_selectors(s == 0 ? q1[l] : qv[cur ^ 1][l][0]);
            if (s == 0) {
                transpose_nibbles(x[cur][l % 2], l / 2);
            } else if (l < 4) {
                transpose_bytes(x[cur][l % 2], l / 2);
                if (l % 2 == 1) put(ch + 2, x[cur], l / 2);
            } else {
                if (l == 4) load_q(fast, ch + 2, qv[cur]);
                load_d(fast, ch + 4, x[cur], 4 * (l - 4), 4);
            }
            if constexpr (TM == 1) __builtin_amdgcn_sched_barrier(0);
        }
        lds_barrier();
    };
    const uint32_t nfull = (r1 - r0) / kParChunk;
    uint32_t ch = 0;
    for (; ch + 5 < nfull; ch += 2) {
        body(Fast{}, ch, 0);
        body(Fast{}, ch + 1, 1);
    }
    for (; ch < nch; ch += 2) {
        body(Slow{}, ch, 0);
        if (ch + 1 < nch) body(Slow{}, ch + 1, 1);
    }

    // Parities: tile c of nibble position wave + 4g holds bit c; register v
    // of lane half h holds query 8 (v/4) + 4 h + v % 4.  The waves' nibbles
    // meet in LDS.
    for (int i = tid; i < 32 * TM * kWgWords; i += 256 * NH) (&s_out[0][0])[i] = 0;
    __syncthreads();
#pragma unroll
    for (int a = 0; a < TM; ++a)
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            uint32_t y = 0;
#pragma unroll
            for (int g = 0; g < 2; ++g)
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    const float unscale = c == 0 ? 2.f : (c == 1 ? 1.f : 0.5f);
                    y |= ((uint32_t)(acc[a][g][c][v] * unscale) & 1u) << (16 * g + c);
                }
            atomicOr(&s_out[32 * a + 8 * (v / 4) + 4 * h + v % 4][half * NW + jn], y << (4 * wave));
        }
    __syncthreads();
    for (int i = tid; i < 32 * TM * kWgWords; i += 256 * NH) {
        const uint32_t b = qg * TM * 32u + i / kWgWords, w = cs * kWgWords + i % kWgWords;
        if (b >= B || w >= W) continue;
        const uint32_t y = (&s_out[0][0])[i];
        const uint64_t at = (uint64_t)b * W + w;
        if (first) out[at] = init ? init[at] ^ y : y;
        else if (y) atomicXor(out + at, y);
    }
}

// Row slabs of a launch.  One workgroup runs per CU, so a launch takes
// ceil(workgroups / 256) rounds, each of a slab's chunks plus the pipeline
// fill and the epilogue, worth about six chunks; take the count with the
// least total (128 queries on 2^18 blocks of 3 KB, 48 workgroups per slab:
// 5 or 16 slabs 375 us, 8 slabs 388 us, 21 slabs 410 us).
struct Slabs {
    uint32_t count, rows;
};

Slabs parity_slabs(uint32_t rows, uint64_t per_slab) {
    const uint32_t chunks = (rows + kParChunk - 1) / kParChunk;
    const uint32_t lo = (rows + kParMaxSlab - 1) / kParMaxSlab;
    const uint32_t hi = std::max(lo, std::min(chunks, 64u));
    uint32_t best = lo;
    double best_t = 1e300;
    for (uint32_t n = lo; n <= hi; ++n) {
        const double t = (double)((per_slab * n + 255) / 256) * ((chunks + n - 1) / n + 6);
        if (t < best_t) {
            best_t = t;
            best = n;
        }
    }
    const uint32_t slab = (chunks + best - 1) / best * kParChunk;
    return {(rows + slab - 1) / slab, slab};
}

template <int TM, int NH>
pir_status launch_parity(const uint32_t* d_DB, uint32_t rows, uint32_t words, uint64_t pitch,
                         const uint32_t* d_Q, uint32_t B, const uint32_t* d_init, uint32_t* d_out,
                         hipStream_t s) {
    const uint32_t n_qg = (B + 32 * TM - 1) / (32 * TM);
    const uint32_t n_cs = (words + kParWords * NH - 1) / (kParWords * NH);
    const uint64_t per_slab = (uint64_t)n_qg * n_cs;
    const Slabs sl = parity_slabs(rows, per_slab);
    const uint64_t blocks = per_slab * sl.count;
    if (blocks > 0x7FFFFFFFull) return PIR_ERR_SHAPE;
    const bool first = sl.count == 1;
    if (!first) {
        const pir_status st = chor_init(d_out, d_init, (uint64_t)B * words, s);
        if (st != PIR_OK) return st;
    }
    // A database read by one query group and larger than the 256 MiB
    // last-level cache is streamed past it; a smaller one may be there from
    // the previous call (32 queries: 2^18 blocks of 3 KB 152 us with plain
    // loads, 142 us non-temporal; 2^16 blocks 40 and 46 us).
    const bool nt = n_qg == 1 && (uint64_t)rows * words * 4u > (256ull << 20);
#define PIR_PARITY(X)                                                                         k_chor_parity<TM, NH, X><<<(uint32_t)blocks, 256 * NH, 0, s>>>(                               d_DB, pitch, rows, words, d_Q, (rows + 31) / 32, B, sl.rows, n_qg, n_cs, first, d_init,         d_out)
    if (nt) PIR_PARITY(true); else PIR_PARITY(false);
#undef PIR_PARITY
    PIR_LAUNCH_CHECK();
    return PIR_OK;
}

pir_status launch_stream(const uint32_t* d_DB, uint32_t rows, uint32_t words, uint64_t pitch,
                         const uint32_t* d_Q, uint32_t* d_out, hipStream_t s) {
    // Enough rows in flight to stream HBM (32 per wave), few enough slabs to
    // keep the output atomics (slabs x words, all onto the same words) down:
    // at most one workgroup per CU, and at least 256 rows per slab.
    // (Measured on 2^18 and 2^16 rows of 3 KB: fewer workgroups starve the
    // stream on the large database, more slabs spend the small one's time in
    // atomics.)
    uint64_t slab = (rows + 255) / 256;
    slab = (slab + 31) / 32 * 32;
    if (slab < 256) slab = 256;
    const uint64_t blocks = (rows + slab - 1) / slab;
    if (blocks > 0x7FFFFFFFull) return PIR_ERR_SHAPE;
    const bool vec = ((uintptr_t)d_DB % 16 == 0) && (words % 4 == 0) && (pitch % 4 == 0);
    if (vec)
        k_chor_stream<true><<<(uint32_t)blocks, kThreads, 0, s>>>(d_DB, pitch, rows, words, d_Q,
                                                                  (uint32_t)slab, d_out);
    else
        k_chor_stream<false><<<(uint32_t)blocks, kThreads, 0, s>>>(d_DB, pitch, rows, words, d_Q,
                                                                   (uint32_t)slab, d_out);
    PIR_LAUNCH_CHECK();
    return PIR_OK;
}

}  // namespace

bool current_is_gfx950() {
    int dev = -1;
    hipDeviceProp_t prop;
    if (hipGetDevice(&dev) != hipSuccess || hipGetDeviceProperties(&prop, dev) != hipSuccess)
        return false;
    return strncmp(prop.gcnArchName, "gfx950", 6) == 0;
}

pir_status chor_init(uint32_t* d_out, const uint32_t* d_init, uint64_t n, hipStream_t s) {
    if (n == 0) return PIR_OK;
    if ((n + 255) / 256 > 0x7FFFFFFFull) return PIR_ERR_SHAPE;
    k_chor_init<<<(uint32_t)((n + 255) / 256), 256, 0, s>>>(d_out, d_init, n);
    PIR_LAUNCH_CHECK();
    return PIR_OK;
}

pir_status chor_xor(const uint32_t* d_DB, uint32_t rows, uint32_t words, uint64_t pitch,
                    const uint32_t* d_Q, uint32_t B, const uint32_t* d_init, uint32_t* d_out,
                    hipStream_t s) {
    if (B == 1) {
        const pir_status st = chor_init(d_out, d_init, words, s);
        if (st != PIR_OK) return st;
        return launch_stream(d_DB, rows, words, pitch, d_Q, d_out, s);
    }
    // Up to 32 queries one 32-query tile with two workgroup halves; above,
    // 64 queries per workgroup, which halves the masks and the transposes
    // per matrix instruction (64 queries on 2^18 blocks: 205 us against 284
    // us as two 32-query groups).
    if (B <= 32) return launch_parity<1, 2>(d_DB, rows, words, pitch, d_Q, B, d_init, d_out, s);
    return launch_parity<2, 1>(d_DB, rows, words, pitch, d_Q, B, d_init, d_out, s);
}

extern "C" {

pir_status pir_chor_answer(const uint32_t* d_DB, uint32_t rows, uint32_t words,
                           uint64_t row_pitch_words, const uint32_t* d_Q, uint32_t B,
                           uint32_t* d_out, pir_stream_t stream) {
    if (B == 0) return PIR_OK;
    if (!d_DB || !d_Q || !d_out) return PIR_ERR_INVALID_ARG;
    if (rows == 0 || words == 0 || row_pitch_words < words || rows > kMaxDim ||
        words > kMaxDim || B > kMaxBatch)
        return PIR_ERR_SHAPE;
    if (!current_is_gfx950()) return PIR_ERR_UNSUPPORTED;
    return chor_xor(d_DB, rows, words, row_pitch_words, d_Q, B, nullptr, d_out,
                    static_cast<hipStream_t>(stream));
}

}  // extern "C"
