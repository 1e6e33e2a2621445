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
//   to 32 rows per wave are in flight (non-temporal loads).  So do two queries
//   on large databases (stream_two).
// * Other batches (k_chor_parity) run on the matrix cores.  XOR is
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
typedef u32x4 u32x4_word __attribute__((aligned(4)));
typedef __attribute__((address_space(3))) void lds_void_t;
typedef __attribute__((address_space(3))) uint32_t lds_word_t;
typedef __attribute__((address_space(3))) u32x4 lds_quad_t;
typedef __attribute__((address_space(1))) void glb_void_t;
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

// One or two queries (G).  Workgroup = one slab of rows [r0, r1), all columns
// in chunks of 1024 words (lane t: words 4t..4t+3).  One load per lane fetches
// the selector words of 64 / G consecutive 32-row blocks (lane l: query l G /
// 64), taken in pairs: the queries' 64-bit masks together name the rows to
// read, up to kDepth of them in flight per wave.
constexpr int kDepth = 32;

template <int G, bool VEC>
__global__ __launch_bounds__(kThreads) void k_chor_stream(const uint32_t* __restrict__ DB,
                                                          uint64_t pitch, uint32_t rows,
                                                          uint32_t W,
                                                          const uint32_t* __restrict__ Q,
                                                          uint32_t qwords, uint32_t slab_rows,
                                                          uint32_t* __restrict__ out) {
    constexpr int kBlocks = 64 / G;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint32_t slab = xcd_remap(blockIdx.x, gridDim.x);
    const uint32_t r0 = slab * slab_rows;
    const uint32_t r1 = min(rows, r0 + slab_rows);

    for (uint32_t c0 = 0; c0 < W; c0 += kChunkWords) {
        if (c0 + 256u * (uint32_t)wave >= W) continue;   // no lane of this wave has words here
        const uint32_t w = c0 + 4u * threadIdx.x;
        const bool active = w < W;
        u32x4 acc[G];
#pragma unroll
        for (int g = 0; g < G; ++g) acc[g] = u32x4{0, 0, 0, 0};
        for (uint32_t base = r0; base < r1; base += 32u * kBlocks) {
            uint32_t qv = 0;
            const uint32_t rb = base + 32u * (uint32_t)(lane % kBlocks);
            if (rb < r1) {
                qv = Q[(uint64_t)(lane / kBlocks) * qwords + rb / 32u];
                const uint32_t nrow = min(32u, r1 - rb);
                if (nrow < 32u) qv &= (1u << nrow) - 1u;
            }
            for (int jb = 0; jb < kBlocks; jb += 2) {
                const uint32_t rblk = base + 32u * (uint32_t)jb;
                if (rblk >= r1) break;                    // uniform
                uint64_t sel[G], any = 0;
#pragma unroll
                for (int g = 0; g < G; ++g) {
                    const uint32_t lo = __builtin_amdgcn_readlane(qv, g * kBlocks + jb);
                    const uint32_t hi = __builtin_amdgcn_readlane(qv, g * kBlocks + jb + 1);
                    sel[g] = (uint64_t)lo | ((uint64_t)hi << 32);
                    any |= sel[g];
                }
                while (any) {
                    u32x4 d[kDepth];
                    uint32_t idx[kDepth];
#pragma unroll
                    for (int k = 0; k < kDepth; ++k) {
                        d[k] = u32x4{0, 0, 0, 0};
                        idx[k] = 0;
                        if (any) {                        // uniform
                            idx[k] = (uint32_t)__builtin_ctzll(any);
                            any &= any - 1u;
                            if (active)
                                d[k] = load_words_nt<VEC>(DB + (uint64_t)(rblk + idx[k]) * pitch, w,
                                                          W);
                        }
                    }
#pragma unroll
                    for (int g = 0; g < G; ++g)
#pragma unroll
                        for (int k = 0; k < kDepth; ++k) {
                            const uint32_t m = G == 1 ? ~0u : 0u - (uint32_t)((sel[g] >> idx[k]) & 1u);
                            acc[g] ^= d[k] & u32x4{m, m, m, m};
                        }
                }
            }
        }
        if (active) {
#pragma unroll
            for (int g = 0; g < G; ++g) {
                uint32_t* o = out + (uint64_t)g * W + w;
                if (acc[g].x) atomicXor(o, acc[g].x);
                if (w + 1 < W && acc[g].y) atomicXor(o + 1, acc[g].y);
                if (w + 2 < W && acc[g].z) atomicXor(o + 2, acc[g].z);
                if (w + 3 < W && acc[g].w) atomicXor(o + 3, acc[g].w);
            }
        }
    }
}

// ---------------------------------------------------------------- matrix cores
// A workgroup (four waves, or NH = 2 groups of four side by side in columns)
// covers a slab of rows, 32 words per group of four waves and 32 TM queries.
// It walks the rows in pairs of chunks of 128 rows = two k-steps of 64.  Of
// the 8 blocks of 32 rows of a pair, lane half h of k-step s of chunk u takes
// block 4h + 2u + s, so a lane's selector words of a pair are 16 bytes.
//
// Operands (32x32x64 instruction, lane l: row or column l % 32, entries of
// half l / 32; the order of a half's 32 entries is free as long as both
// operands share it: register 0, 1, 2, 3 holds rows 4i + 0, 2, 1, 3 of the
// block, nibble i).
// * Queries: a lane's 32 entries are one selector word v; the registers are
//   (v >> j) & 0x11111111 moved to bit 1 (value 1.0): seven instructions.
// * Database: a wave brings its own block of 32 rows x 32 words; each thread
//   takes 16 words of one column (rows 4i + j, two values of j), transposes
//   them by nibbles in registers (and/or, then byte permutes) and stores them
//   to LDS, so that nibble position p of 32 rows becomes one 16-byte read; a
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
// transpose and LDS store of chunk ch + 2, the row loads.  Four LDS buffers
// of transposed rows, one barrier per chunk.  With one wave per SIMD (TM = 2)
// the instructions to issue are the limit (counters at 128 queries: issuing
// 56% of the time, matrix units busy 48%, 13% in waits), so with DMA the rows
// go straight to LDS in 16-byte pieces, into slots private to the wave, and
// the selector words once per workgroup, with buffers and slots known at
// compile time: 257 instructions per chunk instead of 293.
//
// Bound: up to 32 queries by HBM; above, by the matrix cores with the vector
// instructions beside them (about six per matrix instruction; a loop of bare
// 0/1 matrix instructions reaches 7.6 POP/s in the power budget, 7.3 with
// four vector instructions beside each).  Against lookups in 16-entry XOR
// tables in LDS, which this replaces, whole calls on one machine: 2^18 blocks of
// 3 KB, 8 queries 230 -> 146 us (5.5 TB/s), 32 252 -> 145 us, 64 353 -> 201 us,
// 128 618 -> 353 us, 1024 2.88 -> 2.36 ms (5.6 POP/s); 2^13 blocks, 16 queries 53
// -> 16 us, 128 151 -> 22 us, 1024 250 -> 97 us.  Other machines differ by up to
// 5%.
template <int N>
using I = std::integral_constant<int, N>;

constexpr int kParBufs = 4;                      // LDS buffers: transposed chunks,
constexpr int kParSlots = 4;                     // row chunks in flight,
constexpr int kParQSlots = 4;                    // selector words of pairs
constexpr uint32_t kParPair = 256;               // rows per pair of chunks
constexpr uint32_t kParMaxSlab = 1u << 18;       // rows counted in one accumulator
constexpr uint32_t kParWords = 32;               // words per group of four waves

__device__ inline f32x16 mfma_f4(const u32x4 a, const u32x4 b, const f32x16 c) {
    const i32x8 aa = {(int)a.x, (int)a.y, (int)a.z, (int)a.w, 0, 0, 0, 0};
    const i32x8 bb = {(int)b.x, (int)b.y, (int)b.z, (int)b.w, 0, 0, 0, 0};
    return __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(aa, bb, c, 4, 4, 0, 0, 0, 0);
}

__device__ inline u32x4 expand_selectors(uint32_t v) {
    constexpr uint32_t m = 0x22222222u;          // 1.0 in every nibble
    return u32x4{(v << 1) & m, (v >> 1) & m, v & m, (v >> 2) & m};
}

__device__ inline u32x4 bit_plane(const u32x4 t, int c) {
    return c < 3 ? (t & (0x11111111u << c)) : ((t >> 1) & 0x44444444u);
}

// s_waitcnt with only vmcnt constrained.
template <int N>
__device__ inline void wait_vmcnt() {
    static_assert(N >= 0 && N < 64, "vmcnt range");
    __builtin_amdgcn_s_waitcnt((N & 0xF) | ((N >> 4) << 14) | (0x7 << 4) | (0xF << 8));
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

// DMA: rows pass through LDS (16-byte aligned rows of whole 16-byte pieces),
// else through registers.  NT: non-temporal row loads.  `first`: this launch
// writes the output (init or zero, xor the product) instead of adding to it
// with atomics.
template <int TM, int NH, bool DMA, bool NT>
__global__ __launch_bounds__(256 * NH, TM == 1 ? 2 : 1) void k_chor_parity(
    const uint32_t* __restrict__ DB, uint64_t pitch, uint32_t rows, uint32_t W,
    const uint32_t* __restrict__ Q, uint32_t qwords, uint32_t B, uint32_t slab_rows,
    uint32_t n_qg, uint32_t cs0, uint32_t n_cs, bool first, const uint32_t* init, uint32_t* out) {
    constexpr int NW = kParWords;
    constexpr int kWgWords = NW * NH;
    constexpr int kTile = 4 * 8 * NW;                 // 16-byte entries of a transposed chunk
    static_assert(kParBufs * kTile * NH * 16 >= 32 * TM * kWgWords * 4, "outputs reuse the tiles");
    __shared__ u32x4 s_t[NH][kParBufs][4][8][NW];     // [block][nibble position][word]
    __shared__ u32x4 s_raw[DMA ? NH : 1][DMA ? 4 : 1][DMA ? kParSlots : 1][DMA ? 256 : 1];
    __shared__ u32x4 s_q[DMA ? kParQSlots : 1][DMA ? 32 * TM : 1][2];   // [query][half]: a pair's words
    static_assert(!DMA || (NH == 1 && TM == 2), "two selector loads per wave and pair");
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave_wg = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wave = wave_wg & 3, half = wave_wg >> 2;
    // The query groups of a column slice are consecutive and slabs outermost:
    // groups that read the same rows run on one XCD and share its L2.
    const uint32_t bid = xcd_remap(blockIdx.x, gridDim.x);
    const uint32_t qg = bid % n_qg;
    const uint32_t cs = cs0 + (bid / n_qg) % n_cs;
    const uint32_t slab = bid / (n_qg * n_cs);
    const uint32_t r0 = slab * slab_rows;
    const uint32_t r1 = min(rows, r0 + slab_rows);
    const uint32_t nch = 2u * ((r1 - r0 + kParPair - 1) / kParPair);

    // Fast: the chunk's pair lies inside the rows; else the chunk index and
    // the rows are clamped (the selector bits of rows past the end are
    // cleared, and a clamped chunk is not counted).
    typedef std::integral_constant<bool, true> Fast;
    typedef std::integral_constant<bool, false> Slow;
    const int h = lane >> 5;
    const int jn = lane & (NW - 1);
    const uint32_t c0 = (cs * NH + half) * NW;
    // First row of the wave's block of chunk ch: block 2h' + s is wave.
    auto block_row = [&](uint32_t ch) {
        return r0 + kParPair * (ch / 2u) +
               32u * (4u * (uint32_t)(wave >> 1) + 2u * (ch & 1u) + (uint32_t)(wave & 1));
    };
    // Through registers: thread's rows 4i + h and 4i + h + 2 of its column.
    const uint32_t* dcol = DB + min(c0 + jn, W - 1);
    auto load_d = [&](auto fast, uint32_t ch, uint32_t (&x)[2][8], int k0, int n) {
        if constexpr (decltype(fast)::value) {
            const uint32_t* p = dcol + (uint64_t)block_row(ch) * pitch + (uint64_t)h * pitch;
#pragma unroll
            for (int k = k0; k < k0 + n; ++k) {
                const uint32_t* a = p + (uint64_t)(4 * (k % 8) + 2 * (k / 8)) * pitch;
                x[k / 8][k % 8] = NT ? __builtin_nontemporal_load(a) : *a;
            }
        } else {
            const uint32_t rb = block_row(min(ch, nch - 1)) + h;
#pragma unroll
            for (int k = k0; k < k0 + n; ++k)
                x[k / 8][k % 8] =
                    dcol[(uint64_t)min(rb + 4 * (k % 8) + 2 * (k / 8), rows - 1) * pitch];
        }
    };
    // Through LDS: load k covers rows 8k .. 8k + 7 of the wave's block, lane:
    // row lane / 8, 16 bytes at lane % 8.
    const uint32_t* dseg = DB + min(c0 + 4u * (lane & 7), W - 4u);
    // The slots are addressed by LDS offset: with the array's name the
    // compiler orders every read of it behind all loads in flight (vmcnt 0),
    // where waiting for a slot's own loads, as the chunk's start does, is
    // enough.
    uint32_t slots = (uint32_t)(uintptr_t)(lds_word_t*)&s_raw[half % NH][DMA ? wave : 0][0][0];
    asm("" : "+s"(slots));
    // dnext: the lane's row of load 0 of the next pair to load (Fast).
    const uint32_t* dnext = dseg + (uint64_t)(block_row(kParSlots) + (lane >> 3)) * pitch;
    const uint64_t row8 = 8u * pitch;
    auto dma = [&](auto fast, uint32_t ch, auto slot, int odd, int k) {
        const uint32_t* src;
        if constexpr (decltype(fast)::value)
            src = dnext + (uint64_t)(8 * odd + k) * row8;
        else
            src = dseg + (uint64_t)min(block_row(min(ch, nch - 1)) + 8 * k + (lane >> 3), rows - 1) * pitch;
        __builtin_amdgcn_global_load_lds(
            (glb_void_t*)src,
            (lds_void_t*)(uintptr_t)(slots + 4096u * decltype(slot)::value + 1024u * k), 16, 0,
            NT ? 2 : 0);
    };
    auto raw = [&](auto slot, uint32_t (&x)[2][8]) {
        const lds_word_t* s = (const lds_word_t*)(uintptr_t)(slots + 4096u * decltype(slot)::value) +
                              NW * h + jn;
#pragma unroll
        for (int k = 0; k < 16; ++k) x[k / 8][k % 8] = s[(4 * (k % 8) + 2 * (k / 8)) * NW];
    };
    // A pair's selector words through LDS, for the whole workgroup (each wave
    // fetching them for itself cost 14% at 128 queries): load k of the wave
    // covers 8 queries of 8 words.
    uint32_t qslots = (uint32_t)(uintptr_t)(lds_word_t*)&s_q[0][0][0];
    asm("" : "+s"(qslots));
    const uint32_t* qsrc[2];
#pragma unroll
    for (int k = 0; k < 2; ++k)
        qsrc[k] = Q + (uint64_t)min(qg * TM * 32u + 8u * (2 * wave + k) + (lane >> 3), B - 1) * qwords;
    auto dma_q = [&](uint32_t pair) {
        const uint32_t w = (r0 + kParPair * min(pair, nch / 2u - 1)) / 32u + (lane & 7);
#pragma unroll
        for (int k = 0; k < 2; ++k)
            __builtin_amdgcn_global_load_lds(
                (glb_void_t*)(qsrc[k] + min(w, qwords - 1)),
                (lds_void_t*)(uintptr_t)(qslots + 1024u * TM * (pair % kParQSlots) +
                                         256u * (2 * wave + k)),
                4, 0, 0);
    };
    // Bits of the lane's 4 words of a pair that select rows (row < rows).
    auto row_mask = [&](uint32_t pair, int s) -> uint32_t {
        const uint32_t row = r0 + kParPair * min(pair, nch / 2u - 1) + 32u * (4u * h + s);
        const uint32_t n = row < rows ? min(32u, rows - row) : 0u;
        return n == 32u ? 0xFFFFFFFFu : (1u << n) - 1u;
    };
    auto get_q = [&](auto fast, uint32_t pair, u32x4 (&v)[TM]) {
#pragma unroll
        for (int a = 0; a < TM; ++a) {
            v[a] = *(const lds_quad_t*)(uintptr_t)(qslots + 1024u * TM * (pair % kParQSlots) +
                                                   32u * (32 * a + (lane & 31)) + 16u * h);
            if constexpr (!decltype(fast)::value)
#pragma unroll
                for (int s = 0; s < 4; ++s) v[a][s] &= row_mask(pair, s);
        }
    };
    // Selector words of the lane's query and half for a pair of chunks.
    // Queries past B repeat the last one; their outputs are not stored.
    const uint32_t* qrow[TM];
#pragma unroll
    for (int a = 0; a < TM; ++a)
        qrow[a] = Q + (uint64_t)min((qg * TM + a) * 32u + (lane & 31), B - 1) * qwords;
    auto load_q = [&](auto fast, uint32_t pair, u32x4 (&v)[TM]) {
        if constexpr (decltype(fast)::value) {
            const uint32_t w = (r0 + kParPair * pair) / 32u + 4u * h;
#pragma unroll
            for (int a = 0; a < TM; ++a) v[a] = *reinterpret_cast<const u32x4_word*>(qrow[a] + w);
        } else {
            const uint32_t w = (r0 + kParPair * min(pair, nch / 2u - 1)) / 32u + 4u * h;
#pragma unroll
            for (int s = 0; s < 4; ++s) {
                const uint32_t mask = row_mask(pair, s);
#pragma unroll
                for (int a = 0; a < TM; ++a) v[a][s] = qrow[a][min(w + s, qwords - 1)] & mask;
            }
        }
    };
    auto put = [&](int buf, const uint32_t (&x)[2][8], int o) {   // nibbles o, o + 2, ..
        uint32_t* dst = reinterpret_cast<uint32_t*>(&s_t[half][buf][wave][0][jn]) + 2 * h;
#pragma unroll
        for (int p = o; p < 8; p += 2)
            *reinterpret_cast<uint64_t*>(dst + p * NW * 4) =
                (uint64_t)x[0][p] | ((uint64_t)x[1][p] << 32);
    };
    auto get = [&](int buf, u32x4 (&t)[2][2]) {
#pragma unroll
        for (int s = 0; s < 2; ++s)
#pragma unroll
            for (int g = 0; g < 2; ++g)
                t[s][g] = s_t[half][buf][2 * h + s][wave + 4 * g][jn];
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

    uint32_t x[2][2][8];        // rows of chunks ch + 2, ch + 3 (DMA: of ch + 2)
    u32x4 qv[2][TM];            // selector words of this pair of chunks and the next
    u32x4 t[2][2][2];           // database operands of chunks ch, ch + 1
    u32x4 fa[2][TM], fb[2];     // expanded operands: k-step, slice
    {
        uint32_t x0[2][8], x1[2][8];
        if constexpr (DMA) {
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                dma(Slow{}, 0, I<0>{}, 0, k);
                dma(Slow{}, 1, I<1>{}, 1, k);
                dma(Slow{}, 2, I<2>{}, 0, k);
                dma(Slow{}, 3, I<3>{}, 1, k);
            }
            for (int c = 0; c < 3; ++c) dma_q(c);
            wait_vmcnt<0>();
            asm volatile("" ::: "memory");
            raw(I<0>{}, x0);
            raw(I<1>{}, x1);
        } else {
            load_d(Slow{}, 0, x0, 0, 16);
            load_d(Slow{}, 1, x1, 0, 16);
            load_q(Slow{}, 0, qv[0]);
            load_q(Slow{}, 1, qv[1]);
            load_d(Slow{}, 2, x[0], 0, 16);
            load_d(Slow{}, 3, x[1], 0, 16);
        }
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
        if constexpr (DMA) get_q(Slow{}, 0, qv[0]);
        get(0, t[0]);
#pragma unroll
        for (int a = 0; a < TM; ++a) fa[0][a] = expand_selectors(qv[0][a].x);
        fb[0] = bit_plane(t[0][0][0], 0);
    }
    // Chunk ch = 4 (a multiple) + u: the first or second of its pair, whose
    // words are in qv[u / 2].  Buffer u + 2, which it fills, was last read by
    // get() in chunk ch - 2, before two barriers; slot u, which its loads
    // refill, by this wave in chunk ch - 2.
    auto body = [&](auto fast, uint32_t ch, auto u_) {
        constexpr int u = decltype(u_)::value, cur = u % 2, par = u / 2;
        if constexpr (DMA) {
            // Chunk ch + 2 has landed once at most the loads of the chunk
            // since are outstanding: four, and two of selector words if it is
            // even.  The words of pair p, loaded at chunk 2p - 6, have then
            // landed by chunk 2p - 2, and its barrier shows them to all waves
            // before they are read at chunk 2p - 1.
            wait_vmcnt<4 + (cur == 0 ? 0 : 2)>();
            asm volatile("" ::: "memory");
            raw(I<(u + 2) % 4>{}, x[0]);
            if constexpr (cur == 1) get_q(fast, ch / 2u + 1u, qv[par ^ 1]);
        }
        uint32_t (&xc)[2][8] = x[DMA ? 0 : cur];
        get((u + 1) % 4, t[cur ^ 1]);
        uint32_t q1[TM], qn[TM];    // second k-step's words, the next chunk's first
#pragma unroll
        for (int a = 0; a < TM; ++a) {
            q1[a] = qv[par][a][2 * cur + 1];
            qn[a] = cur == 0 ? qv[par][a][2] : qv[par ^ 1][a][0];
        }
#pragma unroll
        for (int sl = 0; sl < 16; ++sl) {
            const int s = sl / 8, l = sl % 8, g = l / 4, c = l % 4;
            // Two waves per SIMD fill each other's gaps best when every
            // slice keeps its place (32 queries 151 -> 142 us).
            if constexpr (TM == 1) __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int a = 0; a < TM; ++a) acc[a][g][c] = mfma_f4(fa[s][a], fb[sl & 1], acc[a][g][c]);
            fb[(sl + 1) & 1] = sl + 1 < 16 ? bit_plane(t[cur][(sl + 1) / 8][(sl + 1) / 4 % 2], (sl + 1) % 4)
                                           : bit_plane(t[cur ^ 1][0][0], 0);
            if (l < TM) fa[s ^ 1][l] = expand_selectors(s == 0 ? q1[l] : qn[l]);
            if (s == 0) {
                transpose_nibbles(xc[l % 2], l / 2);
            } else if (l < 4) {
                transpose_bytes(xc[l % 2], l / 2);
                if (l % 2 == 1) put((u + 2) % 4, xc, l / 2);
            } else {
                if constexpr (DMA) {
                    if (cur == 0 && l == 4) dma_q(ch / 2u + 3u);
                    dma(fast, ch + kParSlots, I<u>{}, cur, l - 4);
                } else {
                    if (cur == 1 && l == 4) load_q(fast, ch / 2u + 2u, qv[par]);
                    load_d(fast, ch + 4, xc, 4 * (l - 4), 4);
                }
            }
            if constexpr (TM == 1) __builtin_amdgcn_sched_barrier(0);
        }
        if constexpr (DMA && cur == 1) dnext += 32u * row8;
        if constexpr (DMA && decltype(fast)::value) {
            // Seven vector instructions after each matrix instruction (there
            // are about six): the one wave of a SIMD cannot issue past a
            // matrix instruction that waits for the unit.
#pragma unroll
            for (int i = 0; i < 16 * TM; ++i) {
                __builtin_amdgcn_sched_group_barrier(0x8, 1, 0);
                __builtin_amdgcn_sched_group_barrier(0x2, 7, 0);
            }
        }
        lds_barrier();
    };
    const uint32_t nfull = 2u * ((r1 - r0) / kParPair);
    uint32_t ch = 0;
    for (; ch + 3 + kParSlots < nfull; ch += 4) {
        body(Fast{}, ch, I<0>{});
        body(Fast{}, ch + 1, I<1>{});
        body(Fast{}, ch + 2, I<2>{});
        body(Fast{}, ch + 3, I<3>{});
    }
    for (; ch < nch; ch += 4) {
        body(Slow{}, ch, I<0>{});
        body(Slow{}, ch + 1, I<1>{});
        if (ch + 2 < nch) {
            body(Slow{}, ch + 2, I<2>{});
            body(Slow{}, ch + 3, I<3>{});
        }
    }
    // Row loads past the last chunk may still be landing in LDS.
    if constexpr (DMA) wait_vmcnt<0>();

    // Parities: tile c of nibble position wave + 4g holds bit c; register v
    // of lane half h holds query 8 (v/4) + 4 h + v % 4.  The waves' nibbles
    // meet in LDS.
    uint32_t* s_out = reinterpret_cast<uint32_t*>(&s_t[0][0][0][0][0]);   // [32 TM][kWgWords]
    __syncthreads();
    for (int i = tid; i < 32 * TM * kWgWords; i += 256 * NH) s_out[i] = 0;
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
            atomicOr(&s_out[(32 * a + 8 * (v / 4) + 4 * h + v % 4) * kWgWords + half * NW + jn],
                     y << (4 * wave));
        }
    __syncthreads();
    for (int i = tid; i < 32 * TM * kWgWords; i += 256 * NH) {
        const uint32_t b = qg * TM * 32u + i / kWgWords, w = cs * kWgWords + i % kWgWords;
        if (b >= B || w >= W) continue;
        const uint32_t y = s_out[i];
        const uint64_t at = (uint64_t)b * W + w;
        if (first) out[at] = init ? init[at] ^ y : y;
        else if (y) atomicXor(out + at, y);
    }
}

// Row slabs of a launch.  One workgroup runs per CU, so a launch takes
// ceil(workgroups / 256) rounds, each of a slab's pairs of chunks plus the
// pipeline fill and the epilogue, worth about three pairs; take the count with
// the least total (2^18 blocks of 3 KB: 128 queries, 48 workgroups per slab, 5
// slabs 359 us, 8 410, 16 (taken) 363, 21 370; 64 queries 10 slabs 193, 16 227, 21
// (taken) 196; 32 queries 10 slabs 226, 21 (taken) 140, 32 173).
struct Slabs {
    uint32_t count, rows;
};

Slabs parity_slabs(uint32_t rows, uint64_t per_slab) {
    const uint32_t pairs = (rows + kParPair - 1) / kParPair;
    const uint32_t lo = (rows + kParMaxSlab - 1) / kParMaxSlab;
    const uint32_t hi = std::max(lo, std::min(pairs, 64u));
    uint32_t best = lo;
    double best_t = 1e300;
    for (uint32_t n = lo; n <= hi; ++n) {
        const double t = (double)((per_slab * n + 255) / 256) * ((pairs + n - 1) / n + 3);
        if (t < best_t) {
            best_t = t;
            best = n;
        }
    }
    const uint32_t slab = (pairs + best - 1) / best * kParPair;
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
    // A grid holds fewer than 2^32 threads; very wide blocks take several
    // launches of `most` column slices each.
    const uint64_t most = ((1ull << 32) - 1) / (256 * NH) / ((uint64_t)n_qg * sl.count);
    if (most == 0) return PIR_ERR_SHAPE;
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
    const bool dma = TM == 2 && (uintptr_t)d_DB % 16 == 0 && words % 4 == 0 && pitch % 4 == 0;
    for (uint64_t cs0 = 0; cs0 < n_cs; cs0 += most) {
        const uint32_t cs = (uint32_t)std::min(most, n_cs - cs0);
        const uint32_t blocks = n_qg * cs * sl.count;
#define PIR_PARITY(DMA, X)                                                                   \
    k_chor_parity<TM, NH, DMA, X><<<blocks, 256 * NH, 0, s>>>(                               \
        d_DB, pitch, rows, words, d_Q, (rows + 31) / 32, B, sl.rows, n_qg, (uint32_t)cs0, cs, first, \
        d_init, d_out)
        if constexpr (TM == 2) {
            if (dma) {
                if (nt) PIR_PARITY(true, true); else PIR_PARITY(true, false);
                PIR_LAUNCH_CHECK();
                continue;
            }
        }
        if (nt) PIR_PARITY(false, true); else PIR_PARITY(false, false);
#undef PIR_PARITY
        PIR_LAUNCH_CHECK();
    }
    return PIR_OK;
}

// Two queries select three quarters of the rows.  Where a database is long
// enough to be bound by HBM, reading only those beats the matrix cores, which
// read all (us, matrix cores / stream: 2^18 blocks of 3 KB 141 / 127, 2^19 271 /
// 221, 800 MB of 2 KB blocks 151 / 135; 600 MB of 8 KB blocks 107 / 115, 2^17
// blocks of 3 KB 79 / 87); short rows leave most of its waves idle (800 MB of 1
// KB blocks 156 / 179), and few rows too few slabs (800 MB of 16 KB blocks 146 /
// 149, 400 MB 77 / 124).
bool stream_two(uint32_t rows, uint32_t words) {
    return words >= 480u && rows >= 65536u && (uint64_t)rows * words >= (700ull << 18);
}

template <int G>
pir_status launch_stream(const uint32_t* d_DB, uint32_t rows, uint32_t words, uint64_t pitch,
                         const uint32_t* d_Q, uint32_t* d_out, hipStream_t s) {
    // Enough rows in flight to stream HBM (32 per wave), few enough slabs to
    // keep the output atomics (slabs x words, all onto the same words) down:
    // at most one workgroup per CU (two for two queries), and at least 256
    // rows per slab.
    // (Measured on 2^18 and 2^16 rows of 3 KB: fewer workgroups starve the
    // stream on the large database, more slabs spend the small one's time in
    // atomics.)
    constexpr uint32_t kTarget = 256u * G;
    uint64_t slab = ((uint64_t)rows + kTarget - 1) / kTarget;
    slab = (slab + 31) / 32 * 32;
    if (slab < 256) slab = 256;
    const uint64_t blocks = (rows + slab - 1) / slab;
    if (blocks > 0x7FFFFFFFull) return PIR_ERR_SHAPE;
    const bool vec = ((uintptr_t)d_DB % 16 == 0) && (words % 4 == 0) && (pitch % 4 == 0);
    const uint32_t qwords = (rows + 31) / 32;
    if (vec)
        k_chor_stream<G, true><<<(uint32_t)blocks, kThreads, 0, s>>>(d_DB, pitch, rows, words, d_Q,
                                                                     qwords, (uint32_t)slab, d_out);
    else
        k_chor_stream<G, false><<<(uint32_t)blocks, kThreads, 0, s>>>(d_DB, pitch, rows, words, d_Q,
                                                                      qwords, (uint32_t)slab, d_out);
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
    if (B == 1 || (B == 2 && stream_two(rows, words))) {
        const pir_status st = chor_init(d_out, d_init, (uint64_t)B * words, s);
        if (st != PIR_OK) return st;
        if (B == 1) return launch_stream<1>(d_DB, rows, words, pitch, d_Q, d_out, s);
        return launch_stream<2>(d_DB, rows, words, pitch, d_Q, d_out, s);
    }
    // Up to 32 queries one 32-query tile with two workgroup halves; above,
    // 64 queries per workgroup, which halves the masks and the transposes
    // per matrix instruction (2^18 blocks of 3 KB: 64 queries 196 us against
    // 255 as two 32-query groups, 40 queries 192 against 249; 32 queries 197
    // against 141 as one).
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
