// Database handle metadata and refresh kernels.
//
// The handle keeps one word per row, rowsum[r] = sum_j D[r][j] (exact for
// C < 2^24).  The matrix-core path works on centred bytes and limbs and adds
// back a term built from it (see answer_mfma.hip); it depends only on the
// database, so it is computed once when the handle is opened and again for
// the rows a refresh rewrites.
#include "qpir_internal.h"

namespace {

// 16 bytes at any alignment.
typedef u32x4 u32x4_any __attribute__((aligned(1)));

__device__ inline uint32_t add_bytes(const u32x4 d, uint32_t acc) {
    acc = __builtin_amdgcn_udot4(d.x, 0x01010101u, acc, false);
    acc = __builtin_amdgcn_udot4(d.y, 0x01010101u, acc, false);
    acc = __builtin_amdgcn_udot4(d.z, 0x01010101u, acc, false);
    return __builtin_amdgcn_udot4(d.w, 0x01010101u, acc, false);
}

// One wave per row: byte sums through v_dot4_u32_u8 against 0x01010101.
// Bound by reading D.  Rows start anywhere and have any length; four loads
// per lane in flight (20000 unaligned rows of 10007 bytes: byte loads 142-189
// us, 30.6 us now).
__global__ __launch_bounds__(256) void k_rowsum(const uint8_t* __restrict__ D, uint64_t pitch,
                                                uint32_t R, uint32_t C,
                                                uint32_t* __restrict__ rowsum) {
    const uint32_t lane = threadIdx.x & 63;
    const uint32_t waves = gridDim.x * (blockDim.x >> 6);
    const uint32_t C16 = C & ~15u;
    for (uint32_t r = blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6); r < R; r += waves) {
        const uint8_t* row = D + (uint64_t)r * pitch;
        uint32_t acc = C16 + lane < C ? row[C16 + lane] : 0u;   // ragged tail, a byte per lane
        uint64_t c = 16u * lane;
        for (; c + 3 * 1024 < C16; c += 4 * 1024) {
            u32x4 d[4];
#pragma unroll
            for (int k = 0; k < 4; ++k)
                d[k] = __builtin_nontemporal_load(
                    reinterpret_cast<const u32x4_any*>(row + c + 1024 * k));
#pragma unroll
            for (int k = 0; k < 4; ++k) acc = add_bytes(d[k], acc);
        }
        for (; c < C16; c += 1024)
            acc = add_bytes(
                __builtin_nontemporal_load(reinterpret_cast<const u32x4_any*>(row + c)), acc);
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) acc += __shfl_xor(acc, off);
        if (lane == 0) rowsum[r] = acc;
    }
}

// A refreshed row: one workgroup copies new row i into place and sums its
// bytes on the way, four 16-byte pieces per thread in flight (a second pass
// that read the row back took as long again: 328 rows of 16384 bytes, 14.3 us
// in two kernels, 5.1 us here).
__global__ __launch_bounds__(256) void k_update_rows(uint8_t* __restrict__ D, uint64_t pitch,
                                                     uint32_t R, uint32_t C,
                                                     const uint32_t* __restrict__ rows,
                                                     const uint8_t* __restrict__ src,
                                                     uint32_t* __restrict__ rowsum) {
    __shared__ uint32_t s_sum[4];
    const uint32_t r = rows[blockIdx.x];
    if (r >= R) return;   // uniform
    uint8_t* dst = D + (uint64_t)r * pitch;
    const uint8_t* s = src + (uint64_t)blockIdx.x * C;
    const uint32_t C16 = C & ~15u;
    uint32_t acc = 0;
    if (C16 + threadIdx.x < C) {
        const uint8_t v = s[C16 + threadIdx.x];
        dst[C16 + threadIdx.x] = v;
        acc = v;
    }
    for (uint64_t c0 = 16u * threadIdx.x; c0 < C16; c0 += 4 * 4096) {
        u32x4 d[4];
#pragma unroll
        for (int k = 0; k < 4; ++k)
            d[k] = c0 + 4096 * k < C16 ? *reinterpret_cast<const u32x4_any*>(s + c0 + 4096 * k)
                                       : u32x4{0, 0, 0, 0};
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            if (c0 + 4096 * k < C16) *reinterpret_cast<u32x4_any*>(dst + c0 + 4096 * k) = d[k];
            acc = add_bytes(d[k], acc);
        }
    }
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) acc += __shfl_xor(acc, off);
    if ((threadIdx.x & 63) == 0) s_sum[threadIdx.x >> 6] = acc;
    __syncthreads();
    if (threadIdx.x == 0) rowsum[r] = s_sum[0] + s_sum[1] + s_sum[2] + s_sum[3];
}

}  // namespace

pir_status launch_rowsum(const pir_db_t* db, hipStream_t s) {
    const uint32_t R = (uint32_t)db->rows;
    const uint32_t blocks = (uint32_t)std::min<uint64_t>((db->rows + 3) / 4, 8192);
    k_rowsum<<<blocks, 256, 0, s>>>(db->D, db->pitch, R, (uint32_t)db->cols, db->rowsum);
    PIR_LAUNCH_CHECK();
    return PIR_OK;
}

pir_status launch_update_rows(const pir_db_t* db, const uint32_t* rows, uint32_t m,
                              const uint8_t* src, hipStream_t s) {
    if (m == 0) return PIR_OK;
    k_update_rows<<<m, 256, 0, s>>>(db->D, db->pitch, (uint32_t)db->rows, (uint32_t)db->cols,
                                    rows, src, db->rowsum);
    PIR_LAUNCH_CHECK();
    return PIR_OK;
}
