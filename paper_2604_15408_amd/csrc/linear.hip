// Linear layers and LayerNorm over packed rows (the "late blocks" of Section 4.3 item 4: after the
// pruning point the projections and the MLP run on the packed buffer, so their cost is linear in the
// number of kept tokens), for gfx950.
//
// The linear kernel itself is in linear_kernel.h (instantiated per input type in linear_f16.hip and linear_bf16.hip); this
// file launches it in the shape that linear_walk.h picks and holds LayerNorm.
//
// layernorm_kernel: one wavefront per row, the row held in registers, two passes (mean, then the
//   biased variance of the centred values) in fp32.
//
// Rows: the caller passes a capacity and, optionally, a device pointer to the real row count (for
// example &cu_seqlens[B]); work-groups past it exit, so nothing is read back to the host.
#include "common.h"
#include "linear_kernel.h"

namespace ragged {
namespace {

// Sum over the 64 lanes of a wavefront (fp32), result in every lane: DPP rotations inside each
// 16-lane row, then the lane-swap instructions across rows.
template <int kCtrl>
__device__ __forceinline__ float dpp_f32(float v) {
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), kCtrl, 0xf, 0xf, true));
}
__device__ __forceinline__ unsigned opaque_copy_u(unsigned x) {
    unsigned yv;
    asm volatile("v_mov_b32 %0, %1" : "=v"(yv) : "v"(x));
    return yv;
}
__device__ __forceinline__ float wave_sum_f32(float v) {
    v += dpp_f32<0x128>(v);                                    // row_ror:8
    v += dpp_f32<0x124>(v);                                    // row_ror:4
    v += dpp_f32<0x122>(v);                                    // row_ror:2
    v += dpp_f32<0x121>(v);                                    // row_ror:1
    const unsigned u = __builtin_bit_cast(unsigned, v);
    const auto a = __builtin_amdgcn_permlane16_swap(u, opaque_copy_u(u), false, false);
    const unsigned a0 = a[0], a1 = a[1];
    v = __builtin_bit_cast(float, a0) + __builtin_bit_cast(float, a1);
    const unsigned u2 = __builtin_bit_cast(unsigned, v);
    const auto b = __builtin_amdgcn_permlane32_swap(u2, opaque_copy_u(u2), false, false);
    const unsigned b0 = b[0], b1 = b[1];
    return __builtin_bit_cast(float, b0) + __builtin_bit_cast(float, b1);
}

constexpr int kLnChunks = 4;                                   // 16-byte chunks per lane: C <= 64 * 4 * 8 = 2048

template <typename In>
__global__ __launch_bounds__(kBlockThreads)
void layernorm_kernel(const uint16_t* x, const uint16_t* __restrict__ gamma,          // y may be x: no restrict
                      const uint16_t* __restrict__ beta, uint16_t* y, int rows_cap,
                      const int32_t* __restrict__ rows_dev, int C, float eps) {
    int rows = rows_cap;
    if (rows_dev) { const int r = *rows_dev; rows = r < rows ? r : rows; }
    const int lane = threadIdx.x & (kWaveSize - 1);
    const int row = blockIdx.x * (kBlockThreads / kWaveSize) + (threadIdx.x >> 6);
    if (row >= rows) return;
    const int chunks = C / 8;
    const uint4* src = reinterpret_cast<const uint4*>(x + (int64_t)row * C);
    // every load of the kernel is issued up front (the row, and the scale / shift vectors the last
    // pass needs), so the two reductions run while gamma and beta are still on their way
    uint4 raw_x[kLnChunks], raw_g[kLnChunks], raw_b[kLnChunks];
#pragma unroll
    for (int i = 0; i < kLnChunks; ++i) {
        const int c = lane + kWaveSize * i;
        if (c < chunks) {
            raw_x[i] = src[c];
            raw_g[i] = reinterpret_cast<const uint4*>(gamma)[c];
            raw_b[i] = reinterpret_cast<const uint4*>(beta)[c];
        }
    }
    float v[kLnChunks][8];
    float sum = 0.f;
#pragma unroll
    for (int i = 0; i < kLnChunks; ++i) {
        const int c = lane + kWaveSize * i;
        if (c < chunks) {
            unpack8(In{}, raw_x[i], v[i]);
#pragma unroll
            for (int e = 0; e < 8; ++e) sum += v[i][e];
        } else {
#pragma unroll
            for (int e = 0; e < 8; ++e) v[i][e] = 0.f;
        }
    }
    const float mean = wave_sum_f32(sum) / (float)C;
    float sq = 0.f;
#pragma unroll
    for (int i = 0; i < kLnChunks; ++i)
        if (lane + kWaveSize * i < chunks)
#pragma unroll
            for (int e = 0; e < 8; ++e) { const float d = v[i][e] - mean; sq = __builtin_fmaf(d, d, sq); }
    const float rstd = 1.0f / sqrtf(wave_sum_f32(sq) / (float)C + eps);
    uint4* dst = reinterpret_cast<uint4*>(y + (int64_t)row * C);
#pragma unroll
    for (int i = 0; i < kLnChunks; ++i) {
        const int c = lane + kWaveSize * i;
        if (c < chunks) {
            float gm[8], bt[8], out[8];
            unpack8(In{}, raw_g[i], gm);
            unpack8(In{}, raw_b[i], bt);
#pragma unroll
            for (int e = 0; e < 8; ++e) out[e] = __builtin_fmaf((v[i][e] - mean) * rstd, gm[e], bt[e]);
            dst[c] = pack8(In{}, out);
        }
    }
}

}  // namespace

hipError_t launch_linear(const void* x, const void* w, const void* bias, const void* res, void* y, int rows_cap,
                         const int32_t* rows_dev, int rows_hint, int N, int K, int act, ragged_dtype dt,
                         hipStream_t stream) {
    const TileShape c = pick_linear_shape(rows_hint, N, K, act);
    const LinearGrid g(c.nj, c.mt, c.per_cu, rows_cap, N);
    const LinearArgs args{static_cast<const uint16_t*>(x), static_cast<const uint16_t*>(w), static_cast<const uint16_t*>(bias),
                          static_cast<const uint16_t*>(res), static_cast<uint16_t*>(y), rows_dev, rows_cap, N, K, act, g.n_tiles,
                          g.panel, div_magic((uint32_t)g.panel), div_magic((uint32_t)g.last)};
    return dt == RAGGED_F16 ? launch_linear_f16(c, g.groups, args, stream)
                            : launch_linear_bf16(c, g.groups, args, stream);
}

int layernorm_max_width() { return kWaveSize * kLnChunks * 8; }

hipError_t launch_layernorm(const void* x, const void* gamma, const void* beta, void* y, int rows_cap,
                            const int32_t* rows_dev, int C, float eps, ragged_dtype dt, hipStream_t stream) {
    const int per = kBlockThreads / kWaveSize;
    const dim3 grid((rows_cap + per - 1) / per), block(kBlockThreads);
    const uint16_t* xp = static_cast<const uint16_t*>(x);
    const uint16_t* gp = static_cast<const uint16_t*>(gamma);
    const uint16_t* bp = static_cast<const uint16_t*>(beta);
    uint16_t* yp = static_cast<uint16_t*>(y);
    hipError_t err;
    if (dt == RAGGED_F16)
        err = launch_kernel((layernorm_kernel<F16>), grid, block, stream, xp, gp, bp, yp, rows_cap, rows_dev, C, eps);
    else
        err = launch_kernel((layernorm_kernel<BF16>), grid, block, stream, xp, gp, bp, yp, rows_cap, rows_dev, C, eps);
    return err;
}

}  // namespace ragged
