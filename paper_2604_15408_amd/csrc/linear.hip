// Linear layers and LayerNorm over packed rows (the "late blocks" of Section 4.3 item 4: after the
// pruning point the projections and the MLP run on the packed buffer, so their cost is linear in the
// number of kept tokens), for gfx950.
//
// The linear kernel itself is in linear_kernel.h (instantiated per input type in linear_f16.hip and linear_bf16.hip); this
// file launches it in the shape that linear_walk.h picks and holds LayerNorm.
//
// layernorm_kernel: 16, 32 or 64 lanes per row, the row held in registers, two passes (mean, then the
//   biased variance of the centred values) in fp32.
//
// Rows: the caller passes a capacity and, optionally, a device pointer to the real row count (for
// example &cu_seqlens[B]); work-groups past it exit, so nothing is read back to the host.
#include "common.h"
#include "linear_kernel.h"

namespace ragged {
namespace {

// Sum over aligned groups of L = 16, 32 or 64 lanes (fp32), result in every lane: DPP rotations inside each
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
template <int L>
__device__ __forceinline__ float lanes_sum_f32(float v) {
    v += dpp_f32<0x128>(v);                                    // row_ror:8
    v += dpp_f32<0x124>(v);                                    // row_ror:4
    v += dpp_f32<0x122>(v);                                    // row_ror:2
    v += dpp_f32<0x121>(v);                                    // row_ror:1
    if (L == 16) return v;
    const unsigned u = __builtin_bit_cast(unsigned, v);
    const auto a = __builtin_amdgcn_permlane16_swap(u, opaque_copy_u(u), false, false);
    const unsigned a0 = a[0], a1 = a[1];
    v = __builtin_bit_cast(float, a0) + __builtin_bit_cast(float, a1);
    if (L == 32) return v;
    const unsigned u2 = __builtin_bit_cast(unsigned, v);
    const auto b = __builtin_amdgcn_permlane32_swap(u2, opaque_copy_u(u2), false, false);
    const unsigned b0 = b[0], b1 = b[1];
    return __builtin_bit_cast(float, b0) + __builtin_bit_cast(float, b1);
}

// A row is NC chunks of V consecutive values for each of L lanes, chunk i of lane l at (L i + l) V; a wavefront has 64 / L rows at
// a time.  FULL: C == L V NC, every lane has all of them; otherwise chunks past C are not there.
// Few rows are a chain of latencies (launch, row, two reductions, store); many are bound by memory, if a row costs little beside
// its own bytes.  So gamma and beta, twice the bytes of a row, stay in registers while a group of lanes takes every stride-th row, the
// next of which is on its way while it works on one; 16 lanes read and write whole cache lines; and narrow rows share the
// divisions and the root of a wavefront.  With a wavefront to every row, eight values a chunk (of which a third of the lanes had
// none at C = 768) and room for C = 2048 in every launch, us before and now: 25 216 x 768 16.1 and 14.1 (5.5 TB/s), 8850 x 768
// 7.7 and 7.4, 25 216 x 384 11.5 and 8.9, 25 216 x 192 11.1 and 6.1, 1334 rows of either 3.9 and 3.7.
constexpr int kLnWaves = 16384;                                // about twice what the chip holds at once (8850 x 1024: 8.1 us, with half of it 8.7)
template <typename In, int L, int V, int NC, bool FULL>
__global__ __launch_bounds__(kBlockThreads)
void layernorm_kernel(const uint16_t* x, const uint16_t* __restrict__ gamma,          // y may be x: no restrict
                      const uint16_t* __restrict__ beta, uint16_t* y, int rows_cap,
                      const int32_t* __restrict__ rows_dev, int C, float eps, int64_t stride) {
    typedef LinearLine<V> Chunk;
    int rows = rows_cap;
    if (rows_dev) { const int r = *rows_dev; rows = r < rows ? r : rows; }
    const int sub = threadIdx.x % L;
    int64_t row = (int64_t)blockIdx.x * (kBlockThreads / L) + threadIdx.x / L;
    if (row >= rows) return;
    auto there = [&](int i) { return FULL || (sub + L * i) * V < C; };
    auto load = [&](const uint16_t* src, Chunk (&c)[NC]) {
#pragma unroll
        for (int i = 0; i < NC; ++i)
            if (there(i)) c[i] = reinterpret_cast<const Chunk*>(src)[sub + L * i];
    };
    // the first row and what the last pass needs are requested together
    Chunk next[NC], g_raw[NC], b_raw[NC];
    load(x + row * C, next);
    load(gamma, g_raw);
    load(beta, b_raw);
    for (; row < rows; row += stride) {
        float v[NC][V];
        float sum = 0.f;
#pragma unroll
        for (int i = 0; i < NC; ++i) {
            if (there(i)) {
                next[i].unpack(In{}, v[i]);
#pragma unroll
                for (int e = 0; e < V; ++e) sum += v[i][e];
            } else {
#pragma unroll
                for (int e = 0; e < V; ++e) v[i][e] = 0.f;
            }
        }
        if (row + stride < rows) load(x + (row + stride) * C, next);
        const float mean = lanes_sum_f32<L>(sum) / (float)C;
        float sq = 0.f;
#pragma unroll
        for (int i = 0; i < NC; ++i)
            if (there(i))
#pragma unroll
                for (int e = 0; e < V; ++e) { const float d = v[i][e] - mean; sq = __builtin_fmaf(d, d, sq); }
        const float rstd = 1.0f / sqrtf(lanes_sum_f32<L>(sq) / (float)C + eps);
        Chunk* dst = reinterpret_cast<Chunk*>(y + row * C);
#pragma unroll
        for (int i = 0; i < NC; ++i) {
            if (there(i)) {
                float gm[V], bt[V], out[V];
                g_raw[i].unpack(In{}, gm);
                b_raw[i].unpack(In{}, bt);
#pragma unroll
                for (int e = 0; e < V; ++e) out[e] = __builtin_fmaf((v[i][e] - mean) * rstd, gm[e], bt[e]);
                dst[sub + L * i] = Chunk::pack(In{}, out);
            }
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

int layernorm_max_width() { return kWaveSize * 4 * 8; }

hipError_t launch_layernorm(const void* x, const void* gamma, const void* beta, void* y, int rows_cap,
                            const int32_t* rows_dev, int C, float eps, ragged_dtype dt, hipStream_t stream) {
    auto launch = [&](auto kernel, int lanes) {
        // the same number of rows for every group of lanes (but for one), as few as the wavefronts that run at once allow
        const int64_t at_once = (int64_t)kLnWaves * (kWaveSize / lanes), each = (rows_cap + at_once - 1) / at_once;
        const int per = kBlockThreads / lanes, groups = (int)(((rows_cap + each - 1) / each + per - 1) / per);
        return launch_kernel(kernel, dim3(groups), dim3(kBlockThreads), stream, static_cast<const uint16_t*>(x),
                             static_cast<const uint16_t*>(gamma), static_cast<const uint16_t*>(beta), static_cast<uint16_t*>(y),
                             rows_cap, rows_dev, C, eps, (int64_t)groups * per);
    };
    auto typed = [&](auto in) {
        typedef decltype(in) In;
        // widths of 8, 12 or 16 values for each of 16, 32 or 64 lanes fill whole wavefronts
#define LN_FULL(L, V, NC) if (C == L * V * NC) return launch(layernorm_kernel<In, L, V, NC, true>, L);
        LN_FULL(16, 8, 1) LN_FULL(16, 4, 3) LN_FULL(32, 8, 1) LN_FULL(32, 4, 3) LN_FULL(64, 8, 1) LN_FULL(64, 4, 3) LN_FULL(64, 8, 2)
        LN_FULL(64, 2, 5) LN_FULL(64, 2, 7)
#undef LN_FULL
        if (C <= 512) return launch(layernorm_kernel<In, 64, 8, 1, false>, 64);
        if (C <= 1024) return launch(layernorm_kernel<In, 64, 8, 2, false>, 64);
        return launch(layernorm_kernel<In, 64, 8, 4, false>, 64);
    };
    return dt == RAGGED_F16 ? typed(F16{}) : typed(BF16{});
}

}  // namespace ragged
