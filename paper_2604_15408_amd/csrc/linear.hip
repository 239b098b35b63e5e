// Linear layers and LayerNorm over packed rows (the "late blocks" of Section 4.3 item 4: after the
// pruning point the projections and the MLP run on the packed buffer, so their cost is linear in the
// number of kept tokens), for gfx950.
//
// The linear kernel itself is in linear_kernel.h (instantiated per input type in linear_f16.hip and linear_bf16.hip); this
// file launches it in the shape that linear_walk.h picks and holds LayerNorm.
//
// layernorm_kernel: 16, 32 or 64 lanes per row, the row held in registers, two passes (mean, then the
//   biased variance of the centred values) in fp32, in an order that does not depend on the form.
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

// Value e of a chunk plus a, rounded once.  fp16: one mixed-precision fma with `one` = 1, which the compiler must not see as a
// constant (it would make a conversion and a sum of it again).
__device__ __forceinline__ float plus_value(F16, const LinearLine<8>& c, int e, float a, float one) {
    return __builtin_fmaf((float)__builtin_bit_cast(_Float16, (uint16_t)(c.w[e / 2] >> 16 * (e % 2))), one, a);
}
__device__ __forceinline__ float plus_value(BF16, const LinearLine<8>& c, int e, float a, float) {
    return __builtin_bit_cast(float, e % 2 ? c.w[e / 2] & 0xffff0000u : c.w[e / 2] << 16) + a;
}

// L lanes have a row, NC chunks of eight consecutive values each: chunk i of lane l is the row's chunk L i + l, and C > 8 L (NC - 1),
// so that only a lane's last chunk may be missing.
// Every form adds up in the same order, so that a row's bits do not depend on how many rows there are: that of 64 lanes with
// chunks l, l + 64, ..., one partial sum a lane, then pairs of lanes 8, 4, 2, 1, 16 and 32 apart.  A lane that stands for
// several of the 64 has a partial sum for each (part).
// Few rows are a chain of latencies (launch, row, two reductions, store), shortest with the row spread over many lanes.  Many are
// bound by memory if a row costs few instructions: no idle lanes in a wavefront, several rows sharing the divisions and the
// root, fp16 values converted by the fma that uses them, and buffer loads and stores, which need no branch for a chunk or a row that is
// not there.  Beyond kLnWaves wavefronts a lane takes every stride-th row, and gamma and beta stay for all of them.
// us, operands from HBM, one wavefront and four chunks a lane to every row / now: 25 216 x 768 fp16 19.1 / 16.3, bf16 19.3 / 16.2;
// 8850 x 768 9.0 / 7.7; 25 216 x 384 14.7 / 10.7; 25 216 x 192 11.3 / 6.3; 12 608 x 1000 14.2 / 12.5; 12 608 x 2048 23.0 / 21.5;
// 394 rows of 768, 384, 192: 2.49, 2.25, 2.23 / 2.21, 2.06, 2.05.
constexpr int kLnWaves = 32768;                                // about four times what the chip holds: 50 432 x 768 31.2 us with half of it, 29.3 now
// More lanes a row up to this capacity.  It is the row count that decides, but only the device knows it: with room for 4000 rows, of
// which 10 / 33 / 100 % are there, bf16, many lanes take 2.25 / 2.93 / 4.40 us and few 2.48 / 2.77 / 4.37 at 768, 2.06 / 2.33 / 3.34 and
// 2.42 / 2.56 / 3.12 at 384; over 10 to 100 % many win by 1 to 4 % up to room for 5000 and few by as much from 8000 on.
constexpr int kLnFewRows = 5000;
template <typename In, int L, int NC>
__global__ __launch_bounds__(kBlockThreads)
void layernorm_kernel(const uint16_t* x, const uint16_t* __restrict__ gamma,          // y may be x: no restrict
                      const uint16_t* __restrict__ beta, uint16_t* y, int rows_cap,
                      const int32_t* __restrict__ rows_dev, int C, float eps, int64_t stride) {
    typedef LinearLine<8> Chunk;
    constexpr int kRows = kWaveSize / L;                       // rows of a wavefront at a time
    constexpr int kParts = kRows < NC ? kRows : NC;
    static_assert(kParts <= 3, "of four partial sums the second pair would be added up first");
    int given = rows_cap;
    if (rows_dev) { const int r = *rows_dev; given = r < given ? r : given; }
    const int rows = __builtin_amdgcn_readfirstlane(given);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int lane = threadIdx.x & (kWaveSize - 1), sub = lane % L;
    int64_t row = ((int64_t)blockIdx.x * (kBlockThreads / kWaveSize) + wave) * kRows;
    if (row >= rows) return;
    const uint32_t row_bytes = (uint32_t)C * 2u;
    const bool last = 8 * (sub + L * (NC - 1)) < C;            // this lane has a last chunk
    // of chunk i, `first` bytes behind its buffer's start; a chunk that is not there lies outside of every buffer
    auto offset = [&](int i, uint32_t first) -> uint32_t { return i < NC - 1 || last ? first + 16u * (sub + L * i) : 1u << 31; };
    auto records = [&]() -> uint32_t { return (uint32_t)(rows - row < kRows ? rows - row : kRows) * row_bytes; };
    const uint32_t lane_row = lane / L * row_bytes;
    auto load = [&](__amdgpu_buffer_rsrc_t rsrc, uint32_t first, Chunk (&c)[NC]) {
#pragma unroll
        for (int i = 0; i < NC; ++i) c[i] = Chunk::load(rsrc, offset(i, first));
    };
    // the first row and what the last pass needs are requested together
    Chunk next[NC], g_raw[NC], b_raw[NC];
    load(buf_rsrc(x + row * C, records()), lane_row, next);
    load(buf_rsrc(gamma, row_bytes), 0, g_raw);
    load(buf_rsrc(beta, row_bytes), 0, b_raw);
    float one = 1.0f;
    asm("" : "+s"(one));
    while (true) {
        const __amdgpu_buffer_rsrc_t y_rsrc = buf_rsrc(y + row * C, records());
        Chunk cur[NC];
        float v[NC][8], part[kParts] = {};
#pragma unroll
        for (int i = 0; i < NC; ++i) {
            cur[i] = next[i];
#pragma unroll
            for (int e = 0; e < 8; ++e) part[i % kParts] = plus_value(In{}, cur[i], e, part[i % kParts], one);
        }
        row += stride;
        const bool more = row < rows;
        if (more) load(buf_rsrc(x + row * C, records()), lane_row, next);
        auto total = [&]() {
            float t = lanes_sum_f32<L>(part[0]);
#pragma unroll
            for (int i = 1; i < kParts; ++i) t += lanes_sum_f32<L>(part[i]);
            return t;
        };
        const float mean = total() / (float)C;
#pragma unroll
        for (int i = 0; i < kParts; ++i) part[i] = 0.f;
#pragma unroll
        for (int i = 0; i < NC; ++i) {
            const float centre = i < NC - 1 || last ? -mean : 0.f;
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                v[i][e] = plus_value(In{}, cur[i], e, centre, one);
                part[i % kParts] = __builtin_fmaf(v[i][e], v[i][e], part[i % kParts]);
            }
        }
        const float rstd = 1.0f / sqrtf(total() / (float)C + eps);
#pragma unroll
        for (int i = 0; i < NC; ++i) {
            float gm[8], bt[8], out[8];
            // (they stay as they are: converted in front of the loop they would fill twice the registers)
#pragma unroll
            for (int k = 0; k < 4; ++k) asm volatile("" : "+v"(g_raw[i].w[k]), "+v"(b_raw[i].w[k]));
            g_raw[i].unpack(In{}, gm);
            b_raw[i].unpack(In{}, bt);
#pragma unroll
            for (int e = 0; e < 8; ++e) out[e] = __builtin_fmaf(v[i][e] * rstd, gm[e], bt[e]);
            Chunk::pack(In{}, out).store(y_rsrc, offset(i, lane_row));
        }
        if (!more) return;
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
        // the same number of rows for every group of lanes (but for one), as few as kLnWaves wavefronts allow
        const int64_t at_once = (int64_t)kLnWaves * (kWaveSize / lanes), each = (rows_cap + at_once - 1) / at_once;
        const int per = kBlockThreads / lanes, groups = (int)(((rows_cap + each - 1) / each + per - 1) / per);
        return launch_kernel(kernel, dim3(groups), dim3(kBlockThreads), stream, static_cast<const uint16_t*>(x),
                             static_cast<const uint16_t*>(gamma), static_cast<const uint16_t*>(beta), static_cast<uint16_t*>(y),
                             rows_cap, rows_dev, C, eps, (int64_t)groups * per);
    };
    auto typed = [&](auto in) {
        typedef decltype(in) In;
#define LN_FORM(L, NC) if (C <= 8 * L * NC) return launch(layernorm_kernel<In, L, NC>, L);
        LN_FORM(16, 1)
        if (rows_cap <= kLnFewRows) {
            LN_FORM(32, 1) LN_FORM(64, 1)
        } else {
            LN_FORM(16, 2) LN_FORM(16, 3) LN_FORM(32, 2) LN_FORM(32, 3)
        }
        LN_FORM(64, 2) LN_FORM(64, 3)
        return launch(layernorm_kernel<In, 64, 4>, 64);
#undef LN_FORM
    };
    return dt == RAGGED_F16 ? typed(F16{}) : typed(BF16{});
}

}  // namespace ragged
