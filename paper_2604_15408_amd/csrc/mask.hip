// A keep-mask producer for the pipeline's first stage (Section 4.3 item 2 accepts any method that
// yields a per-token keep mask; Section 5 prunes by a threshold on the l2 norm of the token features
// at a fixed ratio without defining it further).  Two kernels:
//   token_scores_l2_kernel: score[row] = sum_c x[row][c]^2.  8 to 64 lanes per row, fp64
//     accumulation: a square of a 16-bit value is exact in fp64, so for ordinary data the score does
//     not depend on the summation order and ranking decisions agree with any other exact evaluation.
//   keep_topk_kernel: per image, token 0 (the class token) is kept and, of the others, the k-1 with
//     the largest score (equal scores: lower position first).  Scores of the image in LDS, an O(N)
//     count per token split over eight lanes -- N is a few hundred.
#include "common.h"
#include "mfma_lds.h"

namespace ragged {
namespace {

constexpr int kMaxMaskTokens = 1536;

// L lanes share a row, lane l holds its 16-byte chunks l, L + l, ... (NC of them, all requested before any is used; NC 0: as many
// as there are, one after the other).  The kernel is bound by memory if enough of it is requested at once: with a whole wavefront
// to every row and a loop over its chunks, a third or more of the lanes had nothing to ask for at C = 768, 384 and 192, and
// every row paid six exchanges of 64-bit sums for itself.  fp16, operands from HBM, us before and now: 50 432 x 768 20.1 and 15.1
// (5.1 TB/s), 50 432 x 384 13.2 and 8.5, 50 432 x 192 10.6 and 5.3, 12 608 x 768 6.2 and 5.3, 394 rows of either 2.8 and 2.8.
// (With several rows to a group of lanes, the next on its way: the same up to 384, 50 432 x 768 15.7 to 16.8.)
template <typename V8, int L, int NC>
__global__ __launch_bounds__(kBlockThreads)
void token_scores_l2_kernel(const uint4* __restrict__ x, int64_t rows, int chunks, double* __restrict__ scores) {
    const int sub = threadIdx.x % L;
    const int64_t row = (int64_t)blockIdx.x * (kBlockThreads / L) + threadIdx.x / L;
    if (row >= rows) return;
    const uint4* src = x + row * (NC > 0 ? L * NC : chunks);
    double acc = 0.0;
    auto add = [&](const uint4& raw) {
        const V8 v = as_vec8<V8>(raw);
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const double d = (double)(float)v[e];
            acc = __builtin_fma(d, d, acc);
        }
    };
    if (NC > 0) {
        uint4 raw[NC > 0 ? NC : 1];
#pragma unroll
        for (int i = 0; i < NC; ++i) raw[i] = src[L * i + sub];
#pragma unroll
        for (int i = 0; i < NC; ++i) add(raw[i]);
    } else {
        for (int c = sub; c < chunks; c += L) add(src[c]);
    }
#pragma unroll
    for (int off = L / 2; off >= 1; off >>= 1) acc += __shfl_xor(acc, off, kWaveSize);
    if (sub == 0) scores[row] = acc;
}

// One work-group per (image, 32 tokens): eight lanes share a token and split the range of rivals
// u = 1 .. N-1 between them (u = 1 + part, 9 + part, ...), so the counting loop is an eighth as long and
// the image's scores are read from LDS; the eight partial counts meet in a three-step reduction.
// The loop is bound by its 64-bit compares: rivals in front of the token are counted where they are not smaller, those behind
// it (and itself) where they are larger, one compare each instead of two and a position test.
constexpr int kTopkLanes = 8;
constexpr int kTopkTokens = kBlockThreads / kTopkLanes;

__global__ __launch_bounds__(kBlockThreads)
void keep_topk_kernel(const double* __restrict__ scores, int N, int k, int chunks, uint8_t* __restrict__ keep) {
    __shared__ double s[kMaxMaskTokens];
    const int img = blockIdx.x / chunks;
    const int t = (blockIdx.x - img * chunks) * kTopkTokens + threadIdx.x / kTopkLanes;
    const int part = threadIdx.x % kTopkLanes;
    const double* mine = scores + (int64_t)img * N;
    for (int u = threadIdx.x; u < N; u += kBlockThreads) s[u] = mine[u];
    __syncthreads();
    const double st = s[t < N ? t : 0];
    int before = 0, u = 1 + part;
#pragma unroll 4
    for (; u < t && u < N; u += kTopkLanes) before += s[u] >= st ? 1 : 0;
#pragma unroll 4
    for (; u < N; u += kTopkLanes) before += s[u] > st ? 1 : 0;
    before += __shfl_xor(before, 1, kWaveSize);
    before += __shfl_xor(before, 2, kWaveSize);
    before += __shfl_xor(before, 4, kWaveSize);
    if (part == 0 && t < N) keep[(int64_t)img * N + t] = (uint8_t)((t == 0 || before < k - 1) ? 1 : 0);
}

}  // namespace

int keep_topk_max_tokens() { return kMaxMaskTokens; }

hipError_t launch_token_scores_l2(const void* x, int64_t rows, int C, ragged_dtype dt, double* scores,
                                  hipStream_t stream) {
    auto launch = [&](auto kernel, int lanes) {
        const int per = kBlockThreads / lanes;
        return launch_kernel(kernel, dim3((unsigned)((rows + per - 1) / per)), dim3(kBlockThreads), stream,
                             static_cast<const uint4*>(x), rows, C / 8, scores);
    };
    auto typed = [&](auto vec) {
        typedef decltype(vec) V8;
        // widths that 8 to 64 lanes share out in two or three chunks each
#define SCORES_FULL(L, NC) if (C == 8 * L * NC) return launch(token_scores_l2_kernel<V8, L, NC>, L);
        SCORES_FULL(8, 3) SCORES_FULL(16, 3) SCORES_FULL(32, 2) SCORES_FULL(32, 3) SCORES_FULL(64, 2)
#undef SCORES_FULL
        return launch(token_scores_l2_kernel<V8, 64, 0>, 64);
    };
    return dt == RAGGED_F16 ? typed(f16x8{}) : typed(bf16x8{});
}

hipError_t launch_keep_topk(const double* scores, int B, int N, int k, uint8_t* keep, hipStream_t stream) {
    const int chunks = (N + kTopkTokens - 1) / kTopkTokens;
    const hipError_t err = launch_kernel(keep_topk_kernel, dim3(B * chunks), dim3(kBlockThreads), stream, scores, N, k, chunks, keep);
    return err;
}

}  // namespace ragged
