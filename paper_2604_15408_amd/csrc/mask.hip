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

// L lanes share a row, lane l holds its 16-byte chunks l, L + l, ... (NC <= 3 of them, the last may be missing, all requested before
// any is used; NC 0: as many as there are, one after the other).  The kernel is bound by memory if enough of it is requested at
// once: with a whole wavefront to every row and a loop over its chunks, a third or more of the lanes had nothing to ask for at
// C = 768, 384 and 192, and every row paid six exchanges of 64-bit sums for itself.  So L is the smallest that covers the row in
// three chunks.  fp16, operands from HBM, us with a wavefront to every row and now: 50 432 x 768 18.7 and 14.2 (5.5 TB/s), x 640 17.5
// and 12.1, x 384 12.6 and 8.2, x 192 9.9 and 4.9, x 64 9.6 and 3.1, 12 608 x 768 5.5 and 4.6, x 1536 8.8 and 7.8, 394 rows of any 2.0
// and 2.0.  (With several rows to a group of lanes, the next on its way: the same up to 384, 50 432 x 768 15.7 to 16.8.)
// The sums are formed in one order for every L, that of a wavefront with chunks l, 64 + l, ... on lane l, so that scores (and
// ties) do not depend on the form: a lane that stands for several of the 64 has a partial sum for each, added up in the order of
// the exchanges 32, 16, 8 that it does without.
template <typename V8, int L, int NC>
__global__ __launch_bounds__(kBlockThreads)
void token_scores_l2_kernel(const uint4* __restrict__ x, int64_t rows, int chunks, double* __restrict__ scores) {
    const int sub = threadIdx.x % L;
    const int64_t row = (int64_t)blockIdx.x * (kBlockThreads / L) + threadIdx.x / L;
    if (row >= rows) return;
    const uint4* src = x + row * chunks;
    auto add = [&](const uint4& raw, double& acc) {
        const V8 v = as_vec8<V8>(raw);
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const double d = (double)(float)v[e];
            acc = __builtin_fma(d, d, acc);
        }
    };
    constexpr int kParts = NC == 0 || L == kWaveSize ? 1 : kWaveSize / L < NC ? kWaveSize / L : NC;
    double part[3] = {0.0, 0.0, 0.0};
    if (NC > 0) {
        uint4 raw[NC > 0 ? NC : 1];
        const bool last = sub + L * (NC - 1) < chunks;
#pragma unroll
        for (int i = 0; i < NC; ++i) raw[i] = src[i < NC - 1 || last ? L * i + sub : 0];
        if (!last) raw[NC > 0 ? NC - 1 : 0] = make_uint4(0u, 0u, 0u, 0u);
#pragma unroll
        for (int i = 0; i < NC; ++i) add(raw[i], part[i % kParts]);
    } else {
        for (int c = sub; c < chunks; c += L) add(src[c], part[0]);
    }
    double acc = part[0];
    if (kParts == 3) acc += part[2];
    if (kParts >= 2) acc += part[1];
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
        const int chunks = C / 8;
#define SCORES_FORM(L, NC) if (chunks <= L * NC) return launch(token_scores_l2_kernel<V8, L, NC>, L);
        SCORES_FORM(8, 1) SCORES_FORM(8, 2) SCORES_FORM(8, 3) SCORES_FORM(16, 2) SCORES_FORM(16, 3)
        SCORES_FORM(32, 2) SCORES_FORM(32, 3) SCORES_FORM(64, 2) SCORES_FORM(64, 3)
#undef SCORES_FORM
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
