// linear_kernel: y[m][n] = act( sum_k x[m][k] * w[n][k] + bias[n] ) (+ residual[m][n]) over packed rows, on MFMA
// (internal; the rule that picks a tile shape and the walk over the tiles are in linear_walk.h, one source per input type
// instantiates the kernel).
//
// x [rows, K], w [N, K]: both operands are contiguous along k, which is how an MFMA lane wants them (8 consecutive k per
// 16-byte read).  x is the A operand, so a lane ends up with four rows of a column, and column c of feature tile j stands for
// feature NJ c + j of the wavefront's 16 NJ: a lane then has NJ consecutive features of a row, and 16 neighbouring lanes have
// all of them.  With 128 features a store (or load of the residual) writes four rows of two whole cache lines.  What counts is
// that a quarter of a wavefront, which is what the address unit takes at a time, falls into two lines: with the four lanes of
// a token 16 lanes apart (the product formed the other way round) it fell into sixteen, and a 16-byte store took 230 cycles of
// its wavefront instead of about 90 (epilogue of a 256 x 192 tile 7600 -> 4000 of 31 000 cycles; 8850 x 2304 x 768 34.6 -> 31.1 us,
// 25 216 x 768 x 768 with residual 37.1 -> 34.5, 817 x 768 x 3072 13.4 -> 12.3).  The order of the features costs nothing: the rows of
// w are put in that order where they are loaded into LDS.  A lane's bias is NJ values for all its rows, not four times as many.
//
// A work-group has four wavefronts, one on each SIMD of a CU, each owning 16 NJ features x 16 MT tokens.  With a CU to itself
// (PER_CU 1) a wavefront has the whole register file and holds up to 128 x 128 accumulators, and LDS traffic per product is
// half of that of eight wavefronts of 64 x 128, which kept the LDS pipe busy as long as the matrix core (25 216 rows, us of
// eight and of four when they took their place: 2304 x 768 102 and 86, 768 x 3072 144 and 102).  Its epilogue runs beside nothing,
// though.  With PER_CU 2 two groups of up to 192 x 128 share the CU and one's epilogue runs beside the other's products, which is the
// faster form where the contraction is short or the epilogue has GELU (12 608 x 1536 x 384 with GELU 30.4 us alone and 25.6 in
// pairs, 25 216 x 3072 x 768 with GELU 145 and 119); linear_walk.h has the rule.  By the counters (fp16, no GELU, us and share of
// the cycles with the matrix core busy): 25 216 x 3072 x 768 in 256 x 256 106 and 0.53, 12 608 x 2304 x 768 in pairs of 192 x 128 43 and
// 0.45, 12 608 x 768 x 3072 49 and 0.51, where a loop of products alone on this chip sustains 0.50 to 0.56 of its rate; few
// rows are bound by the time of a step (LDS round trip, barrier) and by launch and first loads (1334 x 768 x 3072 13.5 and
// 0.13, waiting 37 % of the time).
//
// With a single wavefront on a SIMD nothing else fills the gap an instruction leaves, so the loop is laid out by issue slots:
// one instruction between two MFMAs is free, a second independent VALU too, anything more (or an address computed in front of
// an LDS read) delays the next product.  So fragment reads have their addresses ready (immediate offsets; the four registers
// move from stage to stage in slots of their own), a load's M0 set-up and the load sit on the two sides of a product, and
// everything is spread evenly.  The products are inline assembly: accumulators stay where they are, and the order is kept.
// Up to 192 features a tile (NJ <= 6) they are ordinary registers, which the epilogue reads as they are; the 256-wide tiles
// have them in the accumulation registers and copy each once.
//
// Operand tiles (rows x 64 k = 128-byte rows) are brought into LDS by direct loads, row-major with the chunk swizzle
// c ^ ((row>>1)&3) that spreads every 16-byte fragment read over all banks (8 cycles of the LDS pipe for 64 lanes), in a ring
// of as many stages as fit 160 KB (PER_CU 2: half of it).
// A step is two halves of 32 k; fragments of the next half are read while the products of this one run:
//   * more than two stages: one barrier per step, between the halves.  The ring is refilled half a step at a time (w with
//     the first half, x with the second);
//   * two stages (256 x 192 and more, and the pairs of 192 x 128, 192 x 96 and 128 x 128): x of both halves is held a step ahead, which
//     frees the x part of a stage at the start of its step and the w part in the middle, so that its loads spread over the
//     whole step as well (issued in one half they queue up: 4 x 16 KB at 64 bytes a cycle).
// The tiles of a work-group follow each other without a break: the last steps of one load the first of the next.
//
// Epilogue in registers: bias, GELU, residual, one rounding, stores of a row group as soon as it is done.  The residual (a
// kernel of its own: its registers are there for nothing else) is requested with the products of the last step but one:
// 817 x 768 x 3072 13.1 -> 12.3 us, 817 x 768 x 768 5.8 -> 5.7, nothing for many rows.
#pragma once

#include <type_traits>

#include "common.h"
#include "linear_epilogue.h"
#include "linear_walk.h"
#include "mfma_lds.h"

namespace ragged {

typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
typedef unsigned u32x3 __attribute__((ext_vector_type(3)));
typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
__device__ f16x2 vec2_of(F16);
__device__ bf16x2 vec2_of(BF16);

constexpr int kLinWaves = 4;                     // one wavefront per SIMD
static_assert(kLinearXcds == kXcds, "tiles are dealt out per XCD");

struct LinearArgs {
    const uint16_t* x;
    const uint16_t* w;
    const uint16_t* bias;
    const uint16_t* res;                         // may alias y
    uint16_t* y;
    const int32_t* rows_dev;
    int rows_cap, N, K, act;
    int n_tiles;                                 // N / (32 NJ)
    int panel;                                   // feature tiles of a panel, see LinearWalk
    uint32_t panel_magic, last_magic;            // div_magic() of panel and of the last panel's width
};

// N consecutive 16-bit values of a row, as stored.
template <int N>
struct alignas(N == 8 ? 16 : N == 4 ? 8 : 4) LinearLine {
    uint32_t w[N / 2];
    __device__ __forceinline__ void unpack(F16, float (&v)[N]) const {
#pragma unroll
        for (int e = 0; e < N; ++e) v[e] = (float)__builtin_bit_cast(_Float16, (uint16_t)(w[e / 2] >> 16 * (e % 2)));
    }
    __device__ __forceinline__ void unpack(BF16, float (&v)[N]) const {
#pragma unroll
        for (int e = 0; e < N; ++e) v[e] = __builtin_bit_cast(float, e % 2 ? w[e / 2] & 0xffff0000u : w[e / 2] << 16);
    }
    template <typename In>
    static __device__ __forceinline__ LinearLine pack(In, const float (&v)[N]) {
        typedef decltype(vec2_of(In{})) vec2;
        LinearLine l;
#pragma unroll
        for (int e = 0; e < N / 2; ++e) {
            vec2 h;
            h[0] = (decltype(h[0] + h[0]))v[2 * e];
            h[1] = (decltype(h[0] + h[0]))v[2 * e + 1];
            l.w[e] = __builtin_bit_cast(uint32_t, h);
        }
        return l;
    }
    __device__ __forceinline__ void store(__amdgpu_buffer_rsrc_t rsrc, uint32_t voff) const {
        if constexpr (N == 8) __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, *this), rsrc, voff, 0, 0);
        else if constexpr (N == 6) __builtin_amdgcn_raw_buffer_store_b96(u32x3{w[0], w[1], w[2]}, rsrc, voff, 0, 0);
        else if constexpr (N == 4) __builtin_amdgcn_raw_buffer_store_b64(u32x2{w[0], w[1]}, rsrc, voff, 0, 0);
        else __builtin_amdgcn_raw_buffer_store_b32(w[0], rsrc, voff, 0, 0);
    }
    static __device__ __forceinline__ LinearLine load(__amdgpu_buffer_rsrc_t rsrc, uint32_t voff) {
        LinearLine l;
        if constexpr (N == 8) { const u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(rsrc, voff, 0, 0); l.w[0] = v[0]; l.w[1] = v[1]; l.w[2] = v[2]; l.w[3] = v[3]; }
        else if constexpr (N == 6) { const u32x3 v = __builtin_amdgcn_raw_buffer_load_b96(rsrc, voff, 0, 0); l.w[0] = v[0]; l.w[1] = v[1]; l.w[2] = v[2]; }
        else if constexpr (N == 4) { const u32x2 v = __builtin_amdgcn_raw_buffer_load_b64(rsrc, voff, 0, 0); l.w[0] = v[0]; l.w[1] = v[1]; }
        else l.w[0] = __builtin_amdgcn_raw_buffer_load_b32(rsrc, voff, 0, 0);
        return l;
    }
};

#define RAGGED_INLINE_LAMBDA __attribute__((always_inline))

// acc += A B (FIRST: acc = A B), the accumulator in the ordinary registers (ACC_V) or in the accumulation registers.
#define MFMA_TEXT(dt) "v_mfma_f32_16x16x32_" dt " %0, %1, %2, "
#define MFMA_ASM(dt, head, tail, eq, ...) \
    do { \
        if (FIRST && ACC_V) asm volatile(head MFMA_TEXT(dt) "0" tail : eq "v"(acc) : "v"(a), "v"(b) __VA_ARGS__); \
        else if (FIRST) asm volatile(head MFMA_TEXT(dt) "0" tail : eq "a"(acc) : "v"(a), "v"(b) __VA_ARGS__); \
        else if (ACC_V) asm volatile(head MFMA_TEXT(dt) "%0" tail : "+v"(acc) : "v"(a), "v"(b) __VA_ARGS__); \
        else asm volatile(head MFMA_TEXT(dt) "%0" tail : "+a"(acc) : "v"(a), "v"(b) __VA_ARGS__); \
    } while (0)
template <bool FIRST, bool ACC_V>
__device__ __forceinline__ void mma_acc(F16, const u32x4& a, const u32x4& b, f32x4& acc) { MFMA_ASM("f16", "", "", "="); }
template <bool FIRST, bool ACC_V>
__device__ __forceinline__ void mma_acc(BF16, const u32x4& a, const u32x4& b, f32x4& acc) { MFMA_ASM("bf16", "", "", "="); }
// The same with one global->LDS load: lane i fetches the 16 bytes at rsrc.base + voff + soff (zeros past
// rsrc.num_records) and the hardware stores them at LDS address dst + off + 16*i.  Its two instructions sit in front of
// and behind the product, one issue slot each.
#define DMA_HEAD "s_add_u32 m0, %3, %4\n\t"
#define DMA_TAIL "\n\tbuffer_load_dwordx4 %5, %6, %7 offen lds"
#define DMA_ARGS , "s"(dst), "i"(off), "v"(voff), "s"(rsrc), "s"(soff) : "memory", "m0", "scc"
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
template <bool FIRST, bool ACC_V>
__device__ __forceinline__ void mma_acc_dma(F16, const u32x4& a, const u32x4& b, f32x4& acc, uint32_t dst, uint32_t off,
                                            uint32_t voff, const u32x4& rsrc, uint32_t soff) {
    MFMA_ASM("f16", DMA_HEAD, DMA_TAIL, "=&", DMA_ARGS);
}
template <bool FIRST, bool ACC_V>
__device__ __forceinline__ void mma_acc_dma(BF16, const u32x4& a, const u32x4& b, f32x4& acc, uint32_t dst, uint32_t off,
                                            uint32_t voff, const u32x4& rsrc, uint32_t soff) {
    MFMA_ASM("bf16", DMA_HEAD, DMA_TAIL, "=&", DMA_ARGS);
}
__device__ __forceinline__ void buf_dma16(uint32_t dst, uint32_t voff, const u32x4& rsrc, uint32_t soff) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds"
                 :: "s"(dst), "v"(voff), "s"(rsrc), "s"(soff) : "memory", "m0");
}
#pragma clang diagnostic pop

__device__ __forceinline__ float read_acc(float a) {
    float v;
    asm volatile("v_accvgpr_read_b32 %0, %1" : "=v"(v) : "a"(a));
    return v;
}
__device__ __forceinline__ u32x4 lds_vec(uint32_t addr) {
    return *reinterpret_cast<const lds_u32x4*>(static_cast<uintptr_t>(addr));
}

// The bytes from base on, `bytes` of them: a load past them gives zeros, a store is dropped.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t buf_rsrc(const void* base, uint32_t bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), 0, (int)bytes, 0x00020000);
}
// The m-th product's position in rows of n: rows are walked to and fro, so that one operand of two stays from each
// product to the next (the matrix core then draws less power, which is what limits the clock in these kernels).
constexpr int snake(int m, int n) { return (m / n) % 2 ? n - 1 - m % n : m % n; }
// Which of `count` things spread evenly over `slots` issue slots goes with slot s (-1: none).
constexpr int spread_at(int s, int slots, int count) {
    for (int d = 0; d < count; ++d)
        if ((2 * d + 1) * slots / (2 * count) == s) return d;
    return -1;
}

template <typename In, int NJ, int MT, int PER_CU, bool RES, bool WIDE>
__global__ __launch_bounds__(kWaveSize * kLinWaves, PER_CU)
void linear_kernel(const int32_t* rows_ptr, int rows_cap, int n_tiles, const uint16_t* x, const uint16_t* w, int K_, int panel,
                   uint32_t panel_magic, uint32_t last_magic, const uint16_t* bias, const uint16_t* res, uint16_t* y, int N_,
                   int act) {
    // WIDE: rows of more than 2^22 features, whose outputs 32-bit offsets do not reach.
    // What the first loads need comes first: 14 dwords of arguments arrive in scalar registers with the wavefront (a struct
    // would not), which saves a few hundred rows 0.1 to 0.3 us a launch (817 x 768 x 3072 13.4 -> 13.1, 1334 x 768 x 768
    // 6.4 -> 6.2) and large launches nothing.
    const LinearArgs p{x, w, bias, res, y, rows_ptr, rows_cap, N_, K_, act, n_tiles, panel, panel_magic, last_magic};
    typedef LinearShape<NJ, MT, PER_CU> Shape;
    constexpr int TN = Shape::TN, TM = Shape::TM;              // features x tokens of a tile, 2 x 2 wavefronts
    constexpr int kXBytes = TM * kTK * 2, kWBytes = TN * kTK * 2;
    constexpr int kStageBytes = kXBytes + kWBytes;
    constexpr int STAGES = Shape::kStages;
    constexpr bool TWO = Shape::kTwo, RELAX = Shape::kRelax;
    constexpr int kAheadX = Shape::kAheadX, kAheadW = Shape::kAheadW;
    __shared__ __attribute__((aligned(1024))) uint4 stage_lds[STAGES * kStageBytes / 16];

    const int N = p.N;
    int given = p.rows_cap;
    if (p.rows_dev) { const int r = *p.rows_dev; given = r < given ? r : given; }
    const LinearWalk walk(__builtin_amdgcn_readfirstlane(given), TM, p.n_tiles, p.panel, p.panel_magic, p.last_magic, blockIdx.x, gridDim.x);
    const int rows = walk.rows, t_first = walk.t_first, t_end = walk.t_end, stride = walk.stride;
    if (t_first >= t_end) return;

    const int tid = threadIdx.x;
    const int lane = tid & (kWaveSize - 1);
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int col = lane & 15;
    const int g = lane >> 4;
    const int wn = wave & 1, wm = wave >> 1;

    // ---- loads.  Instruction d of this wavefront covers rows 8*(count*wave + d) + lane/8 of its operand tile; the
    // lane's LDS slot is position lane%8 of that row = chunk (lane%8) ^ ((row>>1)&3).
    constexpr int kXI = MT, kWI = NJ;                          // load instructions per wavefront and step
    const uint32_t lds0 = (uint32_t)reinterpret_cast<uintptr_t>((__attribute__((address_space(3))) void*)stage_lds);
    const uint32_t row_bytes = (uint32_t)p.K * 2u;
    const uint32_t chunk = 16u * ((lane & 7) ^ ((lane >> 4) & 3));
    const int ksteps = p.K / kTK;
    uint32_t voff_x[kXI], voff_w[kWI];
#pragma unroll
    for (int i = 0; i < kXI; ++i) voff_x[i] = (uint32_t)(8 * (kXI * wave + i) + (lane >> 3)) * row_bytes + chunk;
#pragma unroll
    for (int i = 0; i < kWI; ++i) {
        const int p_row = 8 * (kWI * wave + i) + (lane >> 3), in_wave = p_row % (16 * NJ);       // LDS row: feature tile in_wave / 16, column in_wave % 16
        voff_w[i] = (uint32_t)(p_row - in_wave + NJ * (in_wave & 15) + (in_wave >> 4)) * row_bytes + chunk;
    }
    const uint32_t x_dst = kXI * 1024 * wave, w_dst = kXBytes + kWI * 1024 * wave;

    // Two cursors walk (tile, step) ahead of the arithmetic.  Rows past the end of x and everything past the last tile are
    // out of range: such loads touch no memory (see LinearCursor) and arrive as zeros (their results are not stored).
    u32x4 x_rsrc, w_rsrc;
    LinearCursor x_cur, w_cur;
    x_cur.tile = w_cur.tile = t_first;
    auto set_rsrc = [&](u32x4& r, const uint16_t* base, uint32_t bytes) RAGGED_INLINE_LAMBDA {
        const uint64_t a = reinterpret_cast<uint64_t>(base);
        r[0] = __builtin_amdgcn_readfirstlane((uint32_t)a);
        r[1] = __builtin_amdgcn_readfirstlane((uint32_t)(a >> 32));
        r[2] = __builtin_amdgcn_readfirstlane(bytes);
        r[3] = 0x00020000u;
    };
    auto set_x = [&]() RAGGED_INLINE_LAMBDA { set_rsrc(x_rsrc, p.x + (int64_t)x_cur.first * p.K, x_cur.bytes); };
    auto set_w = [&]() RAGGED_INLINE_LAMBDA { set_rsrc(w_rsrc, p.w + (int64_t)w_cur.first * p.K, w_cur.bytes); };
    auto next_x = [&]() RAGGED_INLINE_LAMBDA { if (x_cur.next<TM, TN, true>(walk, row_bytes)) set_x(); };
    auto next_w = [&]() RAGGED_INLINE_LAMBDA { if (w_cur.next<TM, TN, false>(walk, row_bytes)) set_w(); };

    // ---- LDS addresses of this lane's operands: x (A operand) row 16 mt + col, w (B operand) row 16 j + col; chunk 2g + half
    const int x_row = wm * 16 * MT + col, w_row = wn * 16 * NJ + col;
    uint32_t rb[2], ra[2];                                     // [half]
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        rb[h] = lds0 + x_row * 128 + 16 * ((2 * g + h) ^ ((x_row >> 1) & 3));
        ra[h] = lds0 + kXBytes + w_row * 128 + 16 * ((2 * g + h) ^ ((w_row >> 1) & 3));
    }
    constexpr bool ACC_V = NJ < 8;                             // there is room for them beside everything else
    f32x4 acc[NJ][MT];
    u32x4 a0[NJ], b0[MT], a1[NJ], b1[MT];
    auto read_a = [&](int h, int j) RAGGED_INLINE_LAMBDA { return lds_vec(ra[h] + j * 2048); };
    auto read_b = [&](int h, int mt) RAGGED_INLINE_LAMBDA { return lds_vec(rb[h] + mt * 2048); };

    constexpr int NS = NJ * MT;                                // products of half a step = issue slots
    static_assert(!TWO || NS >= 16, "the slots before the barrier of a half hold the address updates of two-stage rings");
    // ---- residual: its first kAhead 16-row groups are requested with the first half of the last step but one (all of them where
    // there are registers for it)
    typedef LinearLine<NJ> Line;                               // NJ consecutive outputs of a row
    constexpr int kMost = NJ == 8 && MT == 8 ? 2 : NJ == 8 && MT == 7 ? 4 : NJ == 6 && MT * PER_CU == 8 ? 1 : MT;
    constexpr int kAhead = RES ? kMost : 1;
    Line r_raw[kAhead][4];
    __amdgpu_buffer_rsrc_t r_rsrc = buf_rsrc(p.res, 0);
    const uint32_t out_row = (uint32_t)N * 2u;
    uint32_t out_voff = (uint32_t)(wm * 16 * MT + 4 * g) * out_row + (uint32_t)(wn * 16 * NJ + NJ * col) * 2u;
    auto load_res = [&](int row) RAGGED_INLINE_LAMBDA {        // row 4 mt + r of this lane
        r_raw[row / 4 % kAhead][row % 4] = Line::load(r_rsrc, out_voff + (16 * (row / 4) + row % 4) * out_row);
    };

    // ---- first half of a step: products of (a0, b0)
    auto half_a = [&](auto first_tag, auto res_tag, uint32_t fill, uint32_t delta) RAGGED_INLINE_LAMBDA {
        constexpr bool FIRST = decltype(first_tag)::value;
        constexpr int kResLoads = decltype(res_tag)::value ? 4 * kAhead : 0;
        constexpr int kSync = TWO ? NS / 8 : 0, kLeft = NS - kSync;
#pragma unroll
        for (int m = 0; m < kSync; ++m) {
            if (m == 1) rb[1] += delta;
            __builtin_amdgcn_sched_barrier(0);
            mma_acc<FIRST, ACC_V>(In{}, b0[snake(m, MT)], a0[m / MT], acc[m / MT][snake(m, MT)]);
            __builtin_amdgcn_sched_barrier(0);
        }
        if (TWO) {
            __builtin_amdgcn_s_waitcnt(0xC07F);                // lgkmcnt(0)
            __syncthreads();
        }
        constexpr int kLoads = TWO ? kXI : kWI;
        constexpr int kReads = TWO ? NJ : NJ + MT;
#pragma unroll
        for (int m = kSync; m < NS; ++m) {
            const int q = m - kSync;
#pragma unroll
            for (int r = 0; r < kReads; ++r)
                if (r * kLeft * 3 / (4 * kReads) == q) {
                    if (r < NJ) a1[r < NJ ? r : 0] = read_a(1, r);
                    else b1[r - NJ < MT && r >= NJ ? r - NJ : 0] = read_b(1, r - NJ);
                }
            if (q == kLeft - 1) ra[0] += delta;
            if (q == (kLeft >= 4 ? kLeft - 3 : kLeft - 1)) rb[0] += delta;
#pragma unroll
            for (int e = 0; e < kResLoads; ++e)
                if ((2 * e + 1) * kLeft / (2 * kResLoads + !kResLoads) == q) load_res(e);
            const int d = spread_at(q, kLeft, kLoads);
            __builtin_amdgcn_sched_barrier(0);
            if (d < 0) mma_acc<FIRST, ACC_V>(In{}, b0[snake(m, MT)], a0[m / MT], acc[m / MT][snake(m, MT)]);
            else if (TWO) mma_acc_dma<FIRST, ACC_V>(In{}, b0[snake(m, MT)], a0[m / MT], acc[m / MT][snake(m, MT)], fill + x_dst, d * 1024, voff_x[d < kXI ? d : 0], x_rsrc, x_cur.soff);
            else mma_acc_dma<FIRST, ACC_V>(In{}, b0[snake(m, MT)], a0[m / MT], acc[m / MT][snake(m, MT)], fill + w_dst, d * 1024, voff_w[d < kWI ? d : 0], w_rsrc, w_cur.soff);
            __builtin_amdgcn_sched_barrier(0);
        }
        if (TWO) next_x();
        else next_w();
    };
    // ---- second half: products of (a1, b1); fragments of the next step
    auto half_b = [&](uint32_t fill, uint32_t delta) RAGGED_INLINE_LAMBDA {
        constexpr int kReads = NJ + MT;
#pragma unroll
        for (int m = 0; m < NS; ++m) {
#pragma unroll
            for (int r = 0; r < kReads; ++r)
                if ((TWO ? 2 * r : r * NS * 3 / (4 * kReads)) == m) {
                    if (r < NJ) a0[r < NJ ? r : 0] = read_a(0, r);
                    else b0[r - NJ < MT && r >= NJ ? r - NJ : 0] = read_b(0, r - NJ);
                }
            if (TWO && m % NJ == 1 && m > NJ) b1[m / NJ - 1] = read_b(1, m / NJ - 1);
            if (m == NS - 1) ra[1] += delta;
            if (!TWO && m == (NS >= 4 ? NS - 3 : NS - 1)) rb[1] += delta;
            const int d = spread_at(m, NS, TWO ? kWI : kXI);
            __builtin_amdgcn_sched_barrier(0);
            if (d < 0) mma_acc<false, ACC_V>(In{}, b1[m / NJ], a1[snake(m, NJ)], acc[snake(m, NJ)][m / NJ]);
            else if (TWO) mma_acc_dma<false, ACC_V>(In{}, b1[m / NJ], a1[snake(m, NJ)], acc[snake(m, NJ)][m / NJ], fill + w_dst, d * 1024, voff_w[d < kWI ? d : 0], w_rsrc, w_cur.soff);
            else mma_acc_dma<false, ACC_V>(In{}, b1[m / NJ], a1[snake(m, NJ)], acc[snake(m, NJ)][m / NJ], fill + x_dst, d * 1024, voff_x[d < kXI ? d : 0], x_rsrc, x_cur.soff);
            __builtin_amdgcn_sched_barrier(0);
        }
        if (TWO) {
            b1[MT - 1] = read_b(1, MT - 1);
            __builtin_amdgcn_sched_barrier(0);
            next_w();
        } else {
            next_x();
        }
    };

    int m0, n0;                                                // the tile being computed
    Line bias_raw{};
    auto load_bias = [&]() RAGGED_INLINE_LAMBDA {
        if (p.bias) bias_raw = *reinterpret_cast<const Line*>(p.bias + n0 + wn * 16 * NJ + NJ * col);
    };
    x_cur.set<TM, TN, true>(walk, row_bytes);
    set_x();
    w_cur.set<TM, TN, false>(walk, row_bytes);
    set_w();
    {
        constexpr int kFillX = TWO ? 2 : kAheadX, kFillW = TWO ? 2 : kAheadW;
#pragma unroll
        for (int st = 0; st < kFillX; ++st) {
#pragma unroll
            for (int d = 0; d < kXI; ++d) buf_dma16(lds0 + st * kStageBytes + x_dst + d * 1024, voff_x[d], x_rsrc, x_cur.soff);
            next_x();
            if (st < kFillW) {
#pragma unroll
                for (int d = 0; d < kWI; ++d) buf_dma16(lds0 + st * kStageBytes + w_dst + d * 1024, voff_w[d], w_rsrc, w_cur.soff);
                next_w();
            }
        }
        wait_vm<(kFillX - 1) * kXI + (kFillW - 1) * kWI>();    // step 0 has landed
    }
    walk.tile_of(t_first, TM, TN, m0, n0);
    load_bias();
    __syncthreads();
#pragma unroll
    for (int j = 0; j < NJ; ++j) a0[j] = read_a(0, j);
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) b0[mt] = read_b(0, mt);
    if (TWO)
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) b1[mt] = read_b(1, mt);

    // stage numbers: s of the current step, s_next of the next, fill_a / fill_b the ones that half A / B load into
    auto wrap = [&](uint32_t s) RAGGED_INLINE_LAMBDA { return s == lds0 + (STAGES - 1) * kStageBytes ? lds0 : s + kStageBytes; };
    uint32_t s = lds0;
    uint32_t fill_a = TWO ? lds0 : lds0 + kAheadW * kStageBytes;
    uint32_t fill_b = TWO ? lds0 : lds0 + (kAheadX % STAGES) * kStageBytes;
    bool landed = false;
    auto step = [&](auto first_tag, auto res_tag) RAGGED_INLINE_LAMBDA {
        const uint32_t s_next = wrap(s);
        const uint32_t delta = s_next - s;
        if (TWO) __builtin_amdgcn_s_waitcnt(0xC17F);           // lgkmcnt(1): all but the last fragment
        half_a(first_tag, res_tag, fill_a, delta);
        if (!decltype(first_tag)::value || !landed)            // the next step has landed
            wait_vm<(TWO ? kXI : (kAheadX - 2) * (kXI + kWI)) + (decltype(res_tag)::value ? 4 * kAhead : 0)>();
        if (RELAX) {
            asm volatile("s_barrier" ::: "memory");
        } else {
            __builtin_amdgcn_s_waitcnt(0xC07F);
            __syncthreads();
        }
        half_b(fill_b, delta);
        s = s_next;
        fill_a = wrap(fill_a);
        fill_b = wrap(fill_b);
    };

    const std::true_type yes{};
    const std::false_type no{};
    const bool in_step = RES && !WIDE && ksteps >= 4;
    for (int t = t_first; t < t_end; t += stride) {
        asm volatile("" : "+v"(out_voff));                     // (no register of its own for the offset of every row)
        const int64_t tile_off = (int64_t)m0 * N + n0;
        const uint32_t tile_bytes = WIDE ? 0u : (uint32_t)(rows - m0 < TM ? rows - m0 : TM) * out_row - (uint32_t)n0 * 2u;
        if (RES && !WIDE) r_rsrc = buf_rsrc(p.res + tile_off, tile_bytes);
        step(yes, no);
        int kt = 1;
        for (; kt < (in_step ? ksteps - 2 : ksteps); ++kt) step(no, no);
        if (in_step) {
            step(no, yes);
            step(no, no);
        } else if (RES && !WIDE) {
#pragma unroll
            for (int e = 0; e < 4 * kAhead; ++e) load_res(e);
        }
        // the last products have to leave the matrix core before other instructions may read them
        asm volatile("s_nop 15\n\ts_nop 15" ::: "memory");
        if (ACC_V)
#pragma unroll
            for (int i = 0; i < NJ * MT; ++i) asm volatile("" : "+v"(acc[i / MT][i % MT]));

        // ---- epilogue: this lane owns features n_base + 0 .. NJ-1 of rows m_base + 16 mt + 0 .. 3
        const int m_base = m0 + wm * 16 * MT + 4 * g;
        const __amdgpu_buffer_rsrc_t y_rsrc = buf_rsrc(p.y + tile_off, tile_bytes);
        const int n_base = n0 + wn * 16 * NJ + NJ * col;
        float bias[NJ];
        bias_raw.unpack(In{}, bias);
        if (t + stride < t_end) {
            walk.tile_of(t + stride, TM, TN, m0, n0);
            load_bias();                                       // the next tile's
        }
        auto finish = [&](auto act_tag) RAGGED_INLINE_LAMBDA {
            constexpr bool ACT = decltype(act_tag)::value;
            auto wide_off = [&](int mt, int r) RAGGED_INLINE_LAMBDA -> int64_t {
                const int m = m_base + 16 * mt + r;
                return (int64_t)(m < rows ? m : rows - 1) * N + n_base;
            };
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) {
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    float v[NJ], add[NJ];
                    if (RES) (WIDE ? *reinterpret_cast<const Line*>(p.res + wide_off(mt, r)) : r_raw[mt % kAhead][r]).unpack(In{}, add);
#pragma unroll
                    for (int j = 0; j < NJ; ++j) {
                        float f = (ACC_V ? acc[j][mt][r] : read_acc(acc[j][mt][r])) + bias[j];
                        if (ACT) f = gelu_erf(f);
                        if (RES) f += add[j];
                        v[j] = f;
                    }
                    const Line out = Line::pack(In{}, v);
                    if (mt == 0 && r == 0) wait_vm<0>();       // what the next tile starts with has landed
                    if (!WIDE) out.store(y_rsrc, out_voff + (16 * mt + r) * out_row);
                    else if (m_base + 16 * mt + r < rows) *reinterpret_cast<Line*>(p.y + wide_off(mt, r)) = out;
                    if (RES && !WIDE && mt + kAhead < MT) load_res(4 * (mt + kAhead) + r);
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
        };
        if (p.act) finish(yes);
        else finish(no);
        landed = true;
    }
}

template <typename In>
hipError_t launch_linear_tile(const TileShape& shape, int groups, const LinearArgs& args, hipStream_t stream) {
#define LINEAR_LAUNCH(NJ, MT, PER_CU, WIDE) \
    return launch_kernel(args.res ? linear_kernel<In, NJ, MT, PER_CU, true, WIDE> : linear_kernel<In, NJ, MT, PER_CU, false, WIDE>, \
                         dim3(groups), dim3(kWaveSize * kLinWaves), stream, args.rows_dev, \
                         args.rows_cap, args.n_tiles, args.x, args.w, args.K, args.panel, args.panel_magic, args.last_magic, \
                         args.bias, args.res, args.y, args.N, args.act);
    if (linear_is_wide(args.N)) LINEAR_LAUNCH(2, 1, 1, true)
#define LINEAR_CASE(NJ, MT, PER_CU) \
    if (shape.nj == NJ && shape.mt == MT && shape.per_cu == PER_CU) LINEAR_LAUNCH(NJ, MT, PER_CU, false)
    LINEAR_SHAPES(LINEAR_CASE)
#undef LINEAR_CASE
#undef LINEAR_LAUNCH
    return hipErrorInvalidValue;
}
hipError_t launch_linear_f16(const TileShape& shape, int groups, const LinearArgs& args, hipStream_t stream);
hipError_t launch_linear_bf16(const TileShape& shape, int groups, const LinearArgs& args, hipStream_t stream);

}  // namespace ragged
