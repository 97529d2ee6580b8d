// Convolution as an implicit GEMM on the matrix cores over channels-last tensors (gfx950).
//
// Y[cout x pixels] = W[cout x K] * X~[K x pixels], K = (filter tap, input channel) with the channels of a
// tap contiguous.  In the channels-last layout a K step of a pixel is 64 or 128 contiguous bytes, so
// both operands go from memory straight into LDS with 16-byte `buffer_load ... lds` loads -- no
// register staging, no transposition, no packing -- and each MFMA operand is one 16-byte LDS read.
// The plane (NCHW) layout of the other matrix-core kernel needs 2-byte gathers, a register
// transposition and LDS writes per step, which is what bounds it.
//
//   * LDS rows are RB = 64 or 128 bytes, unpadded (the loads write 16 bytes x lane); the 16-byte pieces of a
//     row are permuted by the row (piece ^ (row / 2) % 8, or (row / 4) % 4 for 64-byte rows), which puts the
//     16 rows a quarter-wave reads into 16 different bank groups.  The permutation is applied to the
//     source addresses of the activations and is baked into the weight plan.
//   * S stage buffers.  A stage's fragments are read into registers one stage ahead of its products and its
//     buffer is loaded again right behind the barrier that follows, between the products: one barrier and
//     one counted wait per stage.
//   * What bounds it is the way into LDS: 50-57 bytes per clock and CU (a kernel of these loads alone, data in L2; 29
//     from behind it), so a 64 x 64 x 64 step of fp16 takes 290 clocks where its products take 128.  Larger tiles reuse more
//     but leave CUs idle.
//   * With one or two workgroups a CU the rest is start and end: 1200 clocks to the first loads and 1500 (with a
//     pass through LDS, which is gone) from the last product to the last store.  So the launch record is fetched whole, the first weights are
//     requested before anything is computed, divisions are multiplications, and bias and residual are
//     requested ahead of the K loop.  ResNet-50 fp16, us per pass before these and the stages above -> behind them:
//     batch 1 371 -> 316, 8 517 -> 427, 32 981 -> 839; MobileNet-V2 fp16 batch 16 490 -> 353.
//     At batch 32 the four matrix pipes of a CU are busy 18 % of the busy CUs' cycles, over all of these launches; L2 hit rate 76 %.
//   * Padding is a zero halo in memory, so no tap is ever tested.
//   * A fused 1x1 projection shortcut (paper Section 4, layer fusion) is more K steps on a second tensor.
//   * The epilogue works on the accumulators where they are: the rows of a block of weights are in an order that leaves a lane
//     16-byte pieces of its pixel's channels, so residual pieces come in and finished ones go out without a pass through LDS (a
//     barrier, a write, a barrier and a read less); bias, residual and ReLU in fp32, one rounding.  The first loads wait for nothing but
//     their own addresses.  fp16 with the pass / without, us: ResNet-50 batch 1 316 / 312, 8 426 / 418, 32 837 / 801 (256 -> 1024 1x1 on
//     14 x 14 14.2 / 11.5), MobileNet-V2 batch 16 352 / 340; results the same to the bit.
//   * fp32 storage: a float scaled by 2^24 is the sum of three bf16, exactly and whatever its size, and a product of two floats is six products of
//     such parts but for 2^-24 of it at the most (2^-28 on average for normally distributed ones).  The bf16 pipes make six in 384 clocks of a 64 x 64 x 32 step, v_mfma_f32_32x32x2_f32
//     the one in 1024.  Weights are laid out as their parts; a wave takes its activations apart in registers, which costs as
//     many clocks as the products and runs beside them.  ResNet-50 fp32 at 8 images 1016 -> 830 us a pass (with two groups
//     of waves and constants of its own).  The products of the leading parts have sums of their own, so that a sum is rounded once for 16 k (all six in
//     one: six times, where fp32 products round once a nonzero, 1.6 to 3 of 16 in a pruned layer).  Against 64 bits, six products with two
//     sums / with one / fp32 products: unpruned K = 576 0.8e-7 / 1.8e-7 / 4.3e-7, 4608 1.4e-7 / 3.7e-7 / 6.1e-7; ResNet-50 of mixed sparsity, the
//     whole net, 1.02e-7 / 1.96e-7 / 1.11e-7.  What bounds a step now (860 to 940 clocks) is the
//     products at the clock they leave the chip (490 for zeros, 610 for random operands and taking apart), then 20 KB into LDS.
//     Sums that are not finite are done again with fp32 products, without overlap: a layer with an infinity in every tile takes two to three
//     times as long (512 -> 512 3x3 on 8 images of 14 x 14 86 -> 235 us).
//   * K groups of waves in a workgroup: groups of four waves with stage buffers of their own walk parts of K side by side and exchange
//     halves of their sums through LDS.  For workgroups that are alone on their CU.
//   * K may be split over `sk` workgroups per tile (partial tiles at device scope, the last to arrive adds
//     them in slice order and finishes): for layers whose tiles leave most of the chip idle.
//   * Workgroups are numbered so that one die (workgroup id % 8) owns a contiguous run of tiles with the
//     output-channel tiles of one pixel tile next to each other: its L2 serves the re-reads.
#include <cmath>
#include <cstring>
#include <type_traits>

#include "conv_cl.h"

namespace cadnn {

namespace {

typedef _Float16 cl_h8 __attribute__((ext_vector_type(8)));
typedef _Float16 cl_h4 __attribute__((ext_vector_type(4)));
typedef __bf16 cl_b8 __attribute__((ext_vector_type(8)));
typedef float cl_f4 __attribute__((ext_vector_type(4)));
typedef float cl_f16v __attribute__((ext_vector_type(16)));
typedef uint32_t cl_u4 __attribute__((ext_vector_type(4)));
typedef uint32_t cl_u2 __attribute__((ext_vector_type(2)));

template <int I, int N, class F>
__device__ __forceinline__ void cl_static_for(F&& f) {
    if constexpr (I < N) {
        f(std::integral_constant<int, I>());
        cl_static_for<I + 1, N>(f);
    }
}

// Waits until at most VM vector-memory operations and no LDS read of this wave are outstanding.  (The builtin
// and not an asm statement: the compiler, which tracks its own loads, then knows that they have landed.)
template <int VM>
__device__ __forceinline__ void cl_wait() {
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt((VM & 15) | (7 << 4) | ((VM >> 4) << 14));
    asm volatile("" ::: "memory");
}
__device__ __forceinline__ void cl_barrier() {
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

// 16 (4) bytes per lane from memory to LDS (lane l: lds + 16 l, 4 l).  The wait for it is the caller's.
__device__ __forceinline__ void cl_dma(cl_u4 rsrc, uint32_t voff, uint32_t soff, uint32_t lds) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds"
                 :: "s"(lds), "v"(voff), "s"(rsrc), "s"(soff) : "memory");
}

__device__ __forceinline__ void cl_dma4(cl_u4 rsrc, uint32_t voff, uint32_t lds) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dword %1, %2, 0 offen lds"
                 :: "s"(lds), "v"(voff), "s"(rsrc) : "memory");
}

__device__ __forceinline__ cl_u4 cl_rsrc(const void* p, uint32_t span) {
    const uint64_t a = (uint64_t)p;
    cl_u4 r;
    r[0] = __builtin_amdgcn_readfirstlane((uint32_t)a);
    r[1] = __builtin_amdgcn_readfirstlane((uint32_t)(a >> 32) & 0xffffu);
    r[2] = __builtin_amdgcn_readfirstlane(span);
    r[3] = 0x00020000u;
    return r;
}

// A tile of 64 MI channels x 64 NI pixels, AM x AN accumulators of 32 x 32 for each of 4 waves; S stage buffers; KG such
// groups of 4 waves, each with buffers and a part of K of its own.
// 2 x 2 waves; in 4-byte storage a wave has 32 pixels, whose activations it takes apart for all of its products.
template <typename T, int RB, int MI, int NI, int S, int KG>
struct ClCfg {
    static constexpr int TM = 64 * MI, TN = 64 * NI;
    static constexpr int WN = sizeof(T) == 4 ? 2 * NI : 2;
    static constexpr int AM = 2 * MI * WN / 4, AN = 2 * NI / WN;
    static constexpr int WB = 64 * cl_weight_bytes(RB, sizeof(T));          // bytes of a step of 64 output channels
    static constexpr int LA = (MI * WB + 4095) / 4096, LB = TN * RB / 4096; // loads per thread and stage
    static constexpr int A_BYTES = LA * 4096;
    static constexpr int STAGE = A_BYTES + TN * RB;
    static constexpr int cmax(int a, int b) { return a > b ? a : b; }
    static constexpr int GROUP = S * STAGE;
    static constexpr int KEPT = AM * AN * 16 / KG;           // sums of a thread behind the K loop
    static constexpr int MAIN = cmax(KG * GROUP, KG == 1 ? 0 : AM * AN * 16 * 1024);       // (the groups exchange sums there)
    static constexpr int LDS = MAIN + TN * 16 + TM * 8 + 16;
};

// What a launch is, beside a layer between channels-last tensors.
enum ClMode { CL_MAPS = 0, CL_PLANES = 1, CL_ODD_ROW = 2 };

// (two waves per SIMD asked for: all registers then are of one kind, no accumulator copies in the loop)
// CL_PLANES: y and the residual are [n][c][h][w] (a layer called on its own).  A lane then stores its pixel of each
// channel straight from the accumulators: 32 lanes write 64 (fp16) or 128 contiguous bytes, which
// costs less than a pass of its own over y (a launch, 4 us at the least).
// CL_ODD_ROW: a first layer in 2-byte storage whose filter rows have an odd number of pixels, 8 bytes each.  A step is
// wider than such a row.  Whole pieces behind it are not requested at all (that goes for every first
// layer); the piece that is half the next pixel's loses that half in the registers, because a zero weight does not
// undo an infinity or a NaN.  (Four more instructions a step; other layers take the kernels without them.)
template <typename T, int RB, int MI, int NI, int S, int KG, int MODE>
__global__ __launch_bounds__(256 * KG, MI * NI == 1 ? 4 : 2) void cl_conv_kernel(const ClArgs a) {
    using C = ClCfg<T, RB, MI, NI, S, KG>;
    static_assert(KG <= 2, "two groups exchange halves of their sums");
    constexpr bool PLANES = MODE == CL_PLANES;
    static_assert(MODE != CL_ODD_ROW || sizeof(T) == 2, "a pixel of 4-byte storage is a whole piece");
    constexpr int TM = C::TM, TN = C::TN, STAGE = C::STAGE;
    constexpr int RPL = 1024 / RB;                 // rows one wave-load fills
    constexpr int LA = C::LA, LB = C::LB;
    constexpr bool SPLIT = sizeof(T) == 4;
    constexpr int AM = C::AM, AN = C::AN;
    constexpr int WB = C::WB;
    constexpr int PIECES = RB / 16;
    constexpr int EPP = 16 / (int)sizeof(T);       // elements per 16-byte piece
    extern __shared__ __attribute__((aligned(16))) char cl_smem[];
    int4* ptab = (int4*)(cl_smem + C::MAIN);       // per pixel of the tile: byte offsets in x, x2, y, residual
    float* bl = (float*)(cl_smem + C::MAIN + TN * 16);
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)cl_smem;

    // ---- the launch record is fetched whole and at once (field by field, as the compiler would place the loads, it
    //      is a chain of a dozen scalar-cache misses in front of the first load of data)
    asm volatile("" :: "s"(a.w), "s"(a.x), "s"(a.x2), "s"(a.y), "s"(a.res), "s"(a.bias), "s"(a.bias2), "s"(a.part), "s"(a.count),
                 "s"(a.wspan), "s"(a.total), "s"(a.hw), "s"(a.ow), "s"(a.cout), "s"(a.relu), "s"(a.steps_tap), "s"(a.steps1), "s"(a.steps),
                 "s"(a.ntaps), "s"(a.tiles_m), "s"(a.tiles), "s"(a.per_die), "s"(a.sk), "s"(a.log_sk), "s"(a.per_slice), "s"(a.magic_hw), "s"(a.magic_ow),
                 "s"(a.magic_tm), "s"(a.row_bytes));
    asm volatile("" :: "s"(a.xt.span), "s"(a.xt.img), "s"(a.xt.row), "s"(a.xt.col), "s"(a.xt.org), "s"(a.x2t.img), "s"(a.x2t.row), "s"(a.x2t.col),
                 "s"(a.x2t.org), "s"(a.yt.span), "s"(a.yt.img), "s"(a.yt.row), "s"(a.yt.col), "s"(a.yt.org), "s"(a.rt.span), "s"(a.rt.img),
                 "s"(a.rt.row), "s"(a.rt.col), "s"(a.rt.org), "s"(a.tap_off[0]));

    // ---- which tile: dies own contiguous runs
    const int t = ((int)blockIdx.x & 7) * a.per_die + ((int)blockIdx.x >> 3);
    if (((int)blockIdx.x >> 3) >= a.per_die || t >= a.tiles) return;
    const int rest = cl_div(t, a.magic_tm, a.tiles_m), mt = t - rest * a.tiles_m;
    const int z = rest & (a.sk - 1), nt = rest >> a.log_sk;
    const int m0 = mt * TM, n0 = nt * TN;

    const int tid = (int)threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), kg = KG == 1 ? 0 : wave >> 2, wv = wave & 3;
    const int wm = wv / C::WN, wn = wv % C::WN;

    // ---- the weights of the first stage need nothing but the tile's number: on their way before all else
    constexpr int L = LA + LB;
    // (all groups of a workgroup go through the steps of the first; what one lacks of them is zeros, fetched from out of range)
    const int s_first = (z * KG + kg) * a.per_slice, steps = min(a.per_slice, a.steps - z * KG * a.per_slice);
    uint32_t va = KG > 1 && s_first >= a.steps ? kClOutOfRange : (uint32_t)(lane * 16);
    const cl_u4 wr = cl_rsrc(a.w, a.wspan);
    // (a load moves 1 KB per wave, and a 64-row block is a whole number of these; the last load of a
    // stage has nothing left to fetch for the waves past the blocks' end)
    uint32_t wsoff[LA];
    uint32_t va_last = LA * 4 > MI * WB / 1024 && LA * 4 - 4 + wv >= MI * WB / 1024 ? kClOutOfRange : va;
    auto start_weights = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < LA; ++i) {
            const int chunk = min(i * 4 + wv, MI * WB / 1024 - 1), block = chunk / (WB / 1024);
            wsoff[i] = (uint32_t)((mt * MI + block) * a.steps + s_first) * (uint32_t)WB + (uint32_t)(chunk - block * (WB / 1024)) * 1024u;
        }
    };
    start_weights();
    const uint32_t lds_w = lds0 + (uint32_t)(kg * C::GROUP + wv * 1024);
    auto issue_w = [&](auto I, uint32_t buf) __attribute__((always_inline)) {
        constexpr int i = decltype(I)::value;
        cl_dma(wr, i == LA - 1 ? va_last : va, wsoff[i], lds_w + buf * STAGE + (uint32_t)i * 4096u);
    };
    cl_static_for<0, LA>([&](auto I) __attribute__((always_inline)) { issue_w(I, 0u); });

    // the biases go to LDS the same way (out of range: 0)
    if (kg == 0 && wv < TM / 32) {
        const bool second = wv >= TM / 64;
        const int chunk = second ? wv - TM / 64 : wv;
        const float* const src = second ? a.bias2 : a.bias;
        cl_dma4(cl_rsrc(src, src ? (uint32_t)a.cout * 4u : 0u), (uint32_t)(m0 + chunk * 64 + lane) * 4u,
                lds0 + (uint32_t)(C::MAIN + TN * 16 + wv * 256));
    }
    // (what the first loads need; a 32-bit product takes as long as four other instructions)
    int img = 0, oh = 0, ow = 0;
    if (tid < TN) {
        const int Q = n0 + tid;
        int4 e = make_int4((int)kClOutOfRange, (int)kClOutOfRange, (int)kClOutOfRange, (int)kClOutOfRange);
        if (Q < a.total) {
            img = cl_div(Q, a.magic_hw, a.hw);
            const int q = Q - img * a.hw;
            oh = cl_div(q, a.magic_ow, a.ow);
            ow = q - oh * a.ow;
            e.x = img * a.xt.img + oh * a.xt.row + ow * a.xt.col + a.xt.org;
            if (a.steps > a.steps1) e.y = img * a.x2t.img + oh * a.x2t.row + ow * a.x2t.col + a.x2t.org;
            if (a.res) e.w = img * a.rt.img + oh * a.rt.row + ow * a.rt.col + a.rt.org;
        }
        ptab[tid] = e;
    }
    int* const odd = (int*)(bl + 2 * TM);           // SPLIT: a sum of this workgroup's is not finite
    if (SPLIT && tid == 0) *odd = 0;
    // (no wait for memory here, as __syncthreads would have: only the table in LDS is awaited)
    __builtin_amdgcn_s_waitcnt(0xc07f);
    cl_barrier();

    // ---- sources: this thread's row (of each group of rows) and 16-byte piece
    const int lrow = lane / PIECES, lpos = lane % PIECES;
    const int sw = RB == 128 ? ((wv * RPL + lrow) >> 1) & 7 : (lrow >> 2) & 3;
    const uint32_t piece = (uint32_t)(lpos ^ sw) * 16u;
    uint32_t vb[LB];
    cl_u4 xr;
    auto start_sources = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < LB; ++j) {
            const int e = ptab[j * 4 * RPL + wv * RPL + lrow].x;
            vb[j] = e == (int)kClOutOfRange || (int)piece >= a.row_bytes ? kClOutOfRange : (uint32_t)e + piece;
        }
        xr = cl_rsrc(a.x, a.xt.span);
    };
    start_sources();

    // ---- the residual's pieces are requested up front where they fit few registers.  (A lane has, of a block of 32 channels and its
    //      pixel, the pieces 2 p + l / 32: the rows of a block of weights are in an order that makes it so.)
    constexpr int PER = 16 / KG, NP = PER / EPP, ITEMS = AM * AN * NP;      // sums of a block that a thread keeps, pieces, pieces in all
    constexpr bool EARLY = ITEMS <= 8 && !PLANES;
    const int l31 = lane & 31, fk = lane >> 5;
    const __amdgpu_buffer_rsrc_t rrs = __builtin_amdgcn_make_buffer_rsrc((void*)a.res, 0, a.rt.span, 0x00020000);
    auto piece_channel = [&](int mi, int p) __attribute__((always_inline)) {
        return m0 + wm * 32 * AM + mi * 32 + kg * 16 + (p * 2 + fk) * EPP;
    };
    cl_u4 resv[EARLY ? ITEMS : 1];
    auto res_load = [&](int at, int mi, int p) __attribute__((always_inline)) {
        const int ch = piece_channel(mi, p);
        const uint32_t off = (ch < a.cout && at != (int)kClOutOfRange) ? (uint32_t)(at + ch * (int)sizeof(T)) : kClOutOfRange;
        return __builtin_bit_cast(cl_u4, __builtin_amdgcn_raw_buffer_load_b128(rrs, off, 0u, 0));
    };
    if constexpr (EARLY) {
        if (a.res) {
#pragma unroll
            for (int ni = 0; ni < AN; ++ni) {
                const int at = ptab[wn * 32 * AN + ni * 32 + l31].w;
#pragma unroll
                for (int k = 0; k < AM * NP; ++k) resv[ni * AM * NP + k] = res_load(at, k / NP, k % NP);
            }
        }
    }

    // ---- the walk over this workgroup's slice of K
    int f_left, f_tap, f_todo, f_own;
    uint32_t f_soff;
    auto enter_shortcut = [&](int at) __attribute__((always_inline)) {
        xr = cl_rsrc(a.x2, a.x2t.span);
#pragma unroll
        for (int j = 0; j < LB; ++j) {
            const int e = ptab[j * 4 * RPL + wv * RPL + lrow].y;
            vb[j] = e == (int)kClOutOfRange ? kClOutOfRange : (uint32_t)e + piece;
        }
        f_left = 0x7fffffff;
        f_soff = (uint32_t)at * RB;
    };
    auto past_end = [&]() __attribute__((always_inline)) {
        va = va_last = kClOutOfRange;
        // (the scalar offsets go back to the start, from where the steps left stay inside the span: what an offset is checked
        // against, the span or the span less the scalar offset, is then never negative)
#pragma unroll
        for (int i = 0; i < LA; ++i) wsoff[i] = 0;
#pragma unroll
        for (int j = 0; j < LB; ++j) vb[j] = kClOutOfRange;
        f_left = 0x7fffffff;
        f_soff = 0;
    };
    auto start_walk = [&]() __attribute__((always_inline)) {
        f_tap = 0;
        f_todo = steps;
        f_own = a.steps - s_first;
        if constexpr (KG > 1) {
            if (f_own <= 0) return past_end();
        }
        if (s_first == 0) {
            f_left = a.steps_tap;
            f_soff = (uint32_t)a.tap_off[0];
        } else if (s_first < a.steps1) {
            f_tap = cl_div(s_first, a.magic_st, a.steps_tap);
            const int at = s_first - f_tap * a.steps_tap;
            f_left = a.steps_tap - at;
            f_soff = (uint32_t)a.tap_off[f_tap] + (uint32_t)at * RB;
        } else {
            enter_shortcut(s_first - a.steps1);
        }
    };
    start_walk();
    // load i of a stage: the weights' first, then the activations'
    auto issue_one = [&](auto I, uint32_t buf) __attribute__((always_inline)) {
        constexpr int i = decltype(I)::value;
        if constexpr (i < LA) issue_w(I, buf);
        else cl_dma(xr, vb[i - LA], f_soff, lds_w + buf * STAGE + (uint32_t)i * 4096u);
    };
    auto advance = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < LA; ++i) wsoff[i] += (uint32_t)WB;
        f_soff += RB;
        --f_todo;
        if constexpr (KG > 1) { if (--f_own == 0) past_end(); }
        if (--f_left == 0 && f_todo > 0) {
            if (++f_tap < a.ntaps) {
                f_left = a.steps_tap;
                f_soff = (uint32_t)a.tap_off[f_tap];
            } else {
                enter_shortcut(0);
            }
        }
    };
    cl_f16v acc[AM][AN], low[SPLIT ? AM : 1][SPLIT ? AN : 1];
    auto clear_sums = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int mi = 0; mi < AM; ++mi)
#pragma unroll
            for (int ni = 0; ni < AN; ++ni)
#pragma unroll
                for (int i = 0; i < 16; ++i) {
                    acc[mi][ni][i] = 0.0f;
                    if constexpr (SPLIT) low[mi][ni][i] = 0.0f;
                }
    };
    clear_sums();

    // fragment addresses: row l % 32 of a 32-row block, piece 2 ks + l / 32 (permuted by the row)
    const int fs = RB == 128 ? (lane >> 1) & 7 : (lane >> 2) & 3;
    const uint32_t fb = (uint32_t)(kg * C::GROUP + C::A_BYTES + (wn * 32 * AN + l31) * RB);
    const uint32_t fp = (uint32_t)((fk ^ fs) * 16);

    // A stage's fragments are read into registers one stage ahead of its products, so LDS latency and
    // the products overlap inside a wave, and a stage's buffer is free again as soon as it is read:
    //   wait until this wave's loads of stage s + 1 have landed -- barrier: everybody's have, and everybody
    //   has read stage s -- load stage s + S into the buffer of stage s -- read stage s + 1 -- multiply stage s
    auto wait_loads = [&](int behind) __attribute__((always_inline)) {
        // `behind` stages may stay in flight behind the one needed now
        cl_static_for<1, S>([&](auto B) __attribute__((always_inline)) {
            if (behind == decltype(B)::value) cl_wait<decltype(B)::value * L>();
        });
        if (behind <= 0) cl_wait<0>();
    };
    static_assert((S - 1) * L <= 63, "the wait counter counts to 63");
    cl_static_for<LA, L>([&](auto I) __attribute__((always_inline)) { issue_one(I, 0u); });
    advance();
    for (int j = 1; j < S && j < steps; ++j) {
        cl_static_for<0, L>([&](auto I) __attribute__((always_inline)) { issue_one(I, (uint32_t)j); });
        advance();
    }
    if (tid < TN && n0 + tid < a.total)             // (read behind the K loop)
        ptab[tid].z = img * a.yt.img + oh * a.yt.row + ow * a.yt.col + a.yt.org;
    typedef std::integral_constant<int, 0> Set0;
    typedef std::integral_constant<int, 1> Set1;
    wait_loads(min(steps, S) - 1);
    cl_barrier();
    if constexpr (!SPLIT) {
        constexpr int KS = RB / 32;                    // MFMA groups per stage
        const uint32_t fa = (uint32_t)(kg * C::GROUP + (wm * 32 * AM + l31) * RB);
        cl_u4 af[2][KS][AM], bf[2][KS][AN];
        auto read_frags = [&](auto F, uint32_t buf) __attribute__((always_inline)) {
            constexpr int f = decltype(F)::value;
            const char* st = cl_smem + buf * STAGE;
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) {
                const uint32_t p = fp ^ (uint32_t)(ks * 32);
#pragma unroll
                for (int mi = 0; mi < AM; ++mi) af[f][ks][mi] = *(const cl_u4*)(st + fa + mi * 32 * RB + p);
#pragma unroll
                for (int ni = 0; ni < AN; ++ni) bf[f][ks][ni] = *(const cl_u4*)(st + fb + ni * 32 * RB + p);
                if constexpr (MODE == CL_ODD_ROW) {
                    const uint32_t own = 2 * ks + fk == a.row_bytes / 16 ? 0u : ~0u;
#pragma unroll
                    for (int ni = 0; ni < AN; ++ni) {
                        bf[f][ks][ni][2] &= own;
                        bf[f][ks][ni][3] &= own;
                    }
                }
            }
        };
        auto multiply = [&](auto F, auto K) __attribute__((always_inline)) {
            constexpr int f = decltype(F)::value, ks = decltype(K)::value;
#pragma unroll
            for (int mi = 0; mi < AM; ++mi)
#pragma unroll
                for (int ni = 0; ni < AN; ++ni) {
                    acc[mi][ni] = __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(cl_h8, af[f][ks][mi]),
                                                                         __builtin_bit_cast(cl_h8, bf[f][ks][ni]), acc[mi][ni], 0, 0, 0);
                }
        };
        read_frags(std::integral_constant<int, 0>(), 0);
        uint32_t cur = 0;                       // buffer of the stage being multiplied
        // (FULL: stage s + S exists, known at compile time)
        auto stage = [&](auto F, auto FULL, int s) __attribute__((always_inline)) {
            constexpr int f = decltype(F)::value;
            constexpr bool full = decltype(FULL)::value;
            const uint32_t nxt = cur + 1 == S ? 0 : cur + 1;
            const bool more = full || s + S < steps;
            if (full || s + 1 < steps) {
                // stages s + 2 .. s + S - 1 are in flight behind stage s + 1
                if (more || s + S == steps) cl_wait<(S - 2) * L>();
                else wait_loads(steps - 2 - s);
                cl_barrier();
                read_frags(std::integral_constant<int, f ^ 1>(), nxt);
            }
            // A load to LDS holds its wave for as long as the memory pipeline takes 64 addresses (16 clocks
            // and more while the other waves' are in front); between products that time is the matrix pipe's.
            // (The scheduler is held to the order: LDS reads, then products and loads in turn.)
            cl_static_for<0, KS>([&](auto K) __attribute__((always_inline)) {
                constexpr int k = decltype(K)::value;
                __builtin_amdgcn_sched_barrier(0);
                multiply(F, K);
                __builtin_amdgcn_sched_barrier(0);
                if (more) cl_static_for<k * L / KS, (k + 1) * L / KS>([&](auto I) __attribute__((always_inline)) { issue_one(I, cur); });
            });
            if (more) advance();
            cur = nxt;
        };
        int s = 0;
        for (; s + 1 + S < steps; s += 2) {
            stage(Set0(), std::true_type(), s);
            stage(Set1(), std::true_type(), s + 1);
        }
        for (; s < steps; s += 2) {
            stage(Set0(), std::false_type(), s);
            if (s + 1 < steps) stage(Set1(), std::false_type(), s + 1);
        }
    } else {
        // Fragments are read one group of 16 k ahead of their products.  The weights of a group lie as
        // three planes of bf16, [64 channels][16 bytes] for either half of the wave: 512 bytes in a row for 32
        // lanes.  Lane half fk takes k = 4 fk + {0..3, 8..11} of a group, as two pieces of the activations hold them.
        constexpr int G = RB / 64;
        const int fr = wm * 32 * AM + l31;
        const uint32_t fa = (uint32_t)(kg * C::GROUP + (fr / 64) * WB + (fr % 64) * 16 + fk * 1024);
        // (The largest tile has registers for one set of weights: a part is read again for the next group behind its last product.)
        constexpr int SETS = AM == 4 ? 1 : 2;
        cl_u4 af[SETS][3][AM], bf[2][2][AN];
        auto read_weights = [&](auto F, auto GRP, auto P, uint32_t buf) __attribute__((always_inline)) {
            constexpr int f = decltype(F)::value % SETS, g = decltype(GRP)::value, p = decltype(P)::value;
            const char* st = cl_smem + buf * STAGE;
#pragma unroll
            for (int mi = 0; mi < AM; ++mi) af[f][p][mi] = *(const cl_u4*)(st + fa + mi / 2 * WB + mi % 2 * 512 + (g * 3 + p) * 2048);
        };
        auto read_pixels = [&](auto F, auto GRP, uint32_t buf) __attribute__((always_inline)) {
            constexpr int f = decltype(F)::value, g = decltype(GRP)::value;
            const char* st = cl_smem + buf * STAGE;
#pragma unroll
            for (int ni = 0; ni < AN; ++ni)
#pragma unroll
                for (int h = 0; h < 2; ++h) bf[f][h][ni] = *(const cl_u4*)(st + fb + ni * 32 * RB + (fp ^ (uint32_t)((2 * g + h) * 32)));
        };
        auto read_all_weights = [&](auto F, auto GRP, uint32_t buf) __attribute__((always_inline)) {
            cl_static_for<0, 3>([&](auto I) __attribute__((always_inline)) {
                read_weights(F, GRP, std::integral_constant<int, 2 - decltype(I)::value>(), buf);
            });
        };
        auto read_group = [&](auto F, auto GRP, uint32_t buf) __attribute__((always_inline)) {
            read_pixels(F, GRP, buf);
            if constexpr (SETS == 2) read_all_weights(F, GRP, buf);
        };
        // (the last product, of the leading parts, has its own sum: the others' are 2^-8 of it and less, and so are their roundings)
        // x w = x1 w1 + (x1 w2 + x2 w1) + (x1 w3 + x2 w2 + x3 w1) + ...: what is left out, x2 w3 + x3 w2, is 2^-24 of a product at
        // the most (operands just above a power of two whose second parts are largest), and of either sign.  (`load(I)`, I < 6: called behind each product; vector and scalar arithmetic
        // moves across, so that the next part is taken off beside the product before it; one set of weights: that of group GRP
        // of buffer `buf` follows, if there is one)
        static_assert(AN == 1, "a wave takes one block of pixels apart");
        auto multiply = [&](auto F, auto GRP, bool follows, uint32_t buf, auto&& load) __attribute__((always_inline)) {
            constexpr int f = decltype(F)::value;
            cl_u4 x1, x2, x3;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                uint32_t p1, p2, p3;
                cl_split2(__uint_as_float(bf[f][j / 2][0][j % 2 * 2]), __uint_as_float(bf[f][j / 2][0][j % 2 * 2 + 1]), &p1, &p2, &p3);
                x1[j] = p1;
                x2[j] = p2;
                x3[j] = p3;
            }
            cl_static_for<0, 6>([&](auto I) __attribute__((always_inline)) {
                constexpr int i = decltype(I)::value, p = i == 0 ? 2 : i < 3 ? 1 : 0;
                const cl_u4 x = i == 0 || i == 1 || i == 5 ? x1 : i == 3 ? x3 : x2;
#pragma unroll
                for (int mi = 0; mi < AM; ++mi) {
                    cl_f16v& to = i == 5 ? acc[mi][0] : low[mi][0];
                    to = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(cl_b8, af[f % SETS][p][mi]), __builtin_bit_cast(cl_b8, x), to, 0, 0, 0);
                }
                __builtin_amdgcn_sched_barrier(6);
                if constexpr (SETS == 1 && (i == 0 || i == 2 || i == 5)) {
                    if (follows) read_weights(F, GRP, std::integral_constant<int, p>(), buf);
                }
                load(I);
                __builtin_amdgcn_sched_barrier(6);
            });
        };
        read_group(Set0(), Set0(), 0);
        if constexpr (SETS == 1) read_all_weights(Set0(), Set0(), 0);
        uint32_t cur = 0;
        // A stage's loads start behind its barrier and end, where it has two groups, in front of the next one, between the
        // products of both: a load to LDS holds its wave until the memory pipeline has its addresses.
        constexpr int HALF = G == 2 && S > 2 ? (L + 1) / 2 : L;
        auto loads = [&](auto FROM, auto TO, auto I, uint32_t buf) __attribute__((always_inline)) {
            constexpr int from = decltype(FROM)::value, n = decltype(TO)::value - from, i = decltype(I)::value;
            cl_static_for<from + i * n / 6, from + (i + 1) * n / 6>([&](auto K) __attribute__((always_inline)) { issue_one(K, buf); });
        };
        typedef std::integral_constant<int, 0> First;
        typedef std::integral_constant<int, HALF> Half;
        typedef std::integral_constant<int, L> Last;
        // (F: the set that holds the stage's first group; pending: the stage before this one has loads left)
        auto stage = [&](auto F, auto FULL, bool pending, int s) __attribute__((always_inline)) {
            constexpr int f = decltype(F)::value;
            constexpr bool full = decltype(FULL)::value;
            const uint32_t nxt = cur + 1 == S ? 0 : cur + 1;
            const bool more = full || s + S < steps;
            constexpr int last = G == 2 ? f ^ 1 : f;
            if constexpr (G == 2) {
                // (the first group has long landed; waited for behind the second's request, both would be)
                if constexpr (SETS == 2) __builtin_amdgcn_s_waitcnt(0xc07f);
                read_group(std::integral_constant<int, last>(), Set1(), cur);
                __builtin_amdgcn_sched_barrier(0);
                const uint32_t before = cur == 0 ? S - 1 : cur - 1;
                multiply(F, Set1(), true, cur, [&](auto I) __attribute__((always_inline)) {
                    if (pending) loads(Half(), Last(), I, before);
                });
                if (pending) advance();
                __builtin_amdgcn_sched_barrier(0);
            }
            if (full || s + 1 < steps) {
                if (more || s + S == steps) cl_wait<(S - 2) * L>();
                else wait_loads(steps - 2 - s);
                cl_barrier();
                read_group(std::integral_constant<int, last ^ 1>(), Set0(), nxt);
            }
            __builtin_amdgcn_sched_barrier(0);
            multiply(std::integral_constant<int, last>(), Set0(), full || s + 1 < steps, nxt, [&](auto I) __attribute__((always_inline)) {
                if (more) loads(First(), Half(), I, cur);
            });
            __builtin_amdgcn_sched_barrier(0);
            if (G == 1 && more) advance();
            cur = nxt;
        };
        int s = 0;
        if constexpr (G == 2) {
            bool pending = S < steps;
            stage(Set0(), std::false_type(), false, 0);
            for (s = 1; s + S < steps; ++s) stage(Set0(), std::true_type(), true, s);
            for (; s < steps; ++s) {
                stage(Set0(), std::false_type(), pending, s);
                pending = false;
            }
        } else {
            for (; s + 1 + S < steps; s += 2) {
                stage(Set0(), std::true_type(), false, s);
                stage(Set1(), std::true_type(), false, s + 1);
            }
            for (; s < steps; s += 2) {
                stage(Set0(), std::false_type(), false, s);
                if (s + 1 < steps) stage(Set1(), std::false_type(), false, s + 1);
            }
        }
        // An infinity or a NaN among the operands, or operands or sums whose scale takes them beyond the range (2^104, 2^80), leave
        // sums that are not finite: a tile with such sums is done again with fp32 products, and they take what these give.
        // (Channels behind the last one have weights that nobody wrote.)
#pragma unroll
        for (int mi = 0; mi < AM; ++mi)
#pragma unroll
            for (int ni = 0; ni < AN; ++ni)
#pragma unroll
                for (int i = 0; i < 16; ++i) acc[mi][ni][i] += low[mi][ni][i];
        float seen = 0.0f;
        auto look = [&](auto ALL) __attribute__((always_inline)) {
#pragma unroll
            for (int mi = 0; mi < AM; ++mi)
#pragma unroll
                for (int ni = 0; ni < AN; ++ni)
#pragma unroll
                    for (int i = 0; i < 16; ++i) {
                        const bool live = decltype(ALL)::value || m0 + wm * 32 * AM + mi * 32 + (i >> 2) * 8 + fk * 4 + (i & 3) < a.cout;
                        seen = fmaf(live ? acc[mi][ni][i] : 0.0f, 0.0f, seen);
                    }
        };
        if (m0 + TM <= a.cout) look(std::true_type());
        else look(std::false_type());
        if (__ballot(!(seen == 0.0f)) != 0 && lane == 0) *odd = 1;
        __syncthreads();
        if (__builtin_amdgcn_readfirstlane(*odd)) {
            if (KG > 1 && s_first < a.steps) {
                va = (uint32_t)(lane * 16);
                va_last = LA * 4 > MI * WB / 1024 && LA * 4 - 4 + wv >= MI * WB / 1024 ? kClOutOfRange : va;
            }
            start_weights();
            start_sources();
            start_walk();
            cl_f16v kept[AM][AN];
#pragma unroll
            for (int mi = 0; mi < AM; ++mi)
#pragma unroll
                for (int ni = 0; ni < AN; ++ni) kept[mi][ni] = acc[mi][ni];
            clear_sums();
            for (int s2 = 0; s2 < steps; ++s2) {
                cl_static_for<0, L>([&](auto I) __attribute__((always_inline)) { issue_one(I, 0u); });
                advance();
                cl_wait<0>();
                cl_barrier();
                cl_static_for<0, G>([&](auto GRP) __attribute__((always_inline)) {
                    read_pixels(Set0(), GRP, 0);
                    read_all_weights(Set0(), GRP, 0);
#pragma unroll
                    for (int i = 0; i < 8; ++i)
#pragma unroll
                        for (int mi = 0; mi < AM; ++mi) {
                            auto part = [&](int p) __attribute__((always_inline)) { return (uint16_t)(af[0][p][mi][i / 2] >> (i % 2 * 16)); };
                            const float w = cl_join_weight(part(0), part(1), part(2));
#pragma unroll
                            for (int ni = 0; ni < AN; ++ni)
                                acc[mi][ni] = __builtin_amdgcn_mfma_f32_32x32x2f32(w, __uint_as_float(bf[0][i / 4][ni][i % 4]), acc[mi][ni], 0, 0, 0);
                        }
                });
                cl_wait<0>();
                cl_barrier();
            }
#pragma unroll
            for (int mi = 0; mi < AM; ++mi)
#pragma unroll
                for (int ni = 0; ni < AN; ++ni)
#pragma unroll
                    for (int i = 0; i < 16; ++i)
                        if (kept[mi][ni][i] * 0.0f == 0.0f) acc[mi][ni][i] = kept[mi][ni][i] * kClSumUnscale;
        } else {
#pragma unroll
            for (int mi = 0; mi < AM; ++mi)
#pragma unroll
                for (int ni = 0; ni < AN; ++ni)
#pragma unroll
                    for (int i = 0; i < 16; ++i) acc[mi][ni][i] *= kClSumUnscale;
        }
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");        // (the residual's pieces)
    // ---- the groups' sums: each keeps one half of every block's (channels 16 kg and up of its 32) and gives away the other,
    //      the first group's part of K added first
    float sum[C::KEPT];
    if constexpr (KG == 1) {
#pragma unroll
        for (int i = 0; i < C::KEPT; ++i) sum[i] = acc[i / 16 / AN][i / 16 % AN][i % 16];
    } else {
        float* const swap = (float*)cl_smem;
        __syncthreads();                            // the stage buffers are free: every wave is past its last read
        auto give = [&](auto MINE) __attribute__((always_inline)) {
            constexpr int mine = decltype(MINE)::value;
#pragma unroll
            for (int i = 0; i < C::KEPT; ++i) {
                const cl_f16v& block = acc[i / PER / AN][i / PER % AN];
                sum[i] = block[mine * PER + i % PER];
                swap[i * 512 + tid] = block[(1 - mine) * PER + i % PER];
            }
        };
        if (kg == 0) give(std::integral_constant<int, 0>());
        else give(std::integral_constant<int, 1>());
        __syncthreads();
#pragma unroll
        for (int i = 0; i < C::KEPT; ++i) {
            const float other = swap[i * 512 + (tid ^ 256)];
            sum[i] = kg == 0 ? sum[i] + other : other + sum[i];
        }
    }
    // ---- K split over workgroups: the slices of a tile meet in memory (device-scope accesses go to the level
    //      all dies share; every thread's stores are acknowledged before the arrival is counted)
    if (a.sk > 1) {
        const size_t tile_id = (size_t)nt * a.tiles_m + mt;
        float* mine = a.part + (tile_id * a.sk + z) * (size_t)(TM * TN);
#pragma unroll
        for (int i = 0; i < C::KEPT; ++i)
            __hip_atomic_store(mine + i * 256 * KG + tid, sum[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
        int* flag = (int*)cl_smem;
        if (tid == 0) {
            const int arrived = __hip_atomic_fetch_add(a.count + tile_id, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            *flag = arrived == a.sk - 1;
            if (arrived == a.sk - 1) a.count[tile_id] = 0;      // every other slice has counted itself: ready for the next launch
        }
        __syncthreads();
        const bool last = *flag != 0;
        __syncthreads();
        if (!last) return;
#pragma unroll
        for (int i = 0; i < C::KEPT; ++i) sum[i] = 0.0f;
        for (int k = 0; k < a.sk; ++k) {
            const float* src = a.part + (tile_id * a.sk + k) * (size_t)(TM * TN);
#pragma unroll
            for (int i = 0; i < C::KEPT; ++i)
                sum[i] += __hip_atomic_load(src + i * 256 * KG + tid, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
    }

    // ---- epilogue, straight from the accumulators: bias, residual and ReLU in fp32, one rounding.  (PLANES: a store takes 32
    //      pixels of a channel.)
    const __amdgpu_buffer_rsrc_t yrs = __builtin_amdgcn_make_buffer_rsrc((void*)a.y, 0, a.yt.span, 0x00020000);
#pragma unroll
    for (int ni = 0; ni < AN; ++ni) {
        const int4 e = ptab[wn * 32 * AN + ni * 32 + l31];
#pragma unroll
        for (int mi = 0; mi < AM; ++mi) {
            float v[PER];
#pragma unroll
            for (int p = 0; p < NP; ++p)
#pragma unroll
                for (int j = 0; j < EPP; j += 4) {
                    const float* const at = bl + piece_channel(mi, p) - m0 + j;
                    const cl_f4 b1 = *(const cl_f4*)at, b2 = *(const cl_f4*)(at + TM);
#pragma unroll
                    for (int i = 0; i < 4; ++i) v[p * EPP + j + i] = sum[(mi * AN + ni) * PER + p * EPP + j + i] + (b1[i] + b2[i]);
                }
            if constexpr (PLANES) {
                uint32_t off[PER];
#pragma unroll
                for (int i = 0; i < PER; ++i) {
                    const int ch = piece_channel(mi, i / EPP) + i % EPP;
                    off[i] = ch < a.cout && e.z != (int)kClOutOfRange ? (uint32_t)(e.z + ch * a.plane) : kClOutOfRange;
                }
                if (a.res) {
                    T r[PER];
#pragma unroll
                    for (int i = 0; i < PER; ++i) {
                        if constexpr (sizeof(T) == 2) r[i] = __builtin_bit_cast(T, (uint16_t)__builtin_amdgcn_raw_buffer_load_b16(rrs, off[i], 0u, 0));
                        else r[i] = __builtin_bit_cast(T, (uint32_t)__builtin_amdgcn_raw_buffer_load_b32(rrs, off[i], 0u, 0));
                    }
#pragma unroll
                    for (int i = 0; i < PER; ++i) v[i] += (float)r[i];
                }
#pragma unroll
                for (int i = 0; i < PER; ++i) {
                    const T o = (T)((a.relu && !(v[i] > 0.0f)) ? 0.0f : v[i]);
                    if constexpr (sizeof(T) == 2) __builtin_amdgcn_raw_buffer_store_b16(__builtin_bit_cast(uint16_t, o), yrs, off[i], 0u, 0);
                    else __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(uint32_t, o), yrs, off[i], 0u, 0);
                }
            } else {
                typedef T Piece __attribute__((ext_vector_type(EPP)));
                if (a.res) {
#pragma unroll
                    for (int p = 0; p < NP; ++p) {
                        cl_u4 q;
                        if constexpr (EARLY) q = resv[(ni * AM + mi) * NP + p];
                        else q = res_load(e.w, mi, p);
                        const Piece r = __builtin_bit_cast(Piece, q);
#pragma unroll
                        for (int j = 0; j < EPP; ++j) v[p * EPP + j] += (float)r[j];
                    }
                }
                cl_u4 o[NP];
#pragma unroll
                for (int p = 0; p < NP; ++p) {
                    Piece q;
#pragma unroll
                    for (int j = 0; j < EPP; ++j) q[j] = (T)((a.relu && !(v[p * EPP + j] > 0.0f)) ? 0.0f : v[p * EPP + j]);
                    o[p] = __builtin_bit_cast(cl_u4, q);
                }
                auto store = [&](cl_u4 q, int at, int p) __attribute__((always_inline)) {
                    const int ch = piece_channel(mi, p);
                    const uint32_t off = ch < a.cout && at != (int)kClOutOfRange ? (uint32_t)(at + ch * (int)sizeof(T)) : kClOutOfRange;
                    __builtin_amdgcn_raw_buffer_store_b128(q, yrs, off, 0u, 0);
                };
                if constexpr (NP == 1) {
                    store(o[0], e.z, 0);
                } else {
                    // neighbouring lanes exchange a piece, so that a store takes 64 bytes side by side of one pixel, not 32 of two
                    auto other = [](uint32_t q) __attribute__((always_inline)) { return (uint32_t)__builtin_amdgcn_mov_dpp((int)q, 0xb1, 0xf, 0xf, true); };
                    const bool odd_lane = (lane & 1) != 0;
                    const int theirs = (int)other((uint32_t)e.z), even = odd_lane ? theirs : e.z, odd_at = odd_lane ? e.z : theirs;
#pragma unroll
                    for (int p = 0; p < NP; p += 2) {
                        cl_u4 first, second;
#pragma unroll
                        for (int j = 0; j < 4; ++j) {
                            const uint32_t got = other(odd_lane ? o[p][j] : o[p + 1][j]);
                            first[j] = odd_lane ? got : o[p][j];
                            second[j] = odd_lane ? o[p + 1][j] : got;
                        }
                        store(first, even, p + (odd_lane ? 1 : 0));
                        store(second, odd_at, p + (odd_lane ? 1 : 0));
                    }
                }
            }
        }
    }
}

template <typename T, int RB, int MI, int NI, int S, int KG, int MODE>
hipError_t launch_cl_tile(const ClArgs& a, hipStream_t s) {
    using C = ClCfg<T, RB, MI, NI, S, KG>;
    // (more than 64 KB of dynamic LDS has to be asked for once per kernel)
    static const hipError_t attr = C::LDS <= 65536 ? hipSuccess
                                                   : hipFuncSetAttribute((const void*)cl_conv_kernel<T, RB, MI, NI, S, KG, MODE>,
                                                                         hipFuncAttributeMaxDynamicSharedMemorySize, C::LDS);
    if (attr != hipSuccess) return attr;
    const unsigned grid = (unsigned)((a.tiles + 7) / 8 * 8);
    CADNN_LAUNCH((cl_conv_kernel<T, RB, MI, NI, S, KG, MODE>), dim3(grid), dim3(256 * KG), (size_t)C::LDS, s, a);
    return hipGetLastError();
}

template <typename T, int RB, int MODE>
hipError_t launch_cl_rb(const ClArgs& a, const ClVariant& v, hipStream_t s) {
    if (v.kg == 2) {
        // (layer calls take the cost rule's pick, which is never one of these in 2-byte storage)
        if constexpr (sizeof(T) == 2 && MODE == CL_PLANES) return hipErrorInvalidValue;
        else return v.ni == 2 ? launch_cl_tile<T, RB, 1, 2, 2, 2, MODE>(a, s) : launch_cl_tile<T, RB, 1, 1, 3, 2, MODE>(a, s);
    }
    if (v.mi == 2) return v.ni == 2 ? launch_cl_tile<T, RB, 2, 2, 2, 1, MODE>(a, s) : launch_cl_tile<T, RB, 2, 1, 3, 1, MODE>(a, s);
    if (v.ni == 2) return launch_cl_tile<T, RB, 1, 2, 3, 1, MODE>(a, s);
    return v.s == 3 ? launch_cl_tile<T, RB, 1, 1, 3, 1, MODE>(a, s) : launch_cl_tile<T, RB, 1, 1, 4, 1, MODE>(a, s);
}

template <typename T, int MODE>
hipError_t launch_cl_type(const ClArgs& a, const ClVariant& v, int rb, hipStream_t s) {
    return rb == 128 ? launch_cl_rb<T, 128, MODE>(a, v, s) : launch_cl_rb<T, 64, MODE>(a, v, s);
}

ClTensorArg tensor_arg(const ClDesc& d, int n, size_t e, int stride, int r0, int c0) {
    ClTensorArg t;
    // (every access lies inside: a slice of a concatenation ends with its last pixel, and a first layer's steps
    // end with its filter rows, or 8 bytes behind them, which the region has room for)
    t.span = (uint32_t)((int64_t)n * d.image * (int64_t)e);
    t.img = (int)(d.image * (int64_t)e);
    t.row = (int)(d.row * (int64_t)e) * stride;
    t.col = (int)(d.pix * (int64_t)e) * stride;
    t.org = (int)(((int64_t)d.origin + (int64_t)r0 * d.row + (int64_t)c0 * d.pix) * (int64_t)e);
    return t;
}

}  // namespace

const std::vector<ClVariant>& all_cl_variants() {
    static const std::vector<ClVariant> v = {
        {"cl_mfma_128x128_s2", 2, 2, 2, 1, 1}, {"cl_mfma_128x64_s3", 2, 1, 3, 1, 1}, {"cl_mfma_64x128_s3", 1, 2, 3, 1, 1},
        {"cl_mfma_64x64_s3", 1, 1, 3, 1, 1}, {"cl_mfma_64x64_s4", 1, 1, 4, 1, 1}, {"cl_mfma_64x64_s3k2", 1, 1, 3, 2, 1},
        {"cl_mfma_64x64_s3k4", 1, 1, 3, 4, 1}, {"cl_mfma_64x64_s4k4", 1, 1, 4, 4, 1}, {"cl_mfma_64x64_s3g2", 1, 1, 3, 1, 2},
        {"cl_mfma_64x64_s3g2k2", 1, 1, 3, 2, 2}, {"cl_mfma_64x64_s3g2k4", 1, 1, 3, 4, 2}, {"cl_mfma_64x128_s2g2", 1, 2, 2, 1, 2},
        {"cl_mfma_16x16_w8", 0, 0, 0, 1, 1, 1, 1}, {"cl_mfma_16x32_w8", 0, 0, 0, 1, 1, 1, 2}, {"cl_mfma_32x16_w8", 0, 0, 0, 1, 1, 2, 1},
        {"cl_mfma_32x32_w8", 0, 0, 0, 1, 1, 2, 2},
    };
    return v;
}

constexpr int64_t kNumCus = 256, kLdsPerCu = 160 * 1024;

static int64_t cl_tiles(const ClVariant& v, int64_t pixels, int cout) {
    return ((pixels + v.tn() - 1) / v.tn()) * ((cout + v.tm() - 1) / v.tm());
}

bool cl_variant_fits(const ClVariant& v, const ClPlan& plan, int64_t pixels, int cout) {
    if (v.mi == 2 && cout <= 64) return false;
    if (cl_tiles(v, pixels, cout) * v.sk >= (1 << 28)) return false;
    if (pixels >= (1 << 30)) return false;      // (32-bit pixel arithmetic)
    if (v.bm) return plan.elem == 2 && plan.maps && !plan.stem;
    const int slices = v.sk * v.kg, per = (plan.steps + slices - 1) / slices;
    if (v.sk == 1) return v.kg == 1 || plan.steps >= 2 * v.kg;
    // every slice gets at least two steps and none is empty; the scratch stays below 256 MiB
    if (per < 2 || (slices - 1) * per >= plan.steps) return false;
    const int64_t tiles = cl_tiles(v, pixels, cout);
    return tiles <= 512 && tiles * v.sk * v.mi * v.ni * 16384 <= (256ll << 20);
}

void cl_split_scratch(const ClVariant& v, int64_t pixels, int cout, size_t* part_bytes, size_t* count_bytes) {
    const int64_t tiles = v.sk > 1 ? cl_tiles(v, pixels, cout) : 0;
    *part_bytes = (size_t)(tiles * v.sk * v.mi * v.ni * 16384);
    *count_bytes = (size_t)tiles * 4;
}

cadnn_status cl_prepare_variant(const ClVariant& v, ClPlan* plan, int64_t pixels, int cout) {
    if (v.sk <= 1) return CADNN_OK;
    size_t part = 0, count = 0;
    cl_split_scratch(v, pixels, cout, &part, &count);
    // what the plan has is replaced only when all of the new is there: the variant in use keeps its scratch
    DevBuf more_part, more_count;
    cadnn_status st = CADNN_OK;
    if (plan->part.bytes < part && (st = more_part.alloc(part, false)) != CADNN_OK) return st;
    if (plan->count.bytes < count) {
        if ((st = more_count.alloc(count, true)) != CADNN_OK) return st;
        // (the zeros are written on the null stream, which a stream of the caller's need not wait for)
        CADNN_HIP(hipDeviceSynchronize());
    }
    if (more_part.p) plan->part.swap(more_part);
    if (more_count.p) plan->count.swap(more_count);
    return CADNN_OK;
}

// The cost of a layer in clocks, up to what is the same for all tiles: rounds of as many workgroups as fit on
// a CU (LDS, and the registers the kernel is bound to), each with a start and an end that grow with the tile and
// with how many run at once, and steps that take a fixed time while a workgroup has the CU to itself
// (the latency of loads that run two stages ahead) and the CU's rate when it does not.  The
// constants are fitted to the times of every variant, in fp16 on 387 layers (ResNet-50 at 1, 8, 16 and 32 images, MobileNet-V2
// at 16, VGG-16 at 1, Inception-V3 at 4), the tiles taken 1.7 % slower in sum than each layer's best; in fp32 on 190 layers (ResNet-50 at 1, 2,
// 4, 8, VGG-16 at 1 and 2, Inception-V3 at 1 and 3, both MobileNets): 0.3 %, against 8.1 % with constants from fp32 products.
// Timed inside the pass, with the kernels as they are now: 3.5 % on 516 fp16 layers (ResNet-50 at 1 to 8 images, MobileNet-V2 at 4 and 16,
// Inception-V3 at 1 and 2, VGG-16), 1.9 % on 254 fp32 ones (ResNet-50 at 2, 4 and 8, VGG-16 at 4, Inception-V3 at 3).  Four stages in fp32 are
// the best of 3 of those 254 and this rule never takes them: a pin and tuning do.  Steps of 64 bytes with two groups have a constant from one
// layer, as they cost more alone than inside a net: 16 -> 58 7x7 on 28 x 28 as a call 17.7 us split in four, 20.2 in two of two groups.
// Two groups of waves pay in fp32 where a workgroup has the CU to itself: 128 -> 128 3x3 on 8 images of 28 x 28 19.2 -> 16.9 us,
// 512 -> 512 3x3 on 14 x 14 (split in four as well) 20.8 -> 17.9.  In fp16 a step is bound by the way into LDS, and what
// they gain on such a layer (7.3 -> 6.5 us launched on its own) is lost again between the launches of a graph: ResNet-50 at 8 images 426 -> 435 us a
// pass.  So in 2-byte storage neither this rule nor tuning, which times layers alone, takes them; a pin does.
// Small tiles (conv_cl_small.hip) are a start, a launch that grows with the workgroups, and their operands at 18 bytes a clock;
// in graphs of equal layers at one image, us a layer, best large tile / best small one: 256 -> 256 3x3 on 14 x 14 8.6 / 7.0, 1024 -> 256
// 1x1 5.5 / 4.0, 128 -> 128 3x3 on 28 x 28 7.2 / 6.4, 2048 -> 512 1x1 on 7 x 7 7.4 / 6.2; 256 -> 1024 1x1 5.9 / 6.7, 64 -> 256 1x1 on
// 56 x 56 4.3 / 8.8; at 4 images 1024 -> 256 5.7 / 5.4, 256 -> 256 3x3 9.1 / 10.7.  Of the 516 layers 269 take one, 3.3 % slower in sum than
// the best (the others 3.7 %).  Four stages pay where workgroups are alone or two to a CU and the K loop is long; there is no use for more: six and eight
// measured the same.
struct ClCost {
    double matrix, bytes;           // the CU's rate: clocks of a 64 x 64 tile's step of 128 bytes, bytes a clock
    double alone3, alone4, wider;   // a step alone on the CU, with three and four stages; how it grows with the tile
    double narrow;                  // ... and shrinks with the step
    double start, tile;             // of a round, of every workgroup of it and 64 x 64 tile
    double split, slice;            // K split over workgroups
    double group_step, group_tile, group, group64;      // two groups of waves; of steps of 128 and of 64 bytes
};

const ClVariant* cl_pick(int cout, const ClPlan& plan, int64_t pixels, bool f16) {
    static const ClCost cost16 = {21.5, 47, 642, 630, 0.25, 0, 367, 3370, 4960, 871, 1, 1, 0, 0};
    static const ClCost cost32 = {146, 27.8, 934, 1609, 1.83, 0.32, 172, 4055, 2557, 1246, 1.06, 1.08, 446, 2000};
    const ClCost& k = f16 ? cost16 : cost32;
    const ClVariant* best = nullptr;
    double best_cost = 0.0;
    for (const ClVariant& v : all_cl_variants()) {
        if (!cl_variant_fits(v, plan, pixels, cout)) continue;
        const int64_t blocks = cl_tiles(v, pixels, cout) * v.sk;
        if (v.bm) {
            const double bytes = (double)plan.steps * plan.rb * (v.tm() + v.tn());      // a workgroup's operands
            const double cost = 3170.0 + 12.0 * (double)blocks + (double)((blocks + kNumCus - 1) / kNumCus) * bytes / 18.0;
            if (!best || cost < best_cost) { best = &v; best_cost = cost; }
            continue;
        }
        if (v.kg == 2 && f16) continue;
        const int slices = v.sk * v.kg, steps = (plan.steps + slices - 1) / slices;
        if (v.s == 4 && (blocks > 2 * kNumCus || steps < 4)) continue;
        const int size = v.mi * v.ni, weights = cl_weight_bytes(plan.rb, f16 ? 2 : 4);
        const int stage = (v.mi * weights * 64 + 4095) / 4096 * 4096 + 64 * v.ni * plan.rb;
        const int lds = v.kg * v.s * stage + 64 * v.ni * 16 + 64 * v.mi * 8 + 16;
        const int64_t per_cu = std::min<int64_t>(kLdsPerCu / lds, (size == 1 ? 4 : 2) / v.kg);
        const double rate = std::max(k.matrix * size * v.kg * plan.rb / 128.0, 64 * (v.mi * weights + v.ni * plan.rb) * v.kg / k.bytes);
        const double alone = std::max(rate, (v.s == 4 ? k.alone4 : k.alone3) * (1.0 + k.wider * (size - 1)) * std::pow(plan.rb / 128.0, k.narrow) *
                                                (v.kg == 2 ? k.group_step : 1.0));
        auto round = [&](int64_t n) {
            return n == 0 ? 0.0 : k.start + k.tile * size * (double)n * (v.kg == 2 ? k.group_tile : 1.0) + steps * std::max(alone, rate * (double)n);
        };
        const int64_t in_cu = (blocks + kNumCus - 1) / kNumCus;
        const double cost = (double)(in_cu / per_cu) * round(per_cu) + round(in_cu % per_cu) + (v.sk > 1 ? k.split + k.slice * v.sk : 0.0) +
                            (v.kg == 2 ? (plan.rb == 64 ? k.group64 : k.group) : 0.0);
        if (!best || cost < best_cost) { best = &v; best_cost = cost; }
    }
    return best;
}

cadnn_status launch_cl_conv(const ClConv& c, const ClVariant& v, bool f16, hipStream_t s) {
    const ClPlan& p = *c.plan;
    const size_t e = f16 ? 2 : 4;
    ClArgs a{};
    a.w = (const char*)c.w;
    a.x = (const char*)c.x;
    a.y = (char*)c.y;
    a.res = (const char*)c.residual;
    a.bias = c.bias;
    a.xt = tensor_arg(c.xd, c.n, e, c.stride, -c.pad, -c.pad);
    if (!c.planes) a.yt = tensor_arg(c.yd, c.n, e, 1, 0, 0);
    if (c.residual && !c.planes) a.rt = tensor_arg(c.rd, c.n, e, 1, 0, 0);
    if (p.steps2 > 0) {
        a.x2 = (const char*)c.x2;
        a.bias2 = c.bias2;
        a.x2t = tensor_arg(c.x2d, c.n, e, c.stride2, 0, 0);
    }
    a.wspan = (uint32_t)c.w_bytes;
    a.hw = c.yd.h * c.yd.w;
    a.total = c.n * a.hw;
    a.ow = c.yd.w;
    a.cout = c.cout;
    a.relu = c.relu ? 1 : 0;
    a.steps_tap = p.steps_tap;
    a.steps1 = p.taps * p.steps_tap;
    a.steps = p.steps;
    a.tiles_m = (c.cout + v.tm() - 1) / v.tm();
    a.sk = v.sk;
    a.log_sk = v.sk == 4 ? 2 : v.sk == 2 ? 1 : 0;
    a.ntaps = p.taps;
    a.row_bytes = p.stem ? p.row_bytes : p.rb;
    a.tiles = (int)cl_tiles(v, a.total, c.cout) * v.sk;
    a.per_slice = (p.steps + v.sk * v.kg - 1) / (v.sk * v.kg);
    a.per_die = (a.tiles + 7) / 8;
    auto magic = [](int d) { return (uint32_t)(((1ull << 32) + (uint64_t)d - 1) / (uint64_t)d); };
    a.magic_hw = magic(a.hw);
    a.magic_ow = magic(a.ow);
    a.magic_tm = magic(a.tiles_m);
    a.magic_st = magic(a.steps_tap);
    a.part = c.part;
    a.count = c.count;
    for (int t = 0; t < p.taps; ++t)
        a.tap_off[t] = (int)(((int64_t)p.tap_r[t] * c.xd.row + (int64_t)p.tap_c[t] * c.xd.pix) * (int64_t)e);
    hipError_t err;
    if (v.bm) {
        err = launch_cl_small(a, v, p.rb, s);
    } else if (c.planes) {
        // one pixel of one channel after the other; images follow each other
        a.yt.img = (int)((int64_t)c.cout * a.hw * (int64_t)e);
        a.yt.row = (int)(a.ow * e);
        a.yt.col = (int)e;
        a.yt.org = 0;
        a.yt.span = (uint32_t)((int64_t)c.n * a.yt.img);
        a.plane = (int)(a.hw * (int64_t)e);
        if (c.residual) a.rt = a.yt;
        err = f16 ? launch_cl_type<_Float16, CL_PLANES>(a, v, p.rb, s) : launch_cl_type<float, CL_PLANES>(a, v, p.rb, s);
    } else if (a.row_bytes % 16 != 0) {
        err = launch_cl_type<_Float16, CL_ODD_ROW>(a, v, p.rb, s);
    } else {
        err = f16 ? launch_cl_type<_Float16, CL_MAPS>(a, v, p.rb, s) : launch_cl_type<float, CL_MAPS>(a, v, p.rb, s);
    }
    CADNN_HIP(err);
    return CADNN_OK;
}

cadnn_status cl_plan_shape(const cadnn_weights* w, const cadnn_weights* shortcut, int rb, bool stem, ClPlan* plan,
                           std::vector<int>* tap_of) {
    const size_t e = w->elem();
    const int taps_all = w->kh * w->kw, kpr = rb / (int)e;      // k per step
    plan->rb = rb;
    plan->elem = (int)e;
    plan->stem = stem;
    plan->taps = 0;
    std::vector<int> tap_index((size_t)taps_all, -1);
    if (stem) {
        // a step is one filter row: kw pixels of 4 channels
        if (w->cin > 4 || w->kw * 4 > kpr || w->kh > kClMaxTaps) return fail(CADNN_EINVAL, "cadnn_net: not a first layer of few channels");
        for (int r = 0; r < w->kh; ++r) { plan->tap_r[r] = r; plan->tap_c[r] = 0; }
        plan->taps = w->kh;
        plan->steps_tap = 1;
        plan->row_bytes = w->kw * 4 * (int)e;
    } else {
        std::vector<char> used((size_t)taps_all, 0);
        // (most filters have weights at all of them, which a few columns show: the rest need not be divided)
        int unused = taps_all;
        for (size_t j = 0; j < w->col_idx.size() && unused > 0; ++j) {
            char& u = used[(size_t)(w->col_idx[j] % taps_all)];
            unused -= u ? 0 : 1;
            u = 1;
        }
        for (int t = 0; t < taps_all; ++t) {
            if (!used[(size_t)t]) continue;
            if (plan->taps == kClMaxTaps) return fail(CADNN_EUNSUPPORTED, "cadnn_net: more than %d filter taps", kClMaxTaps);
            tap_index[(size_t)t] = plan->taps;
            plan->tap_r[plan->taps] = t / w->kw;
            plan->tap_c[plan->taps] = t % w->kw;
            ++plan->taps;
        }
        if (plan->taps == 0) {          // nothing but zeros: one tap of them
            tap_index[0] = 0;
            plan->tap_r[0] = plan->tap_c[0] = 0;
            plan->taps = 1;
        }
        plan->steps_tap = (w->cin + kpr - 1) / kpr;
    }
    plan->steps2 = shortcut ? (shortcut->cin + kpr - 1) / kpr : 0;
    plan->steps = plan->taps * plan->steps_tap + plan->steps2;
    if (tap_of) tap_of->swap(tap_index);
    return CADNN_OK;
}

// The steps of a layer's K (or of a fused shortcut's) in the order of a plan: a chunk of input channels fills one step of each tap
// (of a first layer, all its channels one step of each filter row).
struct ClSteps {
    int channels, chunks, slots;        // of a chunk, of the layer; steps of a chunk
    int first, stride;                  // of chunk c: steps first + slot * stride + c
    std::vector<int> place;             // of column k of a chunk: slot * k per step + k in the step
};

typedef float cl_host_f4 __attribute__((ext_vector_type(4)));
typedef uint32_t cl_host_u4 __attribute__((ext_vector_type(4)));
typedef uint16_t cl_host_h8 __attribute__((ext_vector_type(8)));

// cl_split_weight of four weights at once, each part in the upper half of its place; false where one is to be kept whole.
static bool cl_split_four(cl_host_f4 v, cl_host_u4 part[3]) {
    const cl_host_f4 s = v * kClPartScale;
    const cl_host_u4 u = __builtin_bit_cast(cl_host_u4, s);
    const cl_host_u4 size = u & 0x7fffffffu;
    const cl_host_u4 top = (u + 0x7fffu + (u >> 16 & 1u)) & 0xffff0000u;
    const cl_host_f4 rest = s - __builtin_bit_cast(cl_host_f4, top);
    const cl_host_u4 r = __builtin_bit_cast(cl_host_u4, rest), mid = (r + 0x7fffu + (r >> 16 & 1u)) & 0xffff0000u;
    part[0] = top;
    part[1] = mid;
    part[2] = __builtin_bit_cast(cl_host_u4, rest - __builtin_bit_cast(cl_host_f4, mid));
    const uint32_t a = std::max(size[0], size[1]), b = std::max(size[2], size[3]);
    return std::max(a, b) < 0x7f7f8000u;
}

// 4-byte weights: 64 output channels of a chunk at a time, spread over its steps as floats (a row after the other), then taken apart
// and written whole, a step after the other.  (Written weight by weight, the pieces of a row lie 1 KB apart, in four sets of the
// first cache.  build_net of ResNet-50 in fp32 82 -> 77 ms; 72 with 4-byte weights, a third less to write and to upload.)
static void cl_put_split(const cadnn_weights* src, const ClSteps& k, int kpr, int steps, char* img) {
    const int taps = src->kh * src->kw;
    const size_t width = (size_t)k.slots * kpr, step_bytes = (size_t)64 * cl_weight_bytes(kpr * 4, 4);
    std::vector<int> row_of((size_t)src->cout);
    for (int i = 0; i < src->cout; ++i) row_of[(size_t)src->perm[(size_t)i]] = i;
    std::vector<float> rows(64 * width);
    for (int co0 = 0; co0 < src->cout; co0 += 64) {
        const int have = std::min(64, src->cout - co0);
        char* const block = img + (size_t)(co0 / 64) * steps * step_bytes;
        int32_t at[64], end[64];
        for (int r = 0; r < have; ++r) {
            at[r] = src->row_ptr[(size_t)row_of[(size_t)(co0 + r)]];
            end[r] = src->row_ptr[(size_t)row_of[(size_t)(co0 + r)] + 1];
        }
        for (int c = 0; c < k.chunks; ++c) {
            const int32_t begin = (int32_t)((int64_t)c * k.channels * taps);
            const int32_t behind = (int32_t)std::min<int64_t>((int64_t)(c + 1) * k.channels * taps, (int64_t)src->cin * taps);
            std::fill(rows.begin(), rows.end(), 0.0f);
            for (int r = 0; r < have; ++r) {
                int32_t j = at[r];
                for (; j < end[r] && src->col_idx[(size_t)j] < behind; ++j)
                    rows[(size_t)r * width + (size_t)k.place[(size_t)(src->col_idx[(size_t)j] - begin)]] = src->vals[(size_t)j];
                at[r] = j;
            }
            for (int slot = 0; slot < k.slots; ++slot) {
                char* const step = block + (size_t)(k.first + slot * k.stride + c) * step_bytes;
                for (int k0 = 0; k0 < kpr; k0 += k0 % 16 == 0 ? 4 : 12)         // (eight k of one half of a wave: k0 + {0..3, 8..11})
                    for (int r = 0; r < 64; ++r) {
                        const float* const v = &rows[(size_t)r * width + (size_t)(slot * kpr + k0)];
                        cl_host_f4 lo, hi;
                        std::memcpy(&lo, v, 16);
                        std::memcpy(&hi, v + 8, 16);
                        cl_host_u4 lo_parts[3], hi_parts[3];
                        uint16_t part[3][8];
                        if (cl_split_four(lo, lo_parts) && cl_split_four(hi, hi_parts)) {
                            for (int p = 0; p < 3; ++p) {
                                const auto eight = __builtin_shufflevector(__builtin_bit_cast(cl_host_h8, lo_parts[p]), __builtin_bit_cast(cl_host_h8, hi_parts[p]),
                                                                           1, 3, 5, 7, 9, 11, 13, 15);
                                std::memcpy(part[p], &eight, 16);
                            }
                        } else {
                            for (int i = 0; i < 8; ++i) {
                                uint16_t one[3];
                                cl_split_weight(v[i / 4 * 8 + i % 4], one);
                                for (int p = 0; p < 3; ++p) part[p][i] = one[p];
                            }
                        }
                        for (int p = 0; p < 3; ++p) std::memcpy(step + cl_split_offset(k0, p, r), part[p], 16);
                    }
            }
        }
    }
}

cadnn_status cl_build_plan(const cadnn_weights* w, const cadnn_weights* shortcut, int rb, bool stem, ClPlan* plan, std::vector<char>* image) {
    const size_t e = w->elem();
    const int taps_all = w->kh * w->kw, kpr = rb / (int)e;
    std::vector<int> tap_index;
    const cadnn_status st = cl_plan_shape(w, shortcut, rb, stem, plan, &tap_index);
    if (st != CADNN_OK) return st;
    const size_t row_bytes = (size_t)cl_weight_bytes(rb, (int)e), bytes = cl_plan_bytes(w->cout, *plan, (int)e);
    if (bytes >= kClMaxWeightBytes) return fail(CADNN_EUNSUPPORTED, "cadnn_net: weight matrix of 2 GiB or more");
    // where k lies: the divisions once per k and not once per weight
    ClSteps main, more;
    main.channels = stem ? w->cin : std::min(kpr, w->cin);
    main.chunks = stem ? 1 : plan->steps_tap;
    main.slots = plan->taps;
    main.first = 0;
    main.stride = plan->steps_tap;
    main.place.resize((size_t)main.channels * taps_all);
    for (int ci = 0; ci < main.channels; ++ci)
        for (int t = 0; t < taps_all; ++t)
            main.place[(size_t)ci * taps_all + t] = stem ? t / w->kw * kpr + t % w->kw * 4 + ci : std::max(tap_index[(size_t)t], 0) * kpr + ci;
    if (shortcut) {
        more.channels = std::min(kpr, shortcut->cin);
        more.chunks = plan->steps2;
        more.slots = more.stride = 1;
        more.first = plan->taps * plan->steps_tap;
        more.place.resize((size_t)more.channels);
        for (int ci = 0; ci < more.channels; ++ci) more.place[(size_t)ci] = ci;
    }
    if (e == 4) {
        // (all but the rows of a last half tile is written)
        if (image->size() < bytes) image->resize(bytes);
        const size_t written = (size_t)((w->cout + 63) / 64) * plan->steps * 64 * row_bytes;
        std::memset(image->data() + written, 0, bytes - written);
        cl_put_split(w, main, kpr, plan->steps, image->data());
        if (shortcut) cl_put_split(shortcut, more, kpr, plan->steps, image->data());
        return plan->w.upload(image->data(), bytes);
    }
    image->assign(bytes, 0);
    char* const img = image->data();
    // where k lies in the rows of block 0 (row 0's place of it)
    std::vector<size_t> place;
    std::vector<int> row_of;
    auto put = [&](const cadnn_weights* src, const ClSteps& k) {
        place.resize((size_t)src->cin * src->kh * src->kw);
        for (size_t i = 0; i < place.size(); ++i) {
            const size_t c = i / k.place.size();
            const int at = k.place[i - c * k.place.size()], slot = at / kpr;
            place[i] = (size_t)(k.first + slot * k.stride + (int)c) * 64 * row_bytes + (size_t)(at - slot * kpr) * 2;
        }
        // (in the order of channels: a block of 64 is put together while it is in the cache)
        row_of.resize((size_t)src->cout);
        for (int i = 0; i < src->cout; ++i) row_of[(size_t)src->perm[(size_t)i]] = i;
        for (int co = 0; co < src->cout; ++co) {
            const int i = row_of[(size_t)co], r = cl_weight_row(co, 2), sw = rb == 128 ? (r >> 1) & 7 : (r >> 2) & 3;
            char* const row = img + (size_t)(co / 64) * plan->steps * 64 * row_bytes + (size_t)r * (size_t)rb;
            // (a step is a multiple of 128 bytes, so the piece's bits of the sum are those of the place in the row)
            for (int32_t j = src->row_ptr[(size_t)i]; j < src->row_ptr[(size_t)i + 1]; ++j)
                std::memcpy(row + (place[(size_t)src->col_idx[(size_t)j]] ^ (size_t)(sw * 16)), &src->vals16[(size_t)j], 2);
        }
    };
    put(w, main);
    if (shortcut) put(shortcut, more);
    return plan->w.upload(img, bytes);
}

}  // namespace cadnn
