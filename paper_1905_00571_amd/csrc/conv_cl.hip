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
//   * S stage buffers; a stage's loads are issued S - 1 stages ahead, right behind the barrier that says
//     every wave is done with the buffer: one barrier and one counted wait per stage.
//   * Padding is a zero halo in memory, so no tap is ever tested.
//   * A fused 1x1 projection shortcut (paper Section 4, layer fusion) is more K steps on a second tensor.
//   * The epilogue goes through LDS, [pixel][channel]: residual rows come in and finished rows go out as
//     16-byte pieces of whole pixels; bias, residual and ReLU in fp32, one rounding.
//   * fp32 storage takes v_mfma_f32_32x32x2_f32 on the same bytes: a 16-byte piece is four k of one lane,
//     consumed by four instructions (both operands permute k the same way).
//   * K may be split over `sk` workgroups per tile (partial tiles at device scope, the last to arrive adds
//     them in slice order and finishes): for layers whose tiles leave most of the chip idle.
//   * Workgroups are numbered so that one die (workgroup id % 8) owns a contiguous run of tiles with the
//     output-channel tiles of one pixel tile next to each other: its L2 serves the re-reads.
#include <cmath>
#include <cstring>

#include "channels_last.h"

namespace cadnn {

namespace {

constexpr uint32_t kClOutOfRange = 0x7ffffff0u;

typedef _Float16 cl_h8 __attribute__((ext_vector_type(8)));
typedef _Float16 cl_h4 __attribute__((ext_vector_type(4)));
typedef float cl_f4 __attribute__((ext_vector_type(4)));
typedef float cl_f16v __attribute__((ext_vector_type(16)));
typedef uint32_t cl_u4 __attribute__((ext_vector_type(4)));
typedef uint32_t cl_u2 __attribute__((ext_vector_type(2)));

// Offsets and pitches in bytes.
struct ClTensorArg {
    uint32_t span;              // bytes behind the base pointer
    int img, row, col, org;     // per image, per OUTPUT row and column (strides included), first
};
struct ClArgs {
    const char* w;
    const char* x;
    const char* x2;
    char* y;
    const char* res;
    const float* bias;
    const float* bias2;
    float* part;
    int* count;
    ClTensorArg xt, x2t, yt, rt;
    uint32_t wspan;
    int total, hw, ow, cout, relu;
    int steps_tap, steps1, steps, tiles_m, tiles, sk;
    int tap_off[kClMaxTaps];
};

// 16 bytes per lane from memory to LDS (lane l: lds + 16 l).  The wait for it is the caller's.
__device__ __forceinline__ void cl_dma(cl_u4 rsrc, uint32_t voff, uint32_t soff, uint32_t lds) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds"
                 :: "s"(lds), "v"(voff), "s"(rsrc), "s"(soff) : "memory");
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

template <typename T, int RB, int MI, int NI, int S>
struct ClCfg {
    static constexpr int TM = 64 * MI, TN = 64 * NI;
    static constexpr int STAGE = (TM + TN) * RB;
    static constexpr int PITCH = TM * (int)sizeof(T) + 16;
    static constexpr int MAIN = S * STAGE > TN * PITCH ? S * STAGE : TN * PITCH;
    static constexpr int LDS = MAIN + TN * 16 + TM * 4;
};

template <typename T, int RB, int MI, int NI, int S>
__global__ __launch_bounds__(256) void cl_conv_kernel(const ClArgs a) {
    using C = ClCfg<T, RB, MI, NI, S>;
    constexpr int TM = C::TM, TN = C::TN, STAGE = C::STAGE, PITCH = C::PITCH;
    constexpr int RPL = 1024 / RB;                 // rows one wave-load fills
    constexpr int LA = TM * RB / 4096, LB = TN * RB / 4096;      // loads per thread and stage
    constexpr int PIECES = RB / 16;
    constexpr int EPP = 16 / (int)sizeof(T);       // elements per 16-byte piece
    constexpr int KS = RB / 32;                    // 32-byte halves pairs: MFMA groups per stage
    extern __shared__ __attribute__((aligned(16))) char cl_smem[];
    int4* ptab = (int4*)(cl_smem + C::MAIN);       // per pixel of the tile: byte offsets in x, x2, y, residual
    float* bl = (float*)(cl_smem + C::MAIN + TN * 16);
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)cl_smem;

    // ---- which tile: dies own contiguous runs
    const int per_die = (a.tiles + 7) >> 3;
    const int t = ((int)blockIdx.x & 7) * per_die + ((int)blockIdx.x >> 3);
    if (((int)blockIdx.x >> 3) >= per_die || t >= a.tiles) return;
    const int mt = __builtin_amdgcn_readfirstlane(t % a.tiles_m), rest = t / a.tiles_m;
    const int z = __builtin_amdgcn_readfirstlane(rest % a.sk), nt = __builtin_amdgcn_readfirstlane(rest / a.sk);
    const int m0 = mt * TM, n0 = nt * TN;

    const int tid = (int)threadIdx.x, lane = tid & 63;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wv >> 1, wn = wv & 1;

    if (tid < TN) {
        const int Q = n0 + tid;
        int4 e = make_int4((int)kClOutOfRange, (int)kClOutOfRange, (int)kClOutOfRange, (int)kClOutOfRange);
        if (Q < a.total) {
            const int img = Q / a.hw, q = Q - img * a.hw;
            const int oh = q / a.ow, ow = q - oh * a.ow;
            e.x = img * a.xt.img + oh * a.xt.row + ow * a.xt.col + a.xt.org;
            e.y = img * a.x2t.img + oh * a.x2t.row + ow * a.x2t.col + a.x2t.org;
            e.z = img * a.yt.img + oh * a.yt.row + ow * a.yt.col + a.yt.org;
            e.w = img * a.rt.img + oh * a.rt.row + ow * a.rt.col + a.rt.org;
        }
        ptab[tid] = e;
    }
    if (tid < TM) {
        const int co = m0 + tid;
        bl[tid] = co < a.cout ? (a.bias ? a.bias[co] : 0.0f) + (a.bias2 ? a.bias2[co] : 0.0f) : 0.0f;
    }
    __syncthreads();

    // ---- sources: this thread's row (of each group of rows) and 16-byte piece
    const int lrow = lane / PIECES, lpos = lane % PIECES;
    const int sw = RB == 128 ? ((wv * RPL + lrow) >> 1) & 7 : (lrow >> 2) & 3;
    const uint32_t piece = (uint32_t)(lpos ^ sw) * 16u;
    uint32_t vb[LB];
#pragma unroll
    for (int j = 0; j < LB; ++j) {
        const int e = ptab[j * 4 * RPL + wv * RPL + lrow].x;
        vb[j] = e == (int)kClOutOfRange ? kClOutOfRange : (uint32_t)e + piece;
    }
    const uint32_t va = (uint32_t)(wv * 1024 + lane * 16);
    cl_u4 xr = cl_rsrc(a.x, a.xt.span);
    const cl_u4 wr = cl_rsrc(a.w, a.wspan);

    // ---- the residual's rows are requested up front where they fit few registers
    constexpr int CPR = TM * (int)sizeof(T) / 16, ITEMS = TN * CPR / 256;
    constexpr bool EARLY = ITEMS <= 4;
    const cl_u4 rr_ = cl_rsrc(a.res, a.rt.span);
    const __amdgpu_buffer_rsrc_t rrs = __builtin_amdgcn_make_buffer_rsrc((void*)a.res, 0, a.rt.span, 0x00020000);
    (void)rr_;
    const int ec = tid % CPR, ep = tid / CPR;                    // epilogue: this thread's piece and first pixel
    const bool ec_live = m0 + ec * EPP < a.cout;
    cl_u4 resv[EARLY ? ITEMS : 1];
    auto res_load = [&](int k) __attribute__((always_inline)) {
        const int r = ptab[ep + k * (256 / CPR)].w;
        const uint32_t off = (ec_live && r != (int)kClOutOfRange) ? (uint32_t)(r + m0 * (int)sizeof(T) + ec * 16) : kClOutOfRange;
        return __builtin_bit_cast(cl_u4, __builtin_amdgcn_raw_buffer_load_b128(rrs, off, 0u, 0));
    };
    if constexpr (EARLY) {
        if (a.res) {
#pragma unroll
            for (int k = 0; k < ITEMS; ++k) resv[k] = res_load(k);
        }
    }

    // ---- the walk over this workgroup's slice of K
    const int per_slice = __builtin_amdgcn_readfirstlane((a.steps + a.sk - 1) / a.sk);
    const int s_first = z * per_slice;
    const int steps = min(per_slice, a.steps - s_first);
    int f_left, f_tap = 0, f_todo = steps;
    uint32_t f_soff;
    uint32_t wsoff[MI];
#pragma unroll
    for (int i = 0; i < MI; ++i) wsoff[i] = (uint32_t)((mt * MI + i) * a.steps + s_first) * (64u * RB);
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
    if (s_first < a.steps1) {
        f_tap = __builtin_amdgcn_readfirstlane(s_first / a.steps_tap);
        const int at = s_first - f_tap * a.steps_tap;
        f_left = a.steps_tap - at;
        f_soff = (uint32_t)a.tap_off[f_tap] + (uint32_t)at * RB;
    } else {
        enter_shortcut(s_first - a.steps1);
    }
    const int ntaps = a.steps1 / a.steps_tap;
    const uint32_t lds_w = lds0 + (uint32_t)wv * 1024u;
    auto issue = [&](uint32_t buf) __attribute__((always_inline)) {
        const uint32_t base = lds_w + buf * STAGE;
#pragma unroll
        for (int i = 0; i < LA; ++i) {
            constexpr int PER = 64 * RB / 4096;      // loads of this thread per 64-row block
            cl_dma(wr, va, wsoff[i / PER] + (uint32_t)(i % PER) * 4096u, base + (uint32_t)i * 4096u);
        }
#pragma unroll
        for (int j = 0; j < LB; ++j) cl_dma(xr, vb[j], f_soff, base + (uint32_t)(TM * RB) + (uint32_t)j * 4096u);
#pragma unroll
        for (int i = 0; i < MI; ++i) wsoff[i] += 64u * RB;
        f_soff += RB;
        --f_todo;
        if (--f_left == 0 && f_todo > 0) {
            if (++f_tap < ntaps) {
                f_left = a.steps_tap;
                f_soff = (uint32_t)a.tap_off[f_tap];
            } else {
                enter_shortcut(0);
            }
        }
    };

    cl_f16v acc[MI][NI];
#pragma unroll
    for (int mi = 0; mi < MI; ++mi)
#pragma unroll
        for (int ni = 0; ni < NI; ++ni)
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[mi][ni][i] = 0.0f;

    // fragment addresses: row l % 32 of a 32-row block, piece 2 ks + l / 32 (permuted by the row)
    const int l31 = lane & 31, fk = lane >> 5;
    const int fs = RB == 128 ? (lane >> 1) & 7 : (lane >> 2) & 3;
    const uint32_t fa = (uint32_t)((wm * 32 * MI + l31) * RB), fb = (uint32_t)(TM * RB + (wn * 32 * NI + l31) * RB);
    const uint32_t fp = (uint32_t)((fk ^ fs) * 16);

    // loads in flight per stage and thread; a stage past the end of the slice issues none
    constexpr int L = LA + LB;
    auto wait_stage = [&](int ahead) __attribute__((always_inline)) {
        // `ahead` stages may stay in flight behind the one needed now
        if constexpr (S >= 4) { if (ahead >= 2) { asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" :: "n"(2 * L) : "memory"); return; } }
        if constexpr (S >= 3) { if (ahead >= 1) { asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" :: "n"(L) : "memory"); return; } }
        asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
    };
#pragma unroll
    for (int j = 0; j < S - 1; ++j)
        if (j < steps) issue((uint32_t)j);
    uint32_t rd = 0, wrbuf = S - 1;
    for (int s = 0; s < steps; ++s) {
        wait_stage(min(steps - 1 - s, S - 2));
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        if (s + S - 1 < steps) issue(wrbuf);
        const char* st = cl_smem + rd * STAGE;
        // (scheduling of the reads against the products is left to the compiler: everything below is straight-line)
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            const uint32_t p = fp ^ (uint32_t)(ks * 32);
            cl_u4 af[MI], bf[NI];
#pragma unroll
            for (int mi = 0; mi < MI; ++mi) af[mi] = *(const cl_u4*)(st + fa + mi * 32 * RB + p);
#pragma unroll
            for (int ni = 0; ni < NI; ++ni) bf[ni] = *(const cl_u4*)(st + fb + ni * 32 * RB + p);
#pragma unroll
            for (int mi = 0; mi < MI; ++mi)
#pragma unroll
                for (int ni = 0; ni < NI; ++ni) {
                    if constexpr (sizeof(T) == 2) {
                        acc[mi][ni] = __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(cl_h8, af[mi]),
                                                                             __builtin_bit_cast(cl_h8, bf[ni]), acc[mi][ni], 0, 0, 0);
                    } else {
#pragma unroll
                        for (int e = 0; e < 4; ++e)
                            acc[mi][ni] = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(af[mi][e]), __uint_as_float(bf[ni][e]),
                                                                               acc[mi][ni], 0, 0, 0);
                    }
                }
        }
        rd = rd + 1 == S ? 0 : rd + 1;
        wrbuf = wrbuf + 1 == S ? 0 : wrbuf + 1;
    }

    // ---- K split over workgroups: the slices of a tile meet in memory (device-scope accesses go to the level
    //      all dies share; every thread's stores are acknowledged before the arrival is counted)
    if (a.sk > 1) {
        const size_t tile_id = (size_t)nt * a.tiles_m + mt;
        float* mine = a.part + (tile_id * a.sk + z) * (size_t)(TM * TN);
#pragma unroll
        for (int mi = 0; mi < MI; ++mi)
#pragma unroll
            for (int ni = 0; ni < NI; ++ni)
#pragma unroll
                for (int i = 0; i < 16; ++i)
                    __hip_atomic_store(mine + ((mi * NI + ni) * 16 + i) * 256 + tid, acc[mi][ni][i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
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
        for (int mi = 0; mi < MI; ++mi)
#pragma unroll
            for (int ni = 0; ni < NI; ++ni)
#pragma unroll
                for (int i = 0; i < 16; ++i) acc[mi][ni][i] = 0.0f;
        for (int k = 0; k < a.sk; ++k) {
            const float* src = a.part + (tile_id * a.sk + k) * (size_t)(TM * TN);
#pragma unroll
            for (int mi = 0; mi < MI; ++mi)
#pragma unroll
                for (int ni = 0; ni < NI; ++ni)
#pragma unroll
                    for (int i = 0; i < 16; ++i)
                        acc[mi][ni][i] += __hip_atomic_load(src + ((mi * NI + ni) * 16 + i) * 256 + tid, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
    }

    // ---- epilogue.  Lane l holds, per accumulator, pixel l % 32 and channels 8 g + 4 (l / 32) + i, g, i < 4.
    __syncthreads();                        // the stage buffers are free: every wave is past its last read
    if (a.res) {
#pragma unroll
        for (int k = 0; k < ITEMS; ++k) {
            if constexpr (EARLY) *(cl_u4*)(cl_smem + (ep + k * (256 / CPR)) * PITCH + ec * 16) = resv[k];
            else *(cl_u4*)(cl_smem + (ep + k * (256 / CPR)) * PITCH + ec * 16) = res_load(k);
        }
        __syncthreads();
    }
#pragma unroll
    for (int ni = 0; ni < NI; ++ni)
#pragma unroll
        for (int mi = 0; mi < MI; ++mi)
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                const int ch = wm * 32 * MI + mi * 32 + g * 8 + fk * 4;
                char* at = cl_smem + (wn * 32 * NI + ni * 32 + l31) * PITCH + ch * (int)sizeof(T);
                const cl_f4 b = *(const cl_f4*)(bl + ch);
                float v[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) v[i] = acc[mi][ni][g * 4 + i] + b[i];
                if constexpr (sizeof(T) == 2) {
                    if (a.res) {
                        const cl_h4 r = *(const cl_h4*)at;
#pragma unroll
                        for (int i = 0; i < 4; ++i) v[i] += (float)r[i];
                    }
                    cl_h4 o;
#pragma unroll
                    for (int i = 0; i < 4; ++i) o[i] = (_Float16)((a.relu && !(v[i] > 0.0f)) ? 0.0f : v[i]);
                    *(cl_h4*)at = o;
                } else {
                    if (a.res) {
                        const cl_f4 r = *(const cl_f4*)at;
#pragma unroll
                        for (int i = 0; i < 4; ++i) v[i] += r[i];
                    }
                    cl_f4 o;
#pragma unroll
                    for (int i = 0; i < 4; ++i) o[i] = (a.relu && !(v[i] > 0.0f)) ? 0.0f : v[i];
                    *(cl_f4*)at = o;
                }
            }
    __syncthreads();
    const __amdgpu_buffer_rsrc_t yrs = __builtin_amdgcn_make_buffer_rsrc((void*)a.y, 0, a.yt.span, 0x00020000);
#pragma unroll
    for (int k = 0; k < ITEMS; ++k) {
        const int p = ep + k * (256 / CPR);
        const int yo = ptab[p].z;
        const uint32_t off = (ec_live && yo != (int)kClOutOfRange) ? (uint32_t)(yo + m0 * (int)sizeof(T) + ec * 16) : kClOutOfRange;
        const cl_u4 v = *(const cl_u4*)(cl_smem + p * PITCH + ec * 16);
        __builtin_amdgcn_raw_buffer_store_b128(v, yrs, off, 0u, 0);
    }
}

template <typename T, int RB, int MI, int NI, int S>
hipError_t launch_cl_tile(const ClArgs& a, hipStream_t s) {
    using C = ClCfg<T, RB, MI, NI, S>;
    // (more than 64 KB of dynamic LDS has to be asked for once per kernel)
    static const hipError_t attr = C::LDS <= 65536 ? hipSuccess
                                                   : hipFuncSetAttribute((const void*)cl_conv_kernel<T, RB, MI, NI, S>,
                                                                         hipFuncAttributeMaxDynamicSharedMemorySize, C::LDS);
    if (attr != hipSuccess) return attr;
    const unsigned grid = (unsigned)((a.tiles + 7) / 8 * 8);
    CADNN_LAUNCH((cl_conv_kernel<T, RB, MI, NI, S>), dim3(grid), dim3(256), (size_t)C::LDS, s, a);
    return hipGetLastError();
}

#ifndef CADNN_CL_STAGES
#define CADNN_CL_STAGES(T, RB, MI, NI) ((MI) * (NI) == 4 ? 2 : 3)
#endif
template <typename T, int RB>
hipError_t launch_cl_rb(const ClArgs& a, int mi, int ni, hipStream_t s) {
    if (mi == 2 && ni == 2) return launch_cl_tile<T, RB, 2, 2, CADNN_CL_STAGES(T, RB, 2, 2)>(a, s);
    if (mi == 2) return launch_cl_tile<T, RB, 2, 1, CADNN_CL_STAGES(T, RB, 2, 1)>(a, s);
    if (ni == 2) return launch_cl_tile<T, RB, 1, 2, CADNN_CL_STAGES(T, RB, 1, 2)>(a, s);
    return launch_cl_tile<T, RB, 1, 1, CADNN_CL_STAGES(T, RB, 1, 1)>(a, s);
}

ClTensorArg tensor_arg(const ClDesc& d, int n, size_t e, int stride, int r0, int c0) {
    ClTensorArg t;
    // (a slice of a concatenation ends where its last pixel's own channels end; the slack behind a stem's
    // packed image is part of its region)
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
        {"cl_mfma_128x128", 2, 2, 1}, {"cl_mfma_128x64", 2, 1, 1}, {"cl_mfma_64x128", 1, 2, 1}, {"cl_mfma_64x64", 1, 1, 1},
        {"cl_mfma_64x64_k2", 1, 1, 2}, {"cl_mfma_64x64_k4", 1, 1, 4}, {"cl_mfma_64x64_k8", 1, 1, 8},
        {"cl_mfma_128x64_k2", 2, 1, 2}, {"cl_mfma_128x64_k4", 2, 1, 4}, {"cl_mfma_128x128_k2", 2, 2, 2},
    };
    return v;
}

static int64_t cl_tiles(const ClVariant& v, int64_t pixels, int cout) {
    return ((pixels + 64 * v.ni - 1) / (64 * v.ni)) * ((cout + 64 * v.mi - 1) / (64 * v.mi));
}

bool cl_variant_fits(const ClVariant& v, const ClPlan& plan, int64_t pixels, int cout) {
    if (v.mi == 2 && cout <= 64) return false;
    if (cl_tiles(v, pixels, cout) * v.sk >= (1 << 28)) return false;
    if (v.sk == 1) return true;
    // every slice gets at least two steps and none is empty; the scratch stays below 256 MiB
    const int per = (plan.steps + v.sk - 1) / v.sk;
    if (per < 2 || (v.sk - 1) * per >= plan.steps) return false;
    const int64_t tiles = cl_tiles(v, pixels, cout);
    return tiles <= 512 && tiles * v.sk * v.mi * v.ni * 16384 <= (256ll << 20);
}

cadnn_status cl_prepare_variant(const ClVariant& v, ClPlan* plan, int64_t pixels, int cout) {
    if (v.sk <= 1) return CADNN_OK;
    const int64_t tiles = cl_tiles(v, pixels, cout);
    const size_t part = (size_t)(tiles * v.sk * v.mi * v.ni * 16384), count = (size_t)tiles * 4;
    cadnn_status st = CADNN_OK;
    if (plan->part.bytes < part) {
        plan->part.release();
        if ((st = plan->part.alloc(part, false)) != CADNN_OK) return st;
    }
    if (plan->count.bytes < count) {
        plan->count.release();
        if ((st = plan->count.alloc(count, true)) != CADNN_OK) return st;
    }
    return CADNN_OK;
}

const ClVariant* cl_pick(const cadnn_weights* w, const ClPlan& plan, int64_t pixels, bool f16) {
    const ClVariant* best = nullptr;
    double best_cost = 0.0;
    const double rb = plan.rb / 128.0;
    for (const ClVariant& v : all_cl_variants()) {
        if (!cl_variant_fits(v, plan, pixels, w->cout)) continue;
        const double blocks = (double)cl_tiles(v, pixels, w->cout) * v.sk;
        const double size = v.mi * v.ni;
        const double per_cu = size == 4 ? 2.0 : size == 2 ? 2.0 : 3.0;          // workgroups a CU holds
        const double steps = std::max(1.0, std::ceil((double)plan.steps / v.sk));
        // clocks of a step when a CU's workgroups share it, and of one that has it alone
        const double mfma = (f16 ? 128.0 : 1024.0) * size * rb;
        const double alone = std::max(mfma, 600.0);
        const double shared = std::max(mfma, 600.0 / per_cu);
        const double rounds = std::ceil(blocks / (256.0 * per_cu));
        const double in_cu = std::min(per_cu, std::ceil(blocks / 256.0));
        const double step = in_cu <= 1.0 ? alone : shared * in_cu;
        const double cost = rounds * (4000.0 + steps * std::max(step, alone) + size * 600.0) + (v.sk > 1 ? 4000.0 + 500.0 * v.sk * size : 0.0);
        if (!best || cost < best_cost) { best = &v; best_cost = cost; }
    }
    return best;
}

cadnn_status launch_cl_conv(const ClConv& c, const ClVariant& v, bool f16, hipStream_t s) {
    const ClPlan& p = *c.plan;
    const size_t e = f16 ? 2 : 4;
    ClArgs a{};
    a.w = (const char*)p.w.p;
    a.x = (const char*)c.x;
    a.y = (char*)c.y;
    a.res = (const char*)c.residual;
    a.bias = c.bias;
    a.xt = tensor_arg(c.xd, c.n, e, c.stride, -c.pad, -c.pad);
    a.yt = tensor_arg(c.yd, c.n, e, 1, 0, 0);
    if (c.residual) a.rt = tensor_arg(c.rd, c.n, e, 1, 0, 0);
    if (p.steps2 > 0) {
        a.x2 = (const char*)c.x2;
        a.bias2 = c.bias2;
        a.x2t = tensor_arg(c.x2d, c.n, e, c.stride2, 0, 0);
    }
    a.wspan = (uint32_t)p.w.bytes;
    a.hw = c.yd.h * c.yd.w;
    a.total = c.n * a.hw;
    a.ow = c.yd.w;
    a.cout = c.cout;
    a.relu = c.relu ? 1 : 0;
    a.steps_tap = p.steps_tap;
    a.steps1 = p.taps * p.steps_tap;
    a.steps = p.steps;
    a.tiles_m = (c.cout + 64 * v.mi - 1) / (64 * v.mi);
    a.sk = v.sk;
    a.tiles = (int)cl_tiles(v, a.total, c.cout) * v.sk;
    a.part = (float*)p.part.p;
    a.count = (int*)p.count.p;
    for (int t = 0; t < p.taps; ++t)
        a.tap_off[t] = (int)(((int64_t)p.tap_r[t] * c.xd.row + (int64_t)p.tap_c[t] * c.xd.pix) * (int64_t)e);
    hipError_t err;
    if (f16) err = p.rb == 128 ? launch_cl_rb<_Float16, 128>(a, v.mi, v.ni, s) : launch_cl_rb<_Float16, 64>(a, v.mi, v.ni, s);
    else err = p.rb == 128 ? launch_cl_rb<float, 128>(a, v.mi, v.ni, s) : launch_cl_rb<float, 64>(a, v.mi, v.ni, s);
    CADNN_HIP(err);
    return CADNN_OK;
}

cadnn_status cl_build_plan(const cadnn_weights* w, const cadnn_weights* shortcut, int rb, bool stem, ClPlan* plan) {
    const size_t e = w->elem();
    const int taps_all = w->kh * w->kw, kpr = rb / (int)e;      // k per step
    plan->rb = rb;
    plan->stem = stem;
    plan->taps = 0;
    std::vector<int> tap_index((size_t)taps_all, -1);
    if (stem) {
        // a step is one filter row: kw pixels of 4 channels
        if (w->cin > 4 || w->kw * 4 > kpr || w->kh > kClMaxTaps) return fail(CADNN_EINVAL, "cadnn_net: not a first layer of few channels");
        for (int r = 0; r < w->kh; ++r) { plan->tap_r[r] = r; plan->tap_c[r] = 0; }
        plan->taps = w->kh;
        plan->steps_tap = 1;
    } else {
        std::vector<char> used((size_t)taps_all, 0);
        for (int32_t k : w->col_idx) used[(size_t)(k % taps_all)] = 1;
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
    const size_t blocks = (size_t)(w->cout + 127) / 128 * 2;    // (64-row blocks, whole 128-row tiles)
    const size_t bytes = blocks * (size_t)plan->steps * 64 * (size_t)rb;
    if (bytes >= 0x7ffffff0ull) return fail(CADNN_EUNSUPPORTED, "cadnn_net: weight matrix of 2 GiB or more");
    std::vector<char> img(bytes, 0);
    const int pieces = rb / 16, epp = 16 / (int)e;
    auto put = [&](int co, int step, int k, const cadnn_weights* src, size_t j) {
        const int r = co % 64, sw = rb == 128 ? (r >> 1) & 7 : (r >> 2) & 3;
        const size_t at = (((size_t)(co / 64) * plan->steps + (size_t)step) * 64 + (size_t)r) * (size_t)rb +
                          (size_t)(((k / epp) % pieces) ^ sw) * 16 + (size_t)(k % epp) * e;
        if (e == 2) std::memcpy(&img[at], &src->vals16[j], 2);
        else std::memcpy(&img[at], &src->vals[j], 4);
    };
    for (int i = 0; i < w->cout; ++i)
        for (int32_t j = w->row_ptr[(size_t)i]; j < w->row_ptr[(size_t)i + 1]; ++j) {
            const int k = w->col_idx[(size_t)j], ci = k / taps_all, t = k - ci * taps_all;
            if (stem) put(w->perm[(size_t)i], t / w->kw, (t % w->kw) * 4 + ci, w, (size_t)j);
            else put(w->perm[(size_t)i], tap_index[(size_t)t] * plan->steps_tap + ci / kpr, ci % kpr, w, (size_t)j);
        }
    if (shortcut)
        for (int i = 0; i < shortcut->cout; ++i)
            for (int32_t j = shortcut->row_ptr[(size_t)i]; j < shortcut->row_ptr[(size_t)i + 1]; ++j) {
                const int ci = shortcut->col_idx[(size_t)j];
                put(shortcut->perm[(size_t)i], plan->taps * plan->steps_tap + ci / kpr, ci % kpr, shortcut, (size_t)j);
            }
    return plan->w.upload(img.data(), img.size());
}

}  // namespace cadnn
