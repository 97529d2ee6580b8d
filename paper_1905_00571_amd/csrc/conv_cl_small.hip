// Channels-last convolution with small tiles (gfx950, 2-byte storage): layers of so few pixels and channels that the
// tiles of conv_cl.hip leave most of the chip idle.
//
// What bounds such a layer is what a CU can fetch while it is nearly alone (28 bytes a clock from behind the L2, and a step of a
// 64 x 64 tile is 16 KB), so the work is spread over as many CUs as there are: tiles of 16 or 32 channels x 16 or 32 pixels, and within
// a workgroup K is dealt to 8 waves.  No operand is shared between waves, so both go from memory
// straight into the registers of the product (v_mfma_f32_16x16x32_f16: 16 bytes a lane, the weights from the
// same plan as the large tiles', whole 64-byte pieces of rows), D steps in flight, without LDS and without a barrier.  The waves'
// sums meet in LDS once, added in the order of K.
// us a layer in a graph of equal ones at one image, best large tile / here: 256 -> 256 3x3 on 14 x 14 8.6 / 7.0, 1024 -> 256 1x1 5.5 / 4.0,
// 128 -> 128 3x3 on 28 x 28 7.2 / 6.4; ResNet-50 fp16 312 -> 278.  A launch of one step takes 2.9; the operands then come at 13 to 18 bytes a
// clock and CU (64-byte pieces through the vector L1), which bounds it.
#include "conv_cl.h"

namespace cadnn {

namespace {

typedef _Float16 cs_h8 __attribute__((ext_vector_type(8)));
typedef _Float16 cs_h4 __attribute__((ext_vector_type(4)));
typedef float cs_f4 __attribute__((ext_vector_type(4)));
typedef uint32_t cs_u4 __attribute__((ext_vector_type(4)));
typedef uint32_t cs_u2 __attribute__((ext_vector_type(2)));

constexpr int kWaves = 8;

template <int RB, int BM, int BN, int D>
__global__ __launch_bounds__(64 * kWaves) void cl_small_kernel(const ClArgs a) {
    static_assert(BM * BN <= kWaves, "a wave finishes one block");
    __shared__ cs_f4 part[kWaves][BM * BN][64];
    // (the launch record whole and at once: field by field it is a chain of scalar-cache misses)
    asm volatile("" :: "s"(a.w), "s"(a.x), "s"(a.x2), "s"(a.y), "s"(a.res), "s"(a.bias), "s"(a.bias2), "s"(a.wspan), "s"(a.total), "s"(a.hw),
                 "s"(a.ow), "s"(a.cout), "s"(a.relu), "s"(a.steps_tap), "s"(a.steps1), "s"(a.steps), "s"(a.ntaps), "s"(a.tiles_m), "s"(a.tiles),
                 "s"(a.per_die), "s"(a.magic_hw), "s"(a.magic_ow), "s"(a.magic_tm), "s"(a.magic_st), "s"(a.per_slice), "s"(a.pixels_first));
    asm volatile("" :: "s"(a.xt.span), "s"(a.xt.img), "s"(a.xt.row), "s"(a.xt.col), "s"(a.xt.org), "s"(a.x2t.span), "s"(a.x2t.img), "s"(a.x2t.row),
                 "s"(a.x2t.col), "s"(a.x2t.org), "s"(a.yt.span), "s"(a.yt.img), "s"(a.yt.row), "s"(a.yt.col), "s"(a.yt.org), "s"(a.tap_off[0]));
    const int t = ((int)blockIdx.x & 7) * a.per_die + ((int)blockIdx.x >> 3);       // dies own contiguous runs
    if (((int)blockIdx.x >> 3) >= a.per_die || t >= a.tiles) return;
    // (magic_tm and tiles_m are those of the tiles that follow each other)
    const int slow = cl_div(t, a.magic_tm, a.tiles_m), fast = t - slow * a.tiles_m;
    const int mt = a.pixels_first ? slow : fast, nt = a.pixels_first ? fast : slow;
    const int m0 = mt * 16 * BM, n0 = nt * 16 * BN;
    const int tid = (int)threadIdx.x, lane = tid & 63, r = lane & 15, q = lane >> 4;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);

    // ---- this wave's part of K, in halves of 32 k of a step of 64 (or steps of 32)
    constexpr int HALVES = RB / 64;
    const int s_first = wv * a.per_slice, count = min(a.per_slice, a.steps * HALVES - s_first);

    auto rsrc = [](const void* p, uint32_t span) __attribute__((always_inline)) {
        return __builtin_amdgcn_make_buffer_rsrc((void*)p, 0, span, 0x00020000);
    };
    // ---- weights: lane r, q has 8 k of row r of a block of 16; the pieces of a row are permuted by the row
    uint32_t wv0[BM];
#pragma unroll
    for (int mb = 0; mb < BM; ++mb) {
        const int row = m0 % 64 + mb * 16 + r;
        const int sw = RB == 128 ? (row >> 1) & 7 : (row >> 2) & 3;
        wv0[mb] = (uint32_t)(row * RB + (q ^ sw) * 16);
    }
    uint32_t w_soff = (uint32_t)((m0 / 64) * a.steps + s_first / HALVES) * (64u * RB);
    int half = s_first % HALVES;

    // ---- activations: lane r, q has 8 k of pixel r
    struct Pixel { int img, oh, ow; bool live; };
    auto pixel = [&](int nb) __attribute__((always_inline)) {
        const int Q = n0 + nb * 16 + r;
        Pixel p;
        p.live = Q < a.total;
        p.img = cl_div(Q, a.magic_hw, a.hw);
        const int rest = Q - p.img * a.hw;
        p.oh = cl_div(rest, a.magic_ow, a.ow);
        p.ow = rest - p.oh * a.ow;
        return p;
    };
    auto offset = [](const ClTensorArg& d, const Pixel& p) __attribute__((always_inline)) {
        return p.img * d.img + p.oh * d.row + p.ow * d.col + d.org;
    };
    uint32_t xv[BN], xv2[BN];
#pragma unroll
    for (int nb = 0; nb < BN; ++nb) {
        const Pixel p = pixel(nb);
        xv[nb] = p.live ? (uint32_t)offset(a.xt, p) + (uint32_t)q * 16u : kClOutOfRange;
        xv2[nb] = a.steps > a.steps1 && p.live ? (uint32_t)offset(a.x2t, p) + (uint32_t)q * 16u : kClOutOfRange;
    }
    // ---- the walk over K.  Past the end of the wave's part nothing is fetched (a span and an offset of 0: zeros).
    int left, tap = 0, todo = count;
    uint32_t x_soff;
    bool second = false;
    auto enter_shortcut = [&](int at) __attribute__((always_inline)) {
        second = true;
        left = 0x7fffffff;
        x_soff = (uint32_t)at * 64u;
    };
    if (s_first < a.steps1 * HALVES) {
        tap = cl_div(s_first / HALVES, a.magic_st, a.steps_tap);
        const int at = s_first - tap * a.steps_tap * HALVES;
        left = a.steps_tap * HALVES - at;
        x_soff = (uint32_t)a.tap_off[tap] + (uint32_t)at * 64u;
    } else {
        enter_shortcut(s_first - a.steps1 * HALVES);
    }
    cs_u4 af[D][BM], bf[D][BN];
    auto fetch = [&](int d) __attribute__((always_inline)) {
        const bool live = todo > 0;
        const auto wr = rsrc(a.w, live ? a.wspan : 0u);
        const auto xr = rsrc(second ? a.x2 : a.x, live ? (second ? a.x2t.span : a.xt.span) : 0u);
        // (what an offset is checked against, the span or the span less the scalar offset, is never negative)
        const uint32_t ws = live ? w_soff : 0u, xs = live ? x_soff : 0u;
#pragma unroll
        for (int mb = 0; mb < BM; ++mb)
            af[d][mb] = __builtin_bit_cast(cs_u4, __builtin_amdgcn_raw_buffer_load_b128(wr, HALVES == 2 ? wv0[mb] ^ (uint32_t)(half * 64) : wv0[mb], ws, 0));
#pragma unroll
        for (int nb = 0; nb < BN; ++nb)
            bf[d][nb] = __builtin_bit_cast(cs_u4, __builtin_amdgcn_raw_buffer_load_b128(xr, second ? xv2[nb] : xv[nb], xs, 0));
        --todo;
        x_soff += 64u;
        if (HALVES == 1 || half == 1) w_soff += 64u * RB;
        half ^= HALVES - 1;
        if (--left == 0) {
            if (++tap < a.ntaps) {
                left = a.steps_tap * HALVES;
                x_soff = (uint32_t)a.tap_off[tap];
            } else {
                enter_shortcut(0);
            }
        }
    };
#pragma unroll
    for (int d = 0; d < D; ++d) fetch(d);

    // ---- what the epilogue needs: wave w < BM BN finishes block w, a lane 4 channels side by side of one pixel
    const int mb_out = wv / BN, nb_out = wv % BN;
    const int ch = m0 + mb_out * 16 + (q & 1) * 8 + (q >> 1) * 4;
    cs_f4 bias = {0.0f, 0.0f, 0.0f, 0.0f}, bias2 = bias;
    uint32_t y_off = kClOutOfRange;
    cs_u2 res = {0u, 0u};
    if (wv < BM * BN) {
        const Pixel p = pixel(nb_out);
        if (p.live && ch < a.cout) y_off = (uint32_t)(offset(a.yt, p) + ch * 2);
        const auto b1 = rsrc(a.bias, a.bias ? (uint32_t)a.cout * 4u : 0u), b2 = rsrc(a.bias2, a.bias2 ? (uint32_t)a.cout * 4u : 0u);
        bias = __builtin_bit_cast(cs_f4, __builtin_amdgcn_raw_buffer_load_b128(b1, (uint32_t)ch * 4u, 0u, 0));
        bias2 = __builtin_bit_cast(cs_f4, __builtin_amdgcn_raw_buffer_load_b128(b2, (uint32_t)ch * 4u, 0u, 0));
        if (a.res) {
            const uint32_t off = p.live && ch < a.cout ? (uint32_t)(offset(a.rt, p) + ch * 2) : kClOutOfRange;
            res = __builtin_bit_cast(cs_u2, __builtin_amdgcn_raw_buffer_load_b64(rsrc(a.res, a.rt.span), off, 0u, 0));
        }
    }

    cs_f4 acc[BM][BN];
#pragma unroll
    for (int mb = 0; mb < BM; ++mb)
#pragma unroll
        for (int nb = 0; nb < BN; ++nb) acc[mb][nb] = cs_f4{0.0f, 0.0f, 0.0f, 0.0f};
    for (int s = 0; s < count; s += D) {
#pragma unroll
        for (int d = 0; d < D; ++d) {
#pragma unroll
            for (int mb = 0; mb < BM; ++mb)
#pragma unroll
                for (int nb = 0; nb < BN; ++nb)
                    acc[mb][nb] = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(cs_h8, af[d][mb]), __builtin_bit_cast(cs_h8, bf[d][nb]),
                                                                         acc[mb][nb], 0, 0, 0);
            fetch(d);
        }
    }
#pragma unroll
    for (int mb = 0; mb < BM; ++mb)
#pragma unroll
        for (int nb = 0; nb < BN; ++nb) part[wv][mb * BN + nb][lane] = acc[mb][nb];
    __syncthreads();
    if (wv >= BM * BN) return;
    cs_f4 v = part[0][wv][lane];
#pragma unroll
    for (int w = 1; w < kWaves; ++w) v += part[w][wv][lane];
    const cs_h4 rh = __builtin_bit_cast(cs_h4, res);
    cs_h4 o;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        float f = v[i] + (bias[i] + bias2[i]);
        if (a.res) f += (float)rh[i];
        o[i] = (_Float16)((a.relu && !(f > 0.0f)) ? 0.0f : f);
    }
    __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(cs_u2, o), rsrc(a.y, a.yt.span), y_off, 0u, 0);
}

template <int RB, int BM, int BN, int D>
hipError_t launch_small(const ClArgs& a, hipStream_t s) {
    CADNN_LAUNCH((cl_small_kernel<RB, BM, BN, D>), dim3((unsigned)((a.tiles + 7) / 8 * 8)), dim3(64 * kWaves), 0, s, a);
    return hipGetLastError();
}

template <int RB>
hipError_t launch_small_rb(const ClArgs& a, const ClVariant& v, hipStream_t s) {
    if (v.bm == 1) return v.bn == 1 ? launch_small<RB, 1, 1, 6>(a, s) : launch_small<RB, 1, 2, 4>(a, s);
    return v.bn == 1 ? launch_small<RB, 2, 1, 4>(a, s) : launch_small<RB, 2, 2, 4>(a, s);
}

}  // namespace

hipError_t launch_cl_small(const ClArgs& args, const ClVariant& v, int rb, hipStream_t s) {
    ClArgs a = args;
    a.per_slice = (a.steps * (rb / 64) + kWaves - 1) / kWaves;
    // A die fetches its tiles' operands from behind its L2: where the weights are the larger one, it owns output channels.  (ResNet-50
    // fp16 at one image, always pixels / this: 280.3 / 278.4 us a pass, runs of either within 0.4 %.)
    a.pixels_first = a.wspan > a.xt.span;
    if (a.pixels_first) {
        a.tiles_m = (a.total + v.tn() - 1) / v.tn();
        a.magic_tm = (uint32_t)(((1ull << 32) + (uint64_t)a.tiles_m - 1) / (uint64_t)a.tiles_m);
    }
    return rb == 128 ? launch_small_rb<128>(a, v, s) : launch_small_rb<64>(a, v, s);
}

}  // namespace cadnn
