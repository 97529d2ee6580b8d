// Channels-last tensors and the kernels that work on them (the net runner's matrix-core path).
#pragma once

#include "internal.h"

namespace cadnn {

// One image of a channels-last activation tensor: (h + 2 * ph) rows of (w + 2 * pw) pixels, the
// channels of a pixel side by side.  A pixel holds `pix` elements, the tensor's own c channels first
// (a slice of a concatenation has the pix of the whole); elements behind them and the halo are
// kept at zero by whoever owns the buffer, like the halo of the plane layout.
struct ClDesc {
    int c, h, w;
    int ph, pw;
    int pix, row;       // elements from one pixel to the next, from one row to the next
    int origin;         // element of pixel (0, 0)
    int64_t image;      // elements from one image to the next
};

// A pixel's channels are read 64 or 128 bytes at a time, so regions pad them to 64 bytes.
inline int cl_padded_channels(int c, size_t elem) {
    const int unit = (int)(64 / elem);
    return (c + unit - 1) / unit * unit;
}
inline ClDesc cl_desc(int c, int h, int w, int ph, int pw, int pix) {
    ClDesc d;
    d.c = c; d.h = h; d.w = w; d.ph = ph; d.pw = pw; d.pix = pix;
    // (a row of 2^30 elements or more: an image that no region holds, and no offset in it)
    const int64_t row = ((int64_t)w + 2 * (int64_t)pw) * pix;
    const bool fits = row < (1 << 30);
    d.row = fits ? (int)row : 0;
    d.origin = ph * d.row + pw * pix;
    d.image = fits ? (int64_t)(h + 2 * ph) * d.row : (int64_t)1 << 40;
    return d;
}

constexpr int kClMaxTaps = 64;

// 4-byte weights are kept as three bf16 numbers whose sum they are but for a scale (fp32 products on the bf16 matrix
// pipes): bytes of an output channel's weights in a step of `rb` bytes of activations.
constexpr int cl_weight_bytes(int rb, int elem) { return elem == 4 ? rb / 4 * 6 : rb; }
// The row of an output channel in its block of 64: a 32 x 32 product leaves a lane the rows 8 g + 4 h + {0..3} of its
// column (h the wave's half, g < 4).  These are to be 16 bytes of channels side by side each time, the other half's the next 16: in
// 4-byte storage they are, in 2-byte storage 4 rows of g and 4 of g + 1 go together.
inline __host__ __device__ int cl_weight_row(int co, int elem) {
    const int c = co % 64;
    return elem == 4 ? c : (c & ~15) | (c & 8) >> 1 | (c & 4) << 1 | (c & 3);
}
// Where part p of the weight of k (in the step) and row r (of a block of 64 output channels) lies: by groups of
// 16 k, parts, wave halves (k = 4 half + {0..3, 8..11} of the group), rows.
inline __host__ __device__ int cl_split_offset(int k, int p, int r) {
    return (((k / 16 * 3 + p) * 2 + k / 4 % 2) * 64 + r) * 16 + (k % 4 + k % 16 / 8 * 4) * 2;
}
// Weights and activations are taken apart scaled by 2^24: the last bit of any float, 2^-149, is then 2^-125, which a bf16 has room for as a
// normal number (bf16 ends at 2^-133: unscaled, operands below 2^-109 would lose bits).
constexpr float kClPartScale = 0x1p24f, kClPartUnscale = 0x1p-24f, kClSumUnscale = 0x1p-48f;
// The first part of a weight that has no scaled parts; the other two then hold the upper and the lower half of the float.
constexpr uint16_t kClWholeWeight = 0x7fff;
// A float, scaled, as the sum of three bf16, each the nearest to what the ones before it left.  An infinity, a NaN, or
// a value that scaled rounds to an infinity is kept whole instead behind a NaN, which the kernel sees in the sums.
inline __host__ __device__ void cl_split_weight(float v, uint16_t part[3]) {
    const float s = v * kClPartScale;
    const uint32_t u = __builtin_bit_cast(uint32_t, s);
    if ((u & 0x7fffffffu) >= 0x7f7f8000u) {
        const uint32_t bits = __builtin_bit_cast(uint32_t, v);
        part[0] = kClWholeWeight;
        part[1] = (uint16_t)(bits >> 16);
        part[2] = (uint16_t)bits;
        return;
    }
    const uint32_t top = (u + 0x7fffu + (u >> 16 & 1u)) & 0xffff0000u;
    const float rest = s - __builtin_bit_cast(float, top);
    const uint32_t r = __builtin_bit_cast(uint32_t, rest), mid = (r + 0x7fffu + (r >> 16 & 1u)) & 0xffff0000u;
    part[0] = (uint16_t)(top >> 16);
    part[1] = (uint16_t)(mid >> 16);
    // (8 bits are left: nothing is cut off)
    part[2] = (uint16_t)(__builtin_bit_cast(uint32_t, rest - __builtin_bit_cast(float, mid)) >> 16);
}
// ... and the float again.
inline __host__ __device__ float cl_join_weight(uint16_t p0, uint16_t p1, uint16_t p2) {
    if (p0 == kClWholeWeight) return __builtin_bit_cast(float, (uint32_t)p1 << 16 | p2);
    const float rest = __builtin_bit_cast(float, (uint32_t)p1 << 16) + __builtin_bit_cast(float, (uint32_t)p2 << 16);
    return (__builtin_bit_cast(float, (uint32_t)p0 << 16) + rest) * kClPartUnscale;
}
// (offsets into the weights are 32-bit)
constexpr size_t kClMaxWeightBytes = 0x7ffffff0u;

// The weights of one layer as the matrix-core kernel reads them: K in steps of `rb` bytes per row
// (rb / elem input channels of one filter tap, taps in order, only those that some filter uses; a
// fused shortcut's channels follow), 64 output channels x one step side by side as [64][rb] with
// the 16-byte pieces of a row in the order the kernel keeps them in LDS.
struct ClPlan {
    DevBuf w;
    int elem = 2;               // bytes of an activation
    bool maps = true;           // y and the residual are channels-last tensors
    int rb = 0, steps = 0, steps_tap = 0, taps = 0, steps2 = 0;
    int tap_r[kClMaxTaps], tap_c[kClMaxTaps];
    bool stem = false;          // input packed 4 channels a pixel, a step is one filter row ...
    int row_bytes = 0;          // ... of this many bytes, the rest of the step being padding of the weights alone
    // K split over workgroups: partial tiles and arrival counters
    DevBuf part, count;
};

// Bytes of the weights in this order: blocks of 64 rows, whole 128-row tiles.
inline size_t cl_plan_bytes(int cout, const ClPlan& plan, int elem) {
    return (size_t)((cout + 127) / 128) * 128 * (size_t)plan.steps * (size_t)cl_weight_bytes(plan.rb, elem);
}

// Tiles a layer can be run with: 64 * mi output channels x 64 * ni output pixels, s stage buffers (how far
// the loads run ahead), sk workgroups that share a tile, each a slice of K, kg groups of four waves that share
// a workgroup, each a part of its slice.
struct ClVariant {
    const char* name;
    int mi, ni, s, sk, kg;
    int bm = 0, bn = 0;         // a small tile of 16 bm x 16 bn instead, whose 8 waves share K (2-byte storage)
    int tm() const { return bm ? 16 * bm : 64 * mi; }
    int tn() const { return bm ? 16 * bn : 64 * ni; }
};
const std::vector<ClVariant>& all_cl_variants();

struct ClConv {
    const ClPlan* plan;                          // the shape of K; its buffers are named below
    const void* w; size_t w_bytes;
    float* part; int* count;
    bool planes;                                 // y and residual are [n][c][h][w]; of yd only h and w are read
    const void* x; ClDesc xd;
    void* y; ClDesc yd;
    const void* residual; ClDesc rd;
    const void* x2; ClDesc x2d; int stride2;     // fused 1x1 shortcut (plan->steps2 > 0)
    const float* bias; const float* bias2;
    int n, cout, stride, pad, relu;
};

// The shape of a layer's K (host work only; tap_of: per filter tap its place among the taps in use, or -1), and with
// the weights on the device.
cadnn_status cl_plan_shape(const cadnn_weights* w, const cadnn_weights* shortcut, int rb, bool stem, ClPlan* plan,
                           std::vector<int>* tap_of = nullptr);
// (`image`: where the device form is put together on the host; kept from layer to layer, its pages need not be mapped anew.)
cadnn_status cl_build_plan(const cadnn_weights* w, const cadnn_weights* shortcut, int rb, bool stem, ClPlan* plan, std::vector<char>* image);
// The tile the cost rule takes, and whether a variant can run the layer.
const ClVariant* cl_pick(int cout, const ClPlan& plan, int64_t pixels, bool f16);
bool cl_variant_fits(const ClVariant& v, const ClPlan& plan, int64_t pixels, int cout);
// Scratch of a split-K variant (no-op otherwise), ready for launches on any stream; on failure the plan keeps what it had.
cadnn_status cl_prepare_variant(const ClVariant& v, ClPlan* plan, int64_t pixels, int cout);
void cl_split_scratch(const ClVariant& v, int64_t pixels, int cout, size_t* part_bytes, size_t* count_bytes);
cadnn_status launch_cl_conv(const ClConv& c, const ClVariant& v, bool f16, hipStream_t s);

// One unpruned layer on [n][c][h][w] tensors from raw weights [cout][cin][kh][kw].
bool dense_cl_serves(bool f16, int n, int cin, int h, int w, int cout, int kh, int kw, int stride, int pad);
// (CADNN_ENOMEM, without a text: no workspace was to be had and nothing was launched.)
cadnn_status dense_cl_conv2d(const void* w_dev, const void* x, void* y, const void* residual, int n, int cin, int h, int w,
                             int cout, int kh, int kw, int stride, int pad, const void* bias, int relu, bool f16, hipStream_t s);

// [n][c][h][w] (the caller's input) -> channels-last.
cadnn_status launch_cl_import(const void* x, int n, int c, int h, int w, void* y, const ClDesc& yd, bool f16, hipStream_t s);
// channels-last -> [n][c][h][w].
cadnn_status launch_cl_export(const void* x, const ClDesc& xd, void* y, int n, bool f16, hipStream_t s);
// Window pools (kind 0: maximum, 1: mean over the in-image part); k = 1 copies.  flat: y is [n][c][h][w].
cadnn_status launch_cl_pool(const void* x, const ClDesc& xd, void* y, const ClDesc& yd, bool flat, int n, int k, int stride,
                            int pad, int kind, bool f16, hipStream_t s);
cadnn_status launch_cl_gap(const void* x, const ClDesc& xd, void* y, int n, bool f16, hipStream_t s);
// 3 x 3, `taps` [9][channels].
cadnn_status launch_cl_depthwise(const float* taps, const void* x, const ClDesc& xd, void* y, const ClDesc& yd, int n,
                                 int stride, int pad, const float* bias, int relu, bool f16, hipStream_t s);

}  // namespace cadnn
