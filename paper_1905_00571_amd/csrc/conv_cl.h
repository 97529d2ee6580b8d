// What the channels-last convolution kernels share: the record of a launch.
#pragma once

#include "channels_last.h"

namespace cadnn {

// (an offset beyond every buffer: loads give 0, stores do nothing)
constexpr uint32_t kClOutOfRange = 0x7ffffff0u;

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
    int steps_tap, steps1, steps, ntaps, tiles_m, tiles, per_die, sk, log_sk;
    int per_slice;              // steps of a slice: of a group of waves of a workgroup of the split
    int row_bytes;              // bytes of a step that are the pixel's own; what lies behind them is not used
    int pixels_first;           // small tiles: those of one block of channels follow each other
    int plane;                  // PLANES: bytes from one channel to the next
    uint32_t magic_hw, magic_ow, magic_tm, magic_st;
    int tap_off[kClMaxTaps];
};

// v / d for 0 <= v < 2^31 with magic = ceil(2^32 / d): the product is at most one too large.
__device__ __forceinline__ int cl_div(int v, uint32_t magic, int d) {
    const int q = (int)__umulhi((uint32_t)v, magic);
    return d == 1 ? v : q - (q * d > v ? 1 : 0);
}

typedef __bf16 cl_b2 __attribute__((ext_vector_type(2)));
typedef float cl_f2 __attribute__((ext_vector_type(2)));

// Two floats, scaled, as the sum of three pairs of bf16, exactly: each is rounded to the nearest 8 bits of what
// the ones before it left, and 24 bits are three times 8, down to the smallest subnormal.  An infinity or a
// NaN, or a value that scaled rounds to one (2^104 and more), leaves NaN behind, which the caller sees in the sums.
// (Shifts, masks and subtractions run beside the matrix products; v_dot2_f32_bf16, which would take the place of two of
// them, does not: 12 products 434 clocks, with 60 subtractions between them 470, with 60 of it 844.)
__device__ __forceinline__ void cl_split2(float a, float b, uint32_t* p1, uint32_t* p2, uint32_t* p3) {
    a *= kClPartScale;
    b *= kClPartScale;
    const uint32_t h1 = __builtin_bit_cast(uint32_t, __builtin_convertvector((cl_f2){a, b}, cl_b2));
    const float ra = a - __uint_as_float(h1 << 16), rb = b - __uint_as_float(h1 & 0xffff0000u);
    const uint32_t h2 = __builtin_bit_cast(uint32_t, __builtin_convertvector((cl_f2){ra, rb}, cl_b2));
    const float sa = ra - __uint_as_float(h2 << 16), sb = rb - __uint_as_float(h2 & 0xffff0000u);
    *p1 = h1;
    *p2 = h2;
    *p3 = __builtin_bit_cast(uint32_t, __builtin_convertvector((cl_f2){sa, sb}, cl_b2));
}

// Small tiles (conv_cl_small.hip).
hipError_t launch_cl_small(const ClArgs& a, const ClVariant& v, int rb, hipStream_t s);

}  // namespace cadnn
