// The layers between the convolutions of a channels-last net: import of the caller's [n][c][h][w]
// tensor, export of the last map, window pools, global average pool, depthwise layers.
//
// All of them move each element once and are bound by memory; a thread works on 16 bytes of one
// pixel's channels, neighbouring threads on neighbouring pieces, so every access is a run of whole
// cache lines, and the taps of a window need no unaligned or 2-byte access at all.
#include <algorithm>
#include <type_traits>

#include "channels_last.h"

namespace cadnn {

namespace {

typedef _Float16 clo_h8 __attribute__((ext_vector_type(8)));
typedef float clo_f4 __attribute__((ext_vector_type(4)));
template <typename T> struct ClVec;
template <> struct ClVec<_Float16> { typedef clo_h8 type; static constexpr int N = 8; };
template <> struct ClVec<float> { typedef clo_f4 type; static constexpr int N = 4; };

// Few channels (c <= 4, packed 4 to a pixel): one thread per pixel.
template <typename T>
__global__ __launch_bounds__(256) void cl_import4_kernel(const T* __restrict__ x, T* __restrict__ y, ClDesc yd, int c, int n) {
    const int hw = yd.h * yd.w;
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= (int64_t)n * hw) return;
    const int img = (int)(i / hw), q = (int)(i - (int64_t)img * hw);
    const int r = q / yd.w, col = q - r * yd.w;
    typedef T v4 __attribute__((ext_vector_type(4)));
    v4 v;
#pragma unroll
    for (int k = 0; k < 4; ++k) v[k] = k < c ? x[((int64_t)img * c + k) * hw + q] : (T)0.0f;
    *(v4*)(y + (int64_t)img * yd.image + yd.origin + (int64_t)r * yd.row + (int64_t)col * yd.pix) = v;
}

// A tile of 64 pixels x 64 channels is transposed through LDS, in either direction.
template <typename T>
__global__ __launch_bounds__(256) void cl_import_kernel(const T* __restrict__ x, T* __restrict__ y, ClDesc yd, int c) {
    constexpr int N = ClVec<T>::N, PITCH = 64 + N;
    typedef typename ClVec<T>::type V;
    __shared__ __attribute__((aligned(16))) T tile[64 * PITCH];      // [pixel][channel]
    const int hw = yd.h * yd.w, lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int q0 = blockIdx.x * 64, c0 = blockIdx.y * 64, img = blockIdx.z;
#pragma unroll
    for (int k = 0; k < 16; ++k) {
        const int ch = wv + 4 * k;
        const bool ok = c0 + ch < c && q0 + lane < hw;
        tile[lane * PITCH + ch] = ok ? x[((int64_t)img * c + c0 + ch) * hw + q0 + lane] : (T)0.0f;
    }
    __syncthreads();
    for (int i = threadIdx.x; i < 64 * (64 / N); i += 256) {
        const int p = i / (64 / N), piece = i % (64 / N), q = q0 + p;
        // (whole pieces: the channels behind the last one are the region's zeros)
        if (q >= hw || c0 + piece * N >= c) continue;
        const int r = q / yd.w, col = q - r * yd.w;
        *(V*)(y + (int64_t)img * yd.image + yd.origin + (int64_t)r * yd.row + (int64_t)col * yd.pix + c0 + piece * N) =
            *(const V*)(tile + p * PITCH + piece * N);
    }
}

template <typename T>
__global__ __launch_bounds__(256) void cl_export_kernel(const T* __restrict__ x, ClDesc xd, T* __restrict__ y) {
    constexpr int N = ClVec<T>::N, PITCH = 64 + N;
    typedef typename ClVec<T>::type V;
    __shared__ __attribute__((aligned(16))) T tile[64 * PITCH];
    const int hw = xd.h * xd.w, lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int q0 = blockIdx.x * 64, c0 = blockIdx.y * 64, img = blockIdx.z;
    for (int i = threadIdx.x; i < 64 * (64 / N); i += 256) {
        const int p = i / (64 / N), piece = i % (64 / N), q = q0 + p;
        if (q >= hw || c0 + piece * N >= xd.c) continue;
        const int r = q / xd.w, col = q - r * xd.w;
        *(V*)(tile + p * PITCH + piece * N) =
            *(const V*)(x + (int64_t)img * xd.image + xd.origin + (int64_t)r * xd.row + (int64_t)col * xd.pix + c0 + piece * N);
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < 16; ++k) {
        const int ch = wv + 4 * k;
        if (c0 + ch < xd.c && q0 + lane < hw) y[((int64_t)img * xd.c + c0 + ch) * hw + q0 + lane] = tile[lane * PITCH + ch];
    }
}

// One thread per output pixel and 16-byte piece of channels.  KIND 0: maximum, 1: mean over the
// in-image part of the window.  K: the window's size, known at compile time for the sizes in use, so that all loads of a
// window are on their way together (from clamped coordinates; what lies outside is replaced afterwards);
// 0: any size, one load after the other.  3 x 3 / 2 on 112 x 112 x 64, fp16, us at batch 1 / 8 / 32: 6.1 / 6.5 / 17
// one after the other, 3.2 / 6.3 / 14.7 together (a launch is 2.6 us, the bytes at batch 32 take 10).
template <typename T, int KIND, int K>
__global__ __launch_bounds__(256) void cl_pool_kernel(const T* __restrict__ x, ClDesc xd, T* __restrict__ y, ClDesc yd, int flat,
                                                      int n, int k, int stride, int pad) {
    constexpr int N = ClVec<T>::N;
    typedef typename ClVec<T>::type V;
    // (all of an activation tensor is less than 2 GiB: its 16-byte pieces are counted in 32 bits)
    const uint32_t pieces = (uint32_t)yd.c / N, hw = (uint32_t)(yd.h * yd.w);
    const uint32_t i = blockIdx.x * 256u + threadIdx.x;
    const uint32_t px = i / pieces;
    const int piece = (int)(i - px * pieces);
    if (px >= (uint32_t)n * hw) return;
    const int img = (int)(px / hw), q = (int)(px - (uint32_t)img * hw);
    const int oh = (int)((uint32_t)q / (uint32_t)yd.w), ow = q - oh * yd.w;
    const T* xp = x + (int64_t)img * xd.image + xd.origin + piece * N;
    const int ih0 = oh * stride - pad, iw0 = ow * stride - pad;
    V m;
    float sum[N];
#pragma unroll
    for (int j = 0; j < N; ++j) { m[j] = -(T)__builtin_inff(); sum[j] = 0.0f; }
    int seen = 0;
    // (a maximum starts from the window's first element inside the image and moves to what is greater, as on planes: a
    // NaN in the first place stays, any other is passed over, and a k = 1 copy is one)
    auto take = [&](const V& v) __attribute__((always_inline)) {
        if constexpr (KIND == 0 && K > 0) {
            m = __builtin_elementwise_max(m, v);
        } else if constexpr (KIND == 0) {
#pragma unroll
            for (int j = 0; j < N; ++j) m[j] = seen == 0 || v[j] > m[j] ? v[j] : m[j];
        } else {
#pragma unroll
            for (int j = 0; j < N; ++j) sum[j] += (float)v[j];
        }
    };
    if constexpr (K > 0) {
        V v[K][K];
#pragma unroll
        for (int a = 0; a < K; ++a)
#pragma unroll
            for (int b = 0; b < K; ++b)
                v[a][b] = *(const V*)(xp + (int64_t)min(max(ih0 + a, 0), xd.h - 1) * xd.row + (int64_t)min(max(iw0 + b, 0), xd.w - 1) * xd.pix);
        const V none = m;
#pragma unroll
        for (int a = 0; a < K; ++a)
#pragma unroll
            for (int b = 0; b < K; ++b) {
                const bool inside = ih0 + a >= 0 && ih0 + a < xd.h && iw0 + b >= 0 && iw0 + b < xd.w;
                V u = v[a][b];
#pragma unroll
                for (int j = 0; j < N; ++j) u[j] = inside ? u[j] : (KIND == 0 ? none[j] : (T)0.0f);
                take(u);
                seen += inside ? 1 : 0;
            }
        // (the first element inside is the one at the clamped first coordinates)
        if constexpr (KIND == 0) {
#pragma unroll
            for (int j = 0; j < N; ++j) m[j] = v[0][0][j] != v[0][0][j] ? v[0][0][j] : m[j];
        }
    } else {
        for (int a = 0; a < k; ++a) {
            if (ih0 + a < 0 || ih0 + a >= xd.h) continue;
            for (int b = 0; b < k; ++b) {
                if (iw0 + b < 0 || iw0 + b >= xd.w) continue;
                take(*(const V*)(xp + (int64_t)(ih0 + a) * xd.row + (int64_t)(iw0 + b) * xd.pix));
                ++seen;
            }
        }
    }
    if constexpr (KIND == 1) {
        const float d = seen ? (float)seen : 1.0f;
#pragma unroll
        for (int j = 0; j < N; ++j) m[j] = (T)(sum[j] / d);
    } else if (!seen) {
#pragma unroll
        for (int j = 0; j < N; ++j) m[j] = (T)0.0f;
    }
    if (flat) {
#pragma unroll
        for (int j = 0; j < N; ++j) y[((int64_t)img * yd.c + piece * N + j) * hw + q] = m[j];
    } else {
        *(V*)(y + (int64_t)img * yd.image + yd.origin + (int64_t)oh * yd.row + (int64_t)ow * yd.pix + piece * N) = m;
    }
}

// One workgroup per image and 8 pieces of channels: 32 threads share the pixels of a piece, in two sums each, and the
// threads' sums are added as a tree: as few roundings in a row as the pool on planes has (hw / 64 + 6; one
// after the other, the 33 of a 7 x 7 map were a third of the error of ResNet-50's fp32 logits).
template <typename T>
__global__ __launch_bounds__(256) void cl_gap_kernel(const T* __restrict__ x, ClDesc xd, T* __restrict__ y) {
    constexpr int N = ClVec<T>::N;
    typedef typename ClVec<T>::type V;
    __shared__ float part[32][8 * N + 1];
    const int piece = threadIdx.x & 7, who = threadIdx.x >> 3, img = blockIdx.y;
    const int c0 = (blockIdx.x * 8 + piece) * N, hw = xd.h * xd.w;
    float s[2][N];
#pragma unroll
    for (int j = 0; j < N; ++j) s[0][j] = s[1][j] = 0.0f;
    if (c0 < xd.c) {
        const T* xp = x + (int64_t)img * xd.image + xd.origin + c0;
        for (int q0 = who; q0 < hw; q0 += 64) {
#pragma unroll
            for (int k = 0; k < 2; ++k) {
                const int q = q0 + 32 * k;
                if (q >= hw) break;
                const int r = q / xd.w, col = q - r * xd.w;
                const V v = *(const V*)(xp + (int64_t)r * xd.row + (int64_t)col * xd.pix);
#pragma unroll
                for (int j = 0; j < N; ++j) s[k][j] += (float)v[j];
            }
        }
    }
#pragma unroll
    for (int j = 0; j < N; ++j) part[who][piece * N + j] = s[0][j] + s[1][j];
    __syncthreads();
    const int ch = (int)threadIdx.x, first = (int)blockIdx.x * 8 * N;
    if (ch < 8 * N && first + ch < xd.c) {
        float t[32];
#pragma unroll
        for (int k = 0; k < 32; ++k) t[k] = part[k][ch];
#pragma unroll
        for (int half = 16; half > 0; half >>= 1)
#pragma unroll
            for (int k = 0; k < half; ++k) t[k] += t[k + half];
        y[(int64_t)img * xd.c + first + ch] = (T)(t[0] / (float)hw);
    }
}

// 3 x 3 depthwise layer on a tensor whose halo holds the padding: a thread keeps the filters of its
// piece of channels and three columns of input in registers and walks `rows` output rows down, so a new
// row of output costs 3 (stride 1) or 6 (stride 2) loads instead of 9.  The filters come [tap][channel], so
// neighbouring pieces read neighbouring bytes of them too ([channel][tap], as the layer kernel on planes has them,
// is 72 4-byte loads per thread, 288 bytes from lane to lane: as long as everything else the thread does).
// What bounds it at the sizes of these nets is the chain of waits, not the 1 to 13 MB of a layer: the launch
// record is fetched whole, and the rows of the next output are requested before this one is computed (a row
// awaited where it is used also awaits the store before it).  14 x 14 x 384 at batch 16, fp16, us: 9.3 with
// [channel][tap], 8.4 with [tap][channel], 4.9 with the rows ahead; 56 x 56 x 144: 22 / 16.6 / 13.
template <typename T>
struct ClDwArgs {
    const T* x;
    T* y;
    const float* w;
    const float* bias;
    int64_t x_image, y_image, x_first, y_first;     // elements; x_first: tap (0, 0) of output pixel (0, 0)
    int x_row, x_pix, y_row, y_pix;
    int c, height, width, n, relu, rows, strips;
};

template <typename T, int STRIDE>
__global__ __launch_bounds__(256) void cl_dw3_kernel(const ClDwArgs<T> a) {
    constexpr int N = ClVec<T>::N;
    typedef typename ClVec<T>::type V;
    asm volatile("" :: "s"(a.x), "s"(a.y), "s"(a.w), "s"(a.bias), "s"(a.x_image), "s"(a.y_image), "s"(a.x_first), "s"(a.y_first), "s"(a.x_row),
                 "s"(a.x_pix), "s"(a.y_row), "s"(a.y_pix), "s"(a.c), "s"(a.height), "s"(a.width), "s"(a.n), "s"(a.relu), "s"(a.rows), "s"(a.strips));
    // (all of an activation tensor is less than 2 GiB: its 16-byte pieces are counted in 32 bits)
    const uint32_t pieces = (uint32_t)a.c / N, strips = (uint32_t)a.strips, width = (uint32_t)a.width;
    const uint32_t i = blockIdx.x * 256u + threadIdx.x;
    uint32_t rest = i / pieces;
    const int piece = (int)(i - rest * pieces);
    const uint32_t up = rest / width;
    const int ow = (int)(rest - up * width);
    const int img = (int)(up / strips), strip = (int)(up - (uint32_t)img * strips);
    if (img >= a.n) return;
    const int oh0 = strip * a.rows, oh1 = min(oh0 + a.rows, a.height);
    const T* xp = a.x + (int64_t)img * a.x_image + a.x_first + (int64_t)(oh0 * STRIDE) * a.x_row + (int64_t)(ow * STRIDE) * a.x_pix + piece * N;
    T* yp = a.y + (int64_t)img * a.y_image + a.y_first + (int64_t)oh0 * a.y_row + (int64_t)ow * a.y_pix + piece * N;
    V in[3][3], next[STRIDE][3];
#pragma unroll
    for (int r = 0; r < 3; ++r)
#pragma unroll
        for (int k = 0; k < 3; ++k) in[r][k] = *(const V*)(xp + (int64_t)r * a.x_row + k * a.x_pix);
    float wt[9][N], b[N];
#pragma unroll
    for (int t = 0; t < 9; ++t)
#pragma unroll
        for (int j = 0; j < N; j += 4) {
            const clo_f4 q = *(const clo_f4*)(a.w + (size_t)t * a.c + piece * N + j);
#pragma unroll
            for (int k = 0; k < 4; ++k) wt[t][j + k] = q[k];
        }
#pragma unroll
    for (int j = 0; j < N; ++j) b[j] = 0.0f;
    if (a.bias) {
#pragma unroll
        for (int j = 0; j < N; ++j) b[j] = a.bias[piece * N + j];
    }
    xp += (int64_t)3 * a.x_row;
    for (int oh = oh0; oh < oh1; ++oh) {
        if (oh + 1 < oh1) {
#pragma unroll
            for (int r = 0; r < STRIDE; ++r)
#pragma unroll
                for (int k = 0; k < 3; ++k) next[r][k] = *(const V*)(xp + (int64_t)r * a.x_row + k * a.x_pix);
        }
        float s[N];
#pragma unroll
        for (int j = 0; j < N; ++j) s[j] = 0.0f;
#pragma unroll
        for (int r = 0; r < 3; ++r)
#pragma unroll
            for (int k = 0; k < 3; ++k)
#pragma unroll
                for (int j = 0; j < N; ++j) s[j] = fmaf(wt[r * 3 + k][j], (float)in[r][k][j], s[j]);
        V o;
#pragma unroll
        for (int j = 0; j < N; ++j) {
            float v = s[j] + b[j];
            if (a.relu) v = v > 0.0f ? v : 0.0f;
            o[j] = (T)v;
        }
        *(V*)yp = o;
        yp += a.y_row;
        xp += (int64_t)STRIDE * a.x_row;
#pragma unroll
        for (int r = 0; r < 3; ++r)
#pragma unroll
            for (int k = 0; k < 3; ++k) in[r][k] = r + STRIDE < 3 ? in[r + STRIDE < 3 ? r + STRIDE : 0][k] : next[r + STRIDE >= 3 ? r + STRIDE - 3 : 0][k];
    }
}

}  // namespace

cadnn_status launch_cl_import(const void* x, int n, int c, int h, int w, void* y, const ClDesc& yd, bool f16, hipStream_t s) {
    if (yd.pix == 4) {
        const unsigned blocks = (unsigned)(((int64_t)n * h * w + 255) / 256);
        if (f16) CADNN_LAUNCH(cl_import4_kernel<_Float16>, dim3(blocks), dim3(256), 0, s, (const _Float16*)x, (_Float16*)y, yd, c, n);
        else CADNN_LAUNCH(cl_import4_kernel<float>, dim3(blocks), dim3(256), 0, s, (const float*)x, (float*)y, yd, c, n);
    } else {
        const dim3 grid((unsigned)((h * w + 63) / 64), (unsigned)((c + 63) / 64), (unsigned)n);
        if (f16) CADNN_LAUNCH(cl_import_kernel<_Float16>, grid, dim3(256), 0, s, (const _Float16*)x, (_Float16*)y, yd, c);
        else CADNN_LAUNCH(cl_import_kernel<float>, grid, dim3(256), 0, s, (const float*)x, (float*)y, yd, c);
    }
    CADNN_HIP(hipGetLastError());
    return CADNN_OK;
}

cadnn_status launch_cl_export(const void* x, const ClDesc& xd, void* y, int n, bool f16, hipStream_t s) {
    const dim3 grid((unsigned)((xd.h * xd.w + 63) / 64), (unsigned)((xd.c + 63) / 64), (unsigned)n);
    if (f16) CADNN_LAUNCH(cl_export_kernel<_Float16>, grid, dim3(256), 0, s, (const _Float16*)x, xd, (_Float16*)y);
    else CADNN_LAUNCH(cl_export_kernel<float>, grid, dim3(256), 0, s, (const float*)x, xd, (float*)y);
    CADNN_HIP(hipGetLastError());
    return CADNN_OK;
}

cadnn_status launch_cl_pool(const void* x, const ClDesc& xd, void* y, const ClDesc& yd, bool flat, int n, int k, int stride,
                            int pad, int kind, bool f16, hipStream_t s) {
    const int64_t items = (int64_t)n * yd.h * yd.w * (yd.c / (f16 ? 8 : 4));
    const dim3 grid((unsigned)((items + 255) / 256)), block(256);
    const int fl = flat ? 1 : 0;
#define CADNN_CL_POOL(T, KIND, K) CADNN_LAUNCH((cl_pool_kernel<T, KIND, K>), grid, block, 0, s, (const T*)x, xd, (T*)y, yd, fl, n, k, stride, pad)
#define CADNN_CL_POOL_K(T, KIND)           \
    do {                                   \
        if (k == 3) CADNN_CL_POOL(T, KIND, 3); \
        else if (k == 2) CADNN_CL_POOL(T, KIND, 2); \
        else CADNN_CL_POOL(T, KIND, 0);    \
    } while (0)
    if (f16 && kind == 0) CADNN_CL_POOL_K(_Float16, 0);
    else if (f16) CADNN_CL_POOL_K(_Float16, 1);
    else if (kind == 0) CADNN_CL_POOL_K(float, 0);
    else CADNN_CL_POOL_K(float, 1);
#undef CADNN_CL_POOL_K
#undef CADNN_CL_POOL
    CADNN_HIP(hipGetLastError());
    return CADNN_OK;
}

cadnn_status launch_cl_gap(const void* x, const ClDesc& xd, void* y, int n, bool f16, hipStream_t s) {
    const int per = f16 ? 64 : 32;
    const dim3 grid((unsigned)((xd.c + per - 1) / per), (unsigned)n);
    if (f16) CADNN_LAUNCH(cl_gap_kernel<_Float16>, grid, dim3(256), 0, s, (const _Float16*)x, xd, (_Float16*)y);
    else CADNN_LAUNCH(cl_gap_kernel<float>, grid, dim3(256), 0, s, (const float*)x, xd, (float*)y);
    CADNN_HIP(hipGetLastError());
    return CADNN_OK;
}

cadnn_status launch_cl_depthwise(const float* taps, const void* x, const ClDesc& xd, void* y, const ClDesc& yd, int n,
                                 int stride, int pad, const float* bias, int relu, bool f16, hipStream_t s) {
    // rows a thread walks: as many as still leave the chip a few workgroups per CU
    const int64_t columns = (int64_t)n * yd.w * (yd.c / (f16 ? 8 : 4));
    int rows = 14;
    while (rows > 2 && columns * ((yd.h + rows - 1) / rows) < 256 * 1024) rows = (rows + 1) / 2;
    const int strips = (yd.h + rows - 1) / rows;
    const dim3 grid((unsigned)((columns * strips + 255) / 256)), block(256);
    auto fill = [&](auto& a) {
        typedef typename std::remove_const<typename std::remove_pointer<decltype(a.x)>::type>::type T;
        a.x = (const T*)x; a.y = (T*)y; a.w = taps; a.bias = bias;
        a.x_image = xd.image; a.y_image = yd.image;
        a.x_first = xd.origin - (int64_t)pad * xd.row - (int64_t)pad * xd.pix;
        a.y_first = yd.origin;
        a.x_row = xd.row; a.x_pix = xd.pix; a.y_row = yd.row; a.y_pix = yd.pix;
        a.c = yd.c; a.height = yd.h; a.width = yd.w; a.n = n; a.relu = relu; a.rows = rows; a.strips = strips;
    };
    ClDwArgs<_Float16> h{};
    ClDwArgs<float> f{};
    if (f16) fill(h); else fill(f);
#define CADNN_CL_DW(T, S, A) CADNN_LAUNCH((cl_dw3_kernel<T, S>), grid, block, 0, s, A)
    if (f16 && stride == 1) CADNN_CL_DW(_Float16, 1, h);
    else if (f16) CADNN_CL_DW(_Float16, 2, h);
    else if (stride == 1) CADNN_CL_DW(float, 1, f);
    else CADNN_CL_DW(float, 2, f);
#undef CADNN_CL_DW
    CADNN_HIP(hipGetLastError());
    return CADNN_OK;
}

}  // namespace cadnn
