// One unpruned layer on plain [n][c][h][w] tensors and raw weights, through the channels-last matrix-core kernel.
//
// Two launches: `cl_arrange_kernel` brings the input into the channels-last layout with its zero
// halo and the weights into the order the kernel loads them in; the convolution then writes
// [n][c][h][w] from its accumulators.  Both tensors are moved once more than a kernel on planes
// moves them (256 channels of 14 x 14 at batch 32, fp16: 6.4 MB and 1.2 MB of weights), which buys
// 16-byte loads straight to LDS for 2-byte gathers and a transposition in registers.  us per call, one launch on
// planes / this: that layer 52.9 / 24.1; fp16 192 -> 192 5x5 on 8 x 42 77 / 21, 29 -> 36 5x5 on two 100 x 100 images
// 45 / 17; fp32 62 -> 188 7x7 on 71 x 71 189 / 76, 107 -> 25 7x7 / 2 on 43 x 43 316 / 39.
#include <algorithm>
#include <mutex>
#include <vector>

#include "conv_cl.h"

namespace cadnn {

namespace {

struct ClArrange {
    const void* x;
    void* xr;
    ClDesc xd;
    int positions, pos_blocks, ch_blocks, x_blocks;   // positions: pixels of an image with its halo
    const void* w;
    void* wr;
    int cin, cout, taps, steps_tap, kpr, pieces;
    int* count;
    int ncount;
};

// Bound by latency more than by memory: a workgroup moves 64 positions x 64 channels (8 or 16 KB), or
// four filters x one step of channels x all taps, so that reads and writes are whole runs of 64
// bytes and more and a layer of the usual sizes is some hundred workgroups.  Channels behind the last one
// are zero on both sides; filters behind the last one are not written (they reach only output
// channels that are never stored).
template <typename T>
__global__ __launch_bounds__(256) void cl_arrange_kernel(const ClArrange a) {
    constexpr int N = 16 / (int)sizeof(T), PITCH = 64 + N;
    typedef T V __attribute__((ext_vector_type(16 / sizeof(T))));
    extern __shared__ __attribute__((aligned(16))) char cl_arrange_smem[];
    T* lds = (T*)cl_arrange_smem;
    const int tid = (int)threadIdx.x, lane = tid & 63, wv = tid >> 6;
    if (blockIdx.x == 0)
        for (int i = tid; i < a.ncount; i += 256) a.count[i] = 0;
    if ((int)blockIdx.x < a.x_blocks) {
        const int rest = (int)blockIdx.x / a.pos_blocks, q0 = ((int)blockIdx.x - rest * a.pos_blocks) * 64;
        const int img = rest / a.ch_blocks, c0 = (rest - img * a.ch_blocks) * 64;
        const int pw = a.xd.w + 2 * a.xd.pw, q = q0 + lane, hr = q / pw;
        const int r = hr - a.xd.ph, col = q - hr * pw - a.xd.pw;
        const bool inside = q < a.positions && r >= 0 && r < a.xd.h && col >= 0 && col < a.xd.w;
        const int64_t plane = (int64_t)a.xd.h * a.xd.w;
        const T* src = (const T*)a.x + (int64_t)img * a.cin * plane + (inside ? (int64_t)r * a.xd.w + col : 0);
        T v[16];
#pragma unroll
        for (int k = 0; k < 16; ++k) {
            const int ch = c0 + wv * 16 + k;
            v[k] = inside && ch < a.cin ? src[(int64_t)ch * plane] : (T)0.0f;
        }
#pragma unroll
        for (int k = 0; k < 16; k += N) {
            V p;
#pragma unroll
            for (int j = 0; j < N; ++j) p[j] = v[k + j];
            *(V*)(lds + lane * PITCH + wv * 16 + k) = p;
        }
        __syncthreads();
        T* dst = (T*)a.xr + (int64_t)img * a.xd.image;
        for (int i = tid; i < 64 * (64 / N); i += 256) {
            const int p = i / (64 / N), c = (i % (64 / N)) * N;
            if (q0 + p < a.positions && c0 + c < a.xd.pix) *(V*)(dst + (int64_t)(q0 + p) * a.xd.pix + c0 + c) = *(const V*)(lds + p * PITCH + c);
        }
    } else {
        const int b = (int)blockIdx.x - a.x_blocks, step = b % a.steps_tap, co = b / a.steps_tap * 4 + wv;
        const int c0 = step * a.kpr, have = min(a.kpr, a.cin - c0) * a.taps, all = a.kpr * a.taps;
        T* mine = lds + wv * all;
        if (co < a.cout) {
            const T* src = (const T*)a.w + ((int64_t)co * a.cin + c0) * a.taps;
            // (nine loads in flight: a 3x3 filter's step of 64 channels at once)
            for (int i0 = 0; i0 < all; i0 += 9 * 64) {
                T v[9];
#pragma unroll
                for (int u = 0; u < 9; ++u) {
                    const int i = i0 + u * 64 + lane;
                    v[u] = i < have ? src[i] : (T)0.0f;
                }
#pragma unroll
                for (int u = 0; u < 9; ++u) {
                    const int i = i0 + u * 64 + lane;
                    if (i < all) mine[i] = v[u];
                }
            }
        }
        __syncthreads();
        const int64_t steps = (int64_t)a.taps * a.steps_tap;
        if constexpr (sizeof(T) == 4) {
            // Eight k of one half of a wave: 16 bytes of each of the three parts.  The four filters of the workgroup are four rows side by
            // side, so four lanes write 64 bytes of a part.  (A wave for its own filter, 16 bytes at a time in lines 1 KB apart: us of the
            // launch 5.2 -> 4.1 for 16 -> 58 7x7, 5.6 -> 4.2 for 107 -> 68 1x1 on 102 x 102, 12.8 -> 9.8 for 512 -> 512 3x3; 4-byte weights
            // as they are took 3.9, 4.0, 10.0.)
            const int log_halves = a.kpr == 32 ? 2 : 1;
            for (int i = tid; i < a.taps << (log_halves + 2); i += 256) {
                const int at = i >> 2, t = at >> log_halves, h = at - (t << log_halves), k0 = h / 2 * 16 + h % 2 * 4;
                const int r = i & 3, filter = co - wv + r;
                if (filter >= a.cout) continue;
                const T* const from = lds + r * all + k0 * a.taps + t;
                char* const block = (char*)a.wr + ((filter / 64) * steps + (int64_t)t * a.steps_tap + step) * 64 * cl_weight_bytes(a.kpr * 4, 4);
                float v[8];
                bool large = false;
#pragma unroll
                for (int j = 0; j < 8; ++j) {
                    v[j] = from[(j / 4 * 8 + j % 4) * a.taps];
                    large |= (__float_as_uint(v[j] * kClPartScale) & 0x7fffffffu) >= 0x7f7f8000u;       // has no scaled parts
                }
                uint32_t part[3][4];
                if (large) {
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        uint16_t lo[3], hi[3];
                        cl_split_weight(v[2 * j], lo);
                        cl_split_weight(v[2 * j + 1], hi);
#pragma unroll
                        for (int p = 0; p < 3; ++p) part[p][j] = lo[p] | (uint32_t)hi[p] << 16;
                    }
                } else {
#pragma unroll
                    for (int j = 0; j < 4; ++j) cl_split2(v[2 * j], v[2 * j + 1], &part[0][j], &part[1][j], &part[2][j]);
                }
#pragma unroll
                for (int p = 0; p < 3; ++p)
                    *(uint4*)(block + cl_split_offset(k0, p, filter % 64)) = make_uint4(part[p][0], part[p][1], part[p][2], part[p][3]);
            }
        } else {
            if (co >= a.cout) return;
            const int row = cl_weight_row(co, (int)sizeof(T)), sw = a.pieces == 8 ? (row >> 1) & 7 : (row >> 2) & 3;
            for (int i = lane; i < a.taps * a.pieces; i += 64) {
                const int t = i / a.pieces, pc = i - t * a.pieces;
                V p;
#pragma unroll
                for (int j = 0; j < N; ++j) p[j] = mine[(pc * N + j) * a.taps + t];
                const int64_t at = ((co / 64) * steps + (int64_t)t * a.steps_tap + step) * 64 + row;
                *(V*)((T*)a.wr + at * a.kpr + (pc ^ sw) * N) = p;
            }
        }
    }
}

// Workspaces of layer calls.  hipMallocAsync + hipFreeAsync cost the host 11 to 13 us a call (2 launches 5.4 us, with
// them 16 to 18; and 50 us where every call is waited for, the pool giving its memory back each time), more than
// the kernels of most layers, so blocks are kept: taken under the lock, owned by one call until it returns
// them, and handed on with an event that the next user's stream waits for (8.6 us in all).  At most
// kKeep blocks of at most kKeepBytes together are held, of at most half of that each (96 MiB: 64 MiB of 4-byte weights, which
// take 6 bytes here); one that no longer fits goes back to the device, in the order
// of the stream that takes its place.  For larger workspaces every call allocates for itself in stream
// order.  (No captured stream comes here.)  All of it is given back by release(), which the library calls itself when
// an allocation of its own finds no memory.
struct Workspace {
    char* p = nullptr;
    size_t bytes = 0;
    int device = -1;
    hipEvent_t used = nullptr;       // recorded behind the last call that had it; NULL: not a kept block
};

class WorkspacePool {
  public:
    hipError_t take(size_t bytes, hipStream_t s, Workspace* out) {
        hipError_t e;
        *out = Workspace{};
        out->bytes = bytes;
        if (bytes > kKeepBytes / 2) return allocate(&out->p, bytes, s);
        int device = 0;
        if ((e = hipGetDevice(&device)) != hipSuccess) return e;
        Workspace found, old;
        {
            std::lock_guard<std::mutex> lock(mu_);
            auto best = free_.end(), small = free_.end();
            for (auto it = free_.begin(); it != free_.end(); ++it) {
                if (it->device != device) continue;
                if (it->bytes < bytes) small = it;
                else if (best == free_.end() || it->bytes < best->bytes) best = it;
            }
            if (best != free_.end()) {
                found = *best;
                free_.erase(best);
            } else if (small != free_.end()) {       // one that is too small makes room
                old = *small;
                free_.erase(small);
            }
        }
        if (found.p) {
            if ((e = hipStreamWaitEvent(s, found.used, 0)) != hipSuccess) return give_up(found, e);
            *out = found;
            return hipSuccess;
        }
        if (old.p && hipStreamWaitEvent(s, old.used, 0) == hipSuccess) (void)hipFreeAsync(old.p, s);
        hipEvent_t ev = old.used;
        if (!ev && (e = hipEventCreateWithFlags(&ev, hipEventDisableTiming)) != hipSuccess) return e;
        // (room to grow: sizes that vary a little share a block)
        const size_t round = (bytes + (1u << 20) - 1) >> 20 << 20;
        if ((e = allocate(&out->p, round, s)) != hipSuccess) {
            (void)hipEventDestroy(ev);
            return e;
        }
        out->bytes = round;
        out->device = device;
        out->used = ev;
        return hipSuccess;
    }

    hipError_t give(const Workspace& w, hipStream_t s) {
        if (!w.used) return hipFreeAsync(w.p, s);
        hipError_t e = hipEventRecord(w.used, s);
        if (e != hipSuccess) return give_up(w, e);
        std::lock_guard<std::mutex> lock(mu_);
        size_t held = w.bytes;
        for (const Workspace& f : free_) held += f.bytes;
        if (free_.size() < kKeep && held <= kKeepBytes) {
            try {
                free_.push_back(w);
                return hipSuccess;
            } catch (const std::bad_alloc&) {
            }
        }
        (void)hipEventDestroy(w.used);
        return hipFreeAsync(w.p, s);
    }

    // Every kept block, when the call that had it last is through, back to the device.
    void release() {
        std::vector<Workspace> all;
        {
            std::lock_guard<std::mutex> lock(mu_);
            all.swap(free_);
        }
        for (const Workspace& w : all) {
            if (hipEventSynchronize(w.used) == hipSuccess) (void)hipFree(w.p);
            (void)hipEventDestroy(w.used);
        }
        (void)hipGetLastError();
    }

  private:
    hipError_t allocate(char** p, size_t bytes, hipStream_t s) {
        hipError_t e = hipMallocAsync((void**)p, bytes, s);
        if (e == hipSuccess) return e;
        release();
        e = hipMallocAsync((void**)p, bytes, s);
        if (e != hipSuccess) {
            *p = nullptr;
            (void)hipGetLastError();        // (the launches that take the call's place ask for the last error)
        }
        return e;
    }
    static constexpr size_t kKeep = 8, kKeepBytes = (size_t)192 << 20;
    // (the stream is in an error state: the block is not handed on, nor freed under work that may still run)
    static hipError_t give_up(const Workspace& w, hipError_t e) {
        (void)hipEventDestroy(w.used);
        return e;
    }
    std::mutex mu_;
    std::vector<Workspace> free_;
};

WorkspacePool& workspaces() {
    static WorkspacePool* pool = new WorkspacePool();      // (never destroyed: the runtime may be gone before it would be)
    return *pool;
}

size_t align256(size_t v) { return (v + 255) / 256 * 256; }

}  // namespace

// Fewer than 16 input channels are mostly padding here (a piece of 64 bytes at least).  The kernel on planes takes
// about 2 us per 32 of K and round of workgroups in one launch (K 40: 9.4 us a call, which is the host's; 83: 10.8, 176: 14.0,
// 279: 22, 360: 27, 1989: 107), the two launches here 13.4 us at the least (the same layers: 83, 176 kept; 279 13.7, 360 14.9, 1989 15.4): up to six such steps stay there.
// (fp16 layers of whole 32 channels do not have that kernel to go back to: theirs allocates and reorders on every call.)
bool dense_cl_serves(bool f16, int n, int cin, int h, int w, int cout, int kh, int kw, int stride, int pad) {
    const size_t e = f16 ? 2 : 4;
    if (cin < 16 || kh * kw > kClMaxTaps || n > 65535 || pad > 64 || stride > 64) return false;
    const ClDesc d = cl_desc(cin, h, w, pad, pad, cl_padded_channels(cin, e));
    const int64_t hw = (int64_t)conv_out(h, kh, stride, pad) * conv_out(w, kw, stride, pad);
    const int64_t limit = 0x7fff0000ll, padded_rows = (cout + 127) / 128 * 128;
    const int64_t image = (int64_t)(h + 2 * pad) * (w + 2 * pad) * d.pix;
    if ((int64_t)d.pix * (w + 2 * pad) * (int64_t)e >= limit / 64 || image * (int64_t)e * n >= limit) return false;
    if ((int64_t)n * hw >= (1 << 30) || (int64_t)n * hw * cout * (int64_t)e >= limit) return false;
    if (padded_rows * kh * kw * d.pix * (f16 ? 2 : 6) >= limit) return false;      // (three 2-byte parts a 4-byte weight)
    if (f16 && cin % 32 == 0) return true;
    const int64_t blocks = (hw + 63) / 64 * n * ((cout + 63) / 64);
    return ((int64_t)cin * kh * kw + 31) / 32 * ((blocks + 1023) / 1024) > 6;
}

void release_workspaces() { workspaces().release(); }

cadnn_status dense_cl_conv2d(const void* w_dev, const void* x, void* y, const void* residual, int n, int cin, int h, int w,
                             int cout, int kh, int kw, int stride, int pad, const void* bias, int relu, bool f16, hipStream_t s) {
    const size_t e = f16 ? 2 : 4;
    ClPlan plan;
    plan.elem = (int)e;
    plan.maps = false;
    const ClDesc xd = cl_desc(cin, h, w, pad, pad, cl_padded_channels(cin, e));
    plan.rb = ((size_t)xd.pix * e) % 128 ? 64 : 128;
    const int kpr = plan.rb / (int)e, pieces = plan.rb / 16;
    plan.taps = kh * kw;
    for (int t = 0; t < plan.taps; ++t) { plan.tap_r[t] = t / kw; plan.tap_c[t] = t % kw; }
    plan.steps_tap = xd.pix / kpr;
    plan.steps = plan.taps * plan.steps_tap;
    ClConv c{};
    c.yd.h = conv_out(h, kh, stride, pad);
    c.yd.w = conv_out(w, kw, stride, pad);
    const int64_t pixels = (int64_t)n * c.yd.h * c.yd.w;
    const ClVariant* v = cl_pick(cout, plan, pixels, f16);

    const size_t x_bytes = align256((size_t)n * (size_t)xd.image * e);
    c.w_bytes = cl_plan_bytes(cout, plan, (int)e);
    size_t part = 0, count = 0;
    cl_split_scratch(*v, pixels, cout, &part, &count);
    Workspace block;
    const size_t total = x_bytes + align256(c.w_bytes) + align256(part) + count;
    hipError_t err = workspaces().take(total, s, &block);
    if (err != hipSuccess) return CADNN_ENOMEM;         // (the caller goes on with the kernels on planes)
    char* const ws = block.p;
    c.plan = &plan;
    c.x = ws;
    c.xd = xd;
    c.w = ws + x_bytes;
    c.part = (float*)(ws + x_bytes + align256(c.w_bytes));
    c.count = (int*)(ws + x_bytes + align256(c.w_bytes) + align256(part));
    c.planes = true;
    c.y = y;
    c.residual = residual;
    c.bias = (const float*)bias;
    c.n = n;
    c.cout = cout;
    c.stride = stride;
    c.pad = pad;
    c.relu = relu ? 1 : 0;

    ClArrange a{};
    a.x = x;
    a.xr = ws;
    a.xd = xd;
    a.positions = (h + 2 * pad) * (w + 2 * pad);
    a.pos_blocks = (a.positions + 63) / 64;
    a.ch_blocks = (xd.pix + 63) / 64;
    a.x_blocks = a.pos_blocks * a.ch_blocks * n;
    a.w = w_dev;
    a.wr = (void*)c.w;
    a.cin = cin; a.cout = cout; a.taps = plan.taps; a.steps_tap = plan.steps_tap; a.kpr = kpr; a.pieces = pieces;
    a.count = c.count;
    a.ncount = (int)(count / 4);
    const unsigned blocks = (unsigned)(a.x_blocks + (cout + 3) / 4 * plan.steps_tap);
    const size_t lds = std::max<size_t>(64 * (64 + 16 / e), 4 * (size_t)kpr * (size_t)plan.taps) * e;
    if (f16) CADNN_LAUNCH(cl_arrange_kernel<_Float16>, dim3(blocks), dim3(256), lds, s, a);
    else CADNN_LAUNCH(cl_arrange_kernel<float>, dim3(blocks), dim3(256), lds, s, a);
    err = hipGetLastError();
    cadnn_status st = CADNN_OK;
    if (err == hipSuccess) st = launch_cl_conv(c, *v, f16, s);
    const hipError_t freed = workspaces().give(block, s);
    CADNN_HIP(err);
    if (st != CADNN_OK) return st;
    CADNN_HIP(freed);
    return CADNN_OK;
}

}  // namespace cadnn
