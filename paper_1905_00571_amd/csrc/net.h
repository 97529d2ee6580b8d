// The net runner's data: ops, their layouts, and the opaque cadnn_net itself.
#pragma once

#include "channels_last.h"

namespace cadnn {

enum OpKind { OP_CONV, OP_FC, OP_MAXPOOL, OP_AVGPOOL, OP_DEPTHWISE, OP_AVGPOOL2D, OP_CONCAT };

struct Shape {
    int n = 0, c = 0, h = 0, w = 0;
    size_t elems() const { return (size_t)n * c * h * w; }
    bool operator==(const Shape& o) const { return n == o.n && c == o.c && h == o.h && w == o.w; }
};

// Where a tensor lives: -1 = the caller's x, -2 = the caller's y, otherwise the output of
// op `inst` inside the workspace.  Every op output has a region of its own, so a halo
// that is zeroed once stays zero (kernels only write the image proper).
struct NetOp {
    OpKind kind;
    const cadnn_weights* w = nullptr;
    const void* bias = nullptr;
    int stride = 1, pad = 0, relu = 0, k = 0;
    int src = 0, dst = 0, res = -1;          // buffer ids as given by the caller
    Shape in, out;
    int src_inst = -1, res_inst = -1;        // producing op of each input (-1 = net input)
    TensorDesc xd, yd, rd;
    size_t y_off = 0;                        // byte offset of this op's output region
    int shortcut = -1;                       // conv: the 1x1 projection op fused into this one
    int pool_op = -1;                        // conv: the global average pool op fused into this one
    int dw_op = -1;                          // conv: the depthwise op fused into this one
    int fused_into = -1;                     // projection / pool / depthwise: the op that now computes it (it is skipped)
    // concatenation: its sources (src / src_inst repeat the first), the first output channel of
    // each, and whether the source's producer writes its slice of this op's region itself
    std::vector<int> srcs, src_insts, ch_off;
    std::vector<char> in_place;
    int slice_of = -1;                       // producer: the concatenation whose region it writes into ...
    int slice_ch = 0;                        // ... starting at this channel
    // 1x1 layers that read the same tensor pixel by pixel are merged into ONE launch with the
    // rows of all of them (a horizontal fusion): the first carries the others as `siblings`
    // and writes a region with the channels of all; a sibling is skipped (fused_into = the
    // first) and its output is the channel slice [sib_ch, sib_ch + cout) of that region
    std::vector<int> siblings;
    int sibling_of = -1, sib_ch = 0, launch_c = 0;   // launch_c: channels the launch writes (own + siblings')
    // Independent layers (different inputs, different weights) whose inputs are all ready when
    // the first of them runs are launched with it as ONE kernel: the first carries the others
    // as `comates`; a comate is skipped (fused_into = colaunch_of = the first).  Its tensors are
    // its own, untouched by this.
    std::vector<int> comates;
    int colaunch_of = -1;
    // A window pool is launched right after the op that completes its input (hoisted_to; that op
    // lists it in `hoisted`) instead of at its place in the op list, so that the layer reading
    // it can join the launch of layers that come before the pool in the list.  The members of
    // a group that tuning disbanded stay behind its first op the same way.
    int hoisted_to = -1;
    std::vector<int> hoisted;
    // A large stride-2 layer with a filter wider than 1x1 whose input could not be kept
    // de-interleaved where it is produced (odd sizes, other readers, a concatenation) reads a
    // de-interleaved copy made right before it: xd describes the copy at x_off, src_d the
    // tensor it is made from.
    bool restaged = false;
    size_t x_off = 0;
    TensorDesc src_d;
};

// The one kernel of a group of co-launched layers: the variant that serves them all and the
// members' launch records in device memory (with the plans they point into).
struct CoLaunch {
    const ConvVariant* v = nullptr;
    DevBuf table;
    std::vector<std::shared_ptr<ConvPlan>> plans;
    std::vector<ConvLaunch> records;   // host copy of the table (the launch derives the grid from it)
};

// The channels-last execution of a net (net_cl.cpp): every tensor [row][column][channel], every
// convolution an implicit GEMM on the matrix cores.  It stands beside the plane (NCHW) execution: a
// net uses one or the other as a whole.
struct ClOp {
    ClDesc xd, yd, rd;                       // input (an import of the caller's x included), output, residual
    size_t x_off = 0, y_off = 0;             // byte offsets in the workspace (y_off of a flat last op: the caller's y)
    bool x_stem = false;                     // the input is the op's own packed copy of the caller's x, at x_off
    bool flat = false;                       // the output is [n][c][h][w] without padding (read by an FC layer, or y itself)
    int slice_of = -1;                       // writes its channels into that concatenation's region
    int shortcut = -1;                       // projection op fused into this convolution
    int fused_into = -1;                     // projection: the convolution that computes it
    ClPlan plan;
    DevBuf dw;                               // depthwise: the filters, [tap][channel]
    const ClVariant* v = nullptr;
};
struct ClNet {
    std::vector<std::unique_ptr<ClOp>> ops;
    size_t ws_bytes = 0;
    int import_at = -1;                      // the op ahead of which the caller's x is brought into `in_d` at in_off
    ClDesc in_d;
    size_t in_off = 0;
};

// Launches of a pass, numbered in launch order, that are replayed as a graph.
struct GraphRange { size_t first = 0, last = 0; };

}  // namespace cadnn

struct cadnn_net {
    cadnn_dtype dtype = CADNN_F32;
    cadnn::Shape input;
    std::vector<cadnn::NetOp> ops;
    std::map<int, cadnn::Shape> cur;        // shape currently held by each buffer id while building
    std::map<int, int> producer;     // op that last wrote each buffer id (-1 = net input)
    size_t ws_bytes = 0;
    bool laid_out = false;
    bool finalized = false;
    bool use_graph = false;
    bool want_tune = false;
    bool allow_s2d = true;
    bool allow_fusion = true;
    char* ws = nullptr;
    char* planes_ws = nullptr;       // the caller's (latest) workspace while the net works in cl_ws
    bool static_ws = false;          // the workspace is the library's static array (CADNN_NET_STATIC_WORKSPACE)
    std::map<int, std::unique_ptr<cadnn_weights>> merged_w;   // per first op of a sibling group
    std::map<int, std::unique_ptr<cadnn::DevBuf>> merged_bias;
    std::map<int, std::unique_ptr<cadnn::CoLaunch>> colaunch;        // per first op of a group of co-launched layers
    std::unique_ptr<cadnn::ClNet> cl;   // set: the net runs channels-last
    cadnn::DevBuf cl_ws;                // workspace of a net that was taken there by pinning a variant
    hipGraphExec_t exec = nullptr;
    cadnn::GraphRange range;            // of the pass as it is now (ranged), kept like the graph itself
    bool ranged = false;
    size_t elem() const { return dtype == CADNN_F16 ? 2 : 4; }
};

namespace cadnn {
// net_cl.cpp.  The layout (host work only; NULL: some op of the net has no channels-last kernel),
// whether it is expected to be the faster one, and the runner's operations on it.
std::unique_ptr<ClNet> cl_layout(const cadnn_net* net);
bool cl_expected_faster(const cadnn_net* net);
cadnn_status cl_prepare(cadnn_net* net);
cadnn_status cl_launch_one(cadnn_net* net, size_t i, const void* x, void* y, hipStream_t s);
cadnn_status cl_tune(cadnn_net* net, const void* x, void* y, hipStream_t s);
void cl_op_info(const cadnn_net* net, size_t i, cadnn_op_info* out);
const char* cl_op_variant(const cadnn_net* net, size_t i);
std::vector<const ClVariant*> cl_candidates(const cadnn_net* net, size_t i);
// Whether variant v would serve convolution i in the layout `cl` (host work only, before anything is prepared).
bool cl_would_serve(const cadnn_net* net, const ClNet& cl, size_t i, const ClVariant& v);
cadnn_status cl_read_buffer(cadnn_net* net, size_t i, void* host_out, size_t bytes);
}  // namespace cadnn
