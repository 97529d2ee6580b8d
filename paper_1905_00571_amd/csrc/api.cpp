// C-ABI entry points for single layers: argument checks, variant selection, launch.
#include <cmath>
#include <cstdlib>
#include <cstring>
#include <algorithm>

#include "internal.h"

using namespace cadnn;

namespace cadnn {

struct ConvGeom {
    int n, stride, pad, hout, wout;
    TensorDesc xd;
    int out_s2d = 0;          // output or residual de-interleaved
    const ConvExtra* ex = nullptr;   // fused 1x1 shortcut
    GeomKey key() const {
        return {n, xd.h, xd.w, stride, pad, xd.ph, xd.pw,
                (xd.s2d ? 1 : 0) | (out_s2d ? 2 : 0) | ((ex && ex->w) ? 4 : 0) | ((ex && ex->pool_y) ? 8 : 0) |
                    ((ex && ex->dw) ? (ex->dw_stride == 2 ? 48 : 16) : 0)};
    }
};

static cadnn_status check_conv(const char* who, const cadnn_weights* w, const TensorDesc& xd, int n,
                               int stride, int pad, ConvGeom* g, int out_s2d = 0, const ConvExtra* ex = nullptr) {
    if (!w) return fail(CADNN_EINVAL, "%s: NULL weight handle", who);
    if (n <= 0 || xd.h <= 0 || xd.w <= 0) return fail(CADNN_EINVAL, "%s: non-positive size", who);
    if (stride <= 0 || pad < 0) return fail(CADNN_EINVAL, "%s: bad stride/pad", who);
    if (xd.c != w->cin) return fail(CADNN_EINVAL, "%s: %d input channels, weights take %d", who, xd.c, w->cin);
    if (desc_too_large(xd)) return fail(CADNN_EUNSUPPORTED, "%s: a channel plane of 2^30 elements or more", who);
    g->n = n; g->stride = stride; g->pad = pad; g->xd = xd; g->out_s2d = out_s2d; g->ex = ex;
    if (ex && !ex->w && !ex->pool_y && !ex->dw) return fail(CADNN_EINVAL, "%s: empty fusion request", who);
    if (ex && ex->dw) {
        const cadnn_weights* d = ex->dw;
        if (ex->w || ex->pool_y) return fail(CADNN_EINVAL, "%s: one fusion at a time", who);
        if (d->cin != 1 || d->cout != w->cout || d->kh != 3 || d->kw != 3 || d->dtype != w->dtype ||
            (ex->dw_stride != 1 && ex->dw_stride != 2))
            return fail(CADNN_EINVAL, "%s: the fused depthwise layer must be 3x3, stride 1 or 2, one filter per output channel", who);
    }
    if (ex && ex->w) {
        if (!ex->x) return fail(CADNN_EINVAL, "%s: NULL fused shortcut", who);
        if (ex->w->kh != 1 || ex->w->kw != 1 || ex->w->cout != w->cout || ex->w->dtype != w->dtype ||
            ex->w->cin != ex->xd.c || ex->stride <= 0)
            return fail(CADNN_EINVAL, "%s: the fused shortcut must be a 1x1 layer of the same type and output channels", who);
        if (ex->xd.image * (int64_t)w->elem() >= 0x7ffffff0ll)
            return fail(CADNN_EUNSUPPORTED, "%s: one image of the shortcut's input is 2 GiB or more", who);
    }
    g->hout = conv_out(xd.h, w->kh, stride, pad);
    g->wout = conv_out(xd.w, w->kw, stride, pad);
    if (g->hout <= 0 || g->wout <= 0) return fail(CADNN_EINVAL, "%s: empty output", who);
    if (n > 65535) return fail(CADNN_EUNSUPPORTED, "%s: batch above 65535", who);
    if (xd.image * (int64_t)w->elem() >= 0x7ffffff0ll ||
        (double)w->cout * ((double)g->hout + 64.0) * ((double)g->wout + 64.0) * (double)w->elem() >= (double)0x7ffffff0ll)
        return fail(CADNN_EUNSUPPORTED, "%s: one image of the tensor is 2 GiB or more", who);
    return CADNN_OK;
}

// K split over workgroups (large-tile matrix-core variants with splitk > 1): the number of
// slices in use -- every slice gets at least one 32-deep step -- the output tiles, and the
// scratch the slices meet in: per (variant, layer geometry), allocated on first use and kept.
struct SplitK { int sk = 1; int64_t tiles = 0; };
static SplitK splitk_of(const ConvVariant& v, const cadnn_weights* w, const ConvGeom& g) {
    SplitK r;
    const int tm = v.rows_per_block(), tn = 64 * v.p;
    r.tiles = (((int64_t)g.n * g.hout * g.wout + tn - 1) / tn) * ((w->cout + tm - 1) / tm);
    const int steps = w->cin / 32 * w->kh * w->kw + ((g.ex && g.ex->w) ? g.ex->w->cin / 32 : 0);
    if (v.splitk > 1 && steps > 0) {
        const int per = (steps + v.splitk - 1) / v.splitk;
        r.sk = (steps + per - 1) / per;
    }
    return r;
}
static cadnn_status ensure_sk_scratch(const cadnn_weights* w, const ConvVariant* v, const ConvGeom& g, ConvLaunch* out) {
    const SplitK k = splitk_of(*v, w, g);
    if (k.sk <= 1) return CADNN_OK;
    float* part = nullptr;
    int* count = nullptr;
    const size_t tile_bytes = (size_t)v->rows_per_block() * 64 * v->p * sizeof(float);
    cadnn_status st = get_sk_scratch(w, v, g.key(), (size_t)k.tiles * k.sk * tile_bytes, (size_t)k.tiles * sizeof(int), &part, &count);
    if (st != CADNN_OK) return st;
    if (out) {
        out->sk = k.sk;
        out->sk_part = part;
        out->sk_count = count;
    }
    return CADNN_OK;
}

static bool variant_fits(const ConvVariant& v, const cadnn_weights* w, const ConvGeom& g, bool any_density = false) {
    if (v.is_f16 != (w->dtype == CADNN_F16)) return false;
    if (v.stride != 0 && v.stride != g.stride) return false;
    if ((w->cout + v.rows_per_block() - 1) / v.rows_per_block() > 65535) return false;
    // de-interleaved tensors and fused shortcuts are understood by the linear-address kernels
    // and by the large-tile matrix-core kernel (which fuses a projection shortcut as more of
    // K); the wide-tile family computes every address through the general layout function, so
    // it reads and writes de-interleaved tensors as well, and fuses nothing
    const bool wide_dense = v.family == FAM_DENSE && v.tw == 128;
    if (g.ex && v.family != FAM_LINEAR && !(wide_dense && g.ex->w && !g.ex->pool_y && !g.ex->dw)) return false;
    if ((g.xd.s2d || g.out_s2d) && v.family != FAM_LINEAR && v.family != FAM_WTILE && !wide_dense) return false;
    if (v.family == FAM_DENSE) {
        const bool dense_enough = (double)w->nnz >= 0.25 * (double)w->cout * w->cin * w->kh * w->kw;
        const int64_t pixels = (int64_t)g.n * g.hout * g.wout;
        // in 2-byte storage a candidate for the measured selection at any density, once the batch
        // of pixels gives the matrix cores a few tiles
        const bool by_tuning = v.is_f16 && pixels >= 96;
        if (!wide_dense) return any_density || dense_enough || by_tuning;
        int64_t in_bytes = g.xd.image * 2 * g.n;
        if (g.ex) {
            // (a de-interleaved shortcut input is handed over as the plain view of one phase)
            if (g.ex->w->cin % 32 != 0 || (g.ex->xd.s2d && g.ex->stride != 2)) return false;
            in_bytes = std::max<int64_t>(in_bytes, g.ex->xd.image * 2 * g.n);
        }
        if (!dense_wide_serves(v.is_f16, w->cin, w->kh * w->kw, in_bytes,
                               (int64_t)w->cout * (g.hout + 64) * (g.wout + 64) * 2 * g.n, pixels))
            return false;
        // few input channels: K is walked with a table of offsets by the 64-pixel tiles, on plain
        // tensors, with nothing fused and K in one piece
        if (w->cin % 32 != 0 && (v.p != 1 || g.ex || g.xd.s2d || v.splitk > 1)) return false;
        // a de-interleaved input is walked phase by phase (stride 2, taps starting inside the
        // halo) or pixel by pixel (stride 1, 1x1)
        if (g.xd.s2d && !(g.stride == 2 ? (g.xd.ph >= g.pad && g.xd.pw >= g.pad) : (g.stride == 1 && w->kh * w->kw == 1 && g.pad == 0)))
            return false;
        if (v.splitk > 1) {
            // K is split over workgroups where the tiles alone leave most of the chip idle and
            // every slice still gets a few stages; the scratch stays below 256 MiB
            const SplitK k = splitk_of(v, w, g);
            const int steps = w->cin / 32 * w->kh * w->kw + (g.ex ? g.ex->w->cin / 32 : 0);
            if (k.sk != v.splitk || k.tiles > 384 || steps < 8 * v.splitk ||
                k.tiles * k.sk * (int64_t)v.rows_per_block() * 64 * v.p * 4 > (256ll << 20))
                return false;
        }
        return any_density || dense_enough || by_tuning;
    }
    if (v.family == FAM_LINEAR) {
        const bool one = w->kh == 1 && w->kw == 1;
        if (g.xd.s2d) {
            // a stride-2 layer walks one phase per tap with unit stride (for filters larger
            // than 1x1 the taps must start on an even padded position); a stride-1 layer can
            // only be pixel-wise
            if (g.stride == 2) {
                if (!one && (((g.xd.ph - g.pad) & 1) || ((g.xd.pw - g.pad) & 1))) return false;
            } else if (g.stride != 1 || !one) {
                return false;
            }
        }
        // Writing a de-interleaved tensor, or reading one pixel by pixel, takes the
        // instantiations with the general address arithmetic; a stride-2 layer on a
        // de-interleaved input is handed a plain view of the phase it starts in.
        const bool general = g.out_s2d || (g.xd.s2d && g.stride == 1);
        if (general != (v.s2d != 0)) return false;
        // several rows per wave: the whole image in a row's share of the lanes, nothing fused
        if (v.quad && (g.ex || g.hout * ((g.wout + v.p - 1) / v.p) > 64 / v.rpw)) return false;
        // a fused shortcut takes the dual-input instantiations; its input must be walkable
        // with one stride (plain layout, or de-interleaved and read with stride 2)
        const bool shortcut = g.ex && g.ex->w, pooled = g.ex && g.ex->pool_y, dwf = g.ex && g.ex->dw;
        if (shortcut != (v.dual != 0) || pooled != (v.pool != 0) || dwf != (v.dw != 0)) return false;
        // a fused depthwise layer needs the whole image, at most 16 x 16, in one pixel tile
        // (one wavefront's pixels, or -- tile-per-wave instantiations -- those of all the waves of a workgroup)
        if (dwf && (general || g.hout * g.wout > 64 * v.p * (v.dw == 2 ? v.tw : 1) || g.hout > 28 || g.wout > 28)) return false;
        // a fused pool needs the whole image in one pixel tile of the variant
        if (pooled && (general || shortcut || g.hout * g.wout > 64 * v.p)) return false;
        if (shortcut) {
            if (general) return false;
            if (g.ex->xd.s2d && g.ex->stride != 2) return false;
            const int unit2 = g.ex->xd.s2d ? 2 : 1;
            if (v.adjacent && g.ex->stride != unit2) return false;
        }
        // a lane's adjacent pixels must be adjacent in memory, on both sides; rows that split
        // evenly into groups take the plain instantiations, the others the ragged-row ones
        const int unit = g.xd.s2d ? 2 : 1;
        if (v.adjacent && (g.stride != unit || (!v.quad && (g.wout % v.p != 0) != (v.adjacent == 2)))) return false;
        // The last group of a ragged row reads up to P-1 elements past its row.  Past the end
        // of the image that reads as zero dword by dword, which is fine for 4-byte storage; in
        // 2-byte storage the dword holding the image's last element would be dropped whole,
        // so there the input must end in a halo row instead.
        if (v.adjacent == 2 && v.is_f16 && g.xd.ph < 1 && !(v.quad && g.wout % v.p == 0)) return false;
        // 1x1 filters read only the image proper; larger filters need the zero halo
        if (one) return g.pad == 0;
        return g.xd.ph >= g.pad && g.xd.pw >= g.pad;
    }
    if (v.family == FAM_PTILE) {
        // staging pays only when a staged element is reused by several taps
        if (w->kh * w->kw == 1) return false;
        const PtileGeom pg = ptile_geom(v, w->cin, w->kh, w->kw, g.stride, g.pad, g.wout);
        return pg.nstp <= kPtileMaxSteps && (int64_t)pg.plane * 4 <= (int64_t)kLdsBytesPerCU;
    }
    if (v.family == FAM_WTILE) {
        // pixel-wise layers take the flattened-pixel instantiations, filters with taps the lane grids
        if ((w->kh * w->kw == 1) != (v.flat != 0)) return false;
        if (v.flat && g.pad != 0) return false;
        const WtileGeom wg = wtile_geom(v, w->cin, w->kh, w->kw, g.stride);
        if (wg.nstp > kWtileMaxSteps || wg.lds_bytes > kLdsBytesPerCU) return false;
        // a flattened tile runs over the images of the batch: the whole tensor behind one 32-bit offset
        if (v.flat && (g.xd.image * (int64_t)w->elem() * g.n >= 0x7ffffff0ll ||
                       (int64_t)w->cout * (g.hout + 64) * (g.wout + 64) * (int64_t)w->elem() * g.n >= 0x7ffffff0ll))
            return false;
        return true;
    }
    if (v.kh != w->kh || v.kw != w->kw) return false;
    // the wave-sliced LDS kernel buffers the stream of a (row group, channel chunk)
    return v.family != FAM_STILE || stile_streams_fit(w, &v);
}

static std::vector<const ConvVariant*> candidates(const cadnn_weights* w, const ConvGeom& g) {
    std::vector<const ConvVariant*> out;
    for (const ConvVariant& v : all_linear_variants()) if (variant_fits(v, w, g)) out.push_back(&v);
    for (const ConvVariant& v : all_quad_variants()) if (variant_fits(v, w, g)) out.push_back(&v);
    for (const ConvVariant& v : all_direct_variants()) if (variant_fits(v, w, g)) out.push_back(&v);
    for (const ConvVariant& v : all_tile_variants()) if (variant_fits(v, w, g)) out.push_back(&v);
    for (const ConvVariant& v : all_dense_variants()) if (variant_fits(v, w, g)) out.push_back(&v);
    for (const ConvVariant& v : all_dense_wide_variants()) if (variant_fits(v, w, g)) out.push_back(&v);
    for (const ConvVariant& v : all_stile_variants()) if (variant_fits(v, w, g)) out.push_back(&v);
    for (const ConvVariant& v : all_ptile_variants()) if (variant_fits(v, w, g)) out.push_back(&v);
    for (const ConvVariant& v : all_wtile_variants()) if (variant_fits(v, w, g)) out.push_back(&v);
    // No sparse kernel is instantiated for the geometry (say a 5x5 or a stride-3 7x7 filter on
    // an input without halo): the matrix-core kernel, which takes any geometry, serves it
    // whatever the density, so that every valid layer runs.
    if (out.empty())
        for (const ConvVariant& v : all_dense_variants()) if (variant_fits(v, w, g, true)) out.push_back(&v);
    return out;
}

// Default choice when nothing was tuned or pinned: a model of one launch in microseconds, over a few quantities of it:
//   fixed: 1, and the levels of a split row's reduction;
//   a wave's own latency: the rounds of workgroups a CU runs one after the other, and per round the channel chunks staged,
//   the nonzeros a wave walks and the LDS words it stages;
//   what all waves together issue: the waves of the launch per SIMD, times the nonzeros, times the words.
// The staging-free families have cache lines read in place of the words; the matrix-core kernels K steps as their latency
// and blocks, and blocks times steps, as what is issued (steps once more where the input channels are not whole ones).
// A layer on plain or haloed tensors: the fixed terms plus the cube root of the sum of the cubes of the other
// two (a launch is bound by the longer of the two, and near the crossing by both), with constants per variant,
// fitted to the tuner's times on 8557 layers of 16 to 512 channels, 1x1 to 7x7, both storage types, batch 1 to 16, and on
// the layers of VGG-16, Inception-V3 and ResNet-50.  100 of the 446 variants are modelled: no more of them are worth
// having (all of them: 1.042 times the best variant's time on layers that were not fitted, in the geometric mean;
// these: 1.043; with one set of constants per family and pixels per lane, fitted to 230 layers: 1.10, and 5 % of
// the layers more than a fifth slower than with the choice before that, which knew the staging-free families
// alone and took 1.66 times the best on average.  0.4 % are now).
struct VariantCost { const char* name; float c[9]; };
constexpr VariantCost kVariantCosts[] = {
    {"dense_mfma__Float16_128x64x32_h1", {11.1f, 1.37f, 0.59f, 0.118f, 0.392f, 0.0668f, 0, 0, 0}},
    {"dense_mfma__Float16_64x128x32_h1", {11.8f, 0.369f, 0.594f, 0.147f, 0, 0, 0, 0, 0}},
    {"dense_mfma__Float16_64x64x32", {8.56f, 0.78f, 1.87f, 0.687f, 0.166f, 0, 0, 0, 0}},
    {"dense_mfma__Float16_64x64x32w", {10.2f, 1.11f, 0.457f, 0.195f, 0.456f, 0.154f, 0, 0, 0}},
    {"dense_mfma__Float16_64x64x32w_h1", {9.43f, 1.06f, 0.514f, 0.188f, 0.415f, 0.138f, 0, 0, 0}},
    {"dense_mfma_float_64x64x32", {8.27f, 0.994f, 1.88f, 1.2f, 0, 0, 0, 0, 0}},
    {"sconv__Float16_k7x7s1_t32p2_w4r4c4", {13.2f, 0, 0, 0.0453f, 0.278f, 0, 0, 0, 0}},
    {"sconv_float_k7x7s1_t32p2_w4r4c4", {11.7f, 0, 0, 0.0464f, 0.278f, 0, 0, 0, 0}},
    {"sdirect__Float16_k3x3_p1_r1k1w4", {8.9f, 0, 0.102f, 0, 0.167f, 0, 0.372f, 0, 0}},
    {"sdirect__Float16_k3x3_p1_r1k4w4", {8.13f, 0, 0, 0.0471f, 0.298f, 0, 0.396f, 0.0226f, 0}},
    {"sdirect__Float16_k3x3_p1_r1k8w8", {7.97f, 0, 0, 0.0303f, 0.32f, 0, 0.44f, 0.00968f, 0}},
    {"sdirect_float_k3x3_p1_r1k1w4", {9.05f, 0, 0, 0.0541f, 0.0917f, 0, 0.429f, 0, 0}},
    {"sdirect_float_k3x3_p1_r1k4w4", {8.25f, 0, 0, 0.0493f, 0.276f, 0, 0.463f, 0.0135f, 0}},
    {"sdirect_float_k3x3_p1_r1k8w8", {0.0408f, 0, 0.0565f, 0.00055f, 0.303f, 0, 0.516f, 2.74f, 0}},
    {"slinear__Float16_a2_r1k1w4u8", {5.91f, 0.0138f, 0.00137f, 0.0262f, 0.166f, 0, 0.202f, 0, 0}},
    {"slinear__Float16_a2_r1k2w4u8", {3.36f, 0.15f, 0.0132f, 0.0202f, 0.173f, 0.00208f, 0.141f, 2.38f, 0}},
    {"slinear__Float16_a2_r1k8w8u4", {0, 0.123f, 0, 0.0302f, 0.184f, 0.00118f, 0.0684f, 1.85f, 0}},
    {"slinear__Float16_p1_r1k2w4u8", {5.64f, 0.443f, 0, 0.0175f, 0.0113f, 0, 0.519f, 0, 0}},
    {"slinear__Float16_p1_r1k4w4u8", {5.68f, 0.427f, 0, 0, 0.0544f, 0, 0.521f, 0, 0}},
    {"slinear__Float16_p1_r1k8w8u4", {5.68f, 0.271f, 0, 0, 0.0602f, 0, 0.511f, 0, 0}},
    {"slinear__Float16_p2_r1k1w4u4", {6.01f, 0, 0.087f, 0, 0.116f, 0, 0.438f, 0, 0}},
    {"slinear__Float16_p2_r1k4w4u4", {0.379f, 0, 0.0905f, 0, 0.137f, 0, 0.385f, 2.76f, 0}},
    {"slinear__Float16_p2_r2k1w4u4", {6.34f, 0, 0.0837f, 0.0047f, 0.173f, 0, 0.466f, 0, 0}},
    {"slinear__Float16_p4_r4k1w4u2", {8.79f, 0, 0.12f, 0, 0.318f, 0, 0.522f, 0, 0}},
    {"slinear_float_a4_r1k2w4u4", {0.507f, 0.326f, 0.0726f, 0.00289f, 0.275f, 0.0353f, 0, 5.49f, 0}},
    {"slinear_float_d1_r1k1w4u8", {4.86f, 0.181f, 0, 0.0306f, 0.256f, 0.0044f, 0.413f, 0, 0}},
    {"slinear_float_d1_r1k4w4u8", {0.269f, 0.327f, 0.0102f, 0.0421f, 0.214f, 0.00615f, 0.21f, 2.02f, 0}},
    {"slinear_float_g4_r1k1w4u4", {6.33f, 0.156f, 0.000232f, 0.0413f, 0.366f, 0.0386f, 0, 0, 0}},
    {"slinear_float_g4_r1k2w4u4", {0.204f, 0.248f, 0.0726f, 0.000373f, 0.252f, 0.0367f, 0, 5.87f, 0}},
    {"slinear_float_g4_r1k4w4u8", {4.15f, 0.292f, 0.0774f, 0, 0.315f, 0.0319f, 0, 0.901f, 0}},
    {"slinear_float_p1_r1k16w16u4", {0.0386f, 0.429f, 0, 0, 0.12f, 0, 0.497f, 1.36f, 0}},
    {"slinear_float_p1_r1k1w4u4", {5.97f, 0, 0, 0.0364f, 0.105f, 0, 0.415f, 0, 0}},
    {"slinear_float_p1_r1k1w4u8", {5.92f, 0, 0, 0.0248f, 0.108f, 0, 0.475f, 0, 0}},
    {"slinear_float_p1_r1k4w4u8", {4.52f, 0.433f, 0, 0, 0.051f, 0, 0.558f, 0.595f, 0}},
    {"slinear_float_p2_r1k1w4u4", {6.13f, 0, 0.000437f, 0.0436f, 0.116f, 0, 0.471f, 0, 0}},
    {"slinear_float_p4_r4k1w4u2", {8.23f, 0, 0, 0.0851f, 0.343f, 0, 0.546f, 0, 0}},
    {"sptile__Float16_p1_r1k16w16u4", {0, 2.76f, 0, 0.0526f, 0.224f, 0.663f, 0.00326f, 0.0208f, 1.49f}},
    {"sptile__Float16_p1_r1k2w16u4", {0.149f, 2.19f, 0, 0.0528f, 0.265f, 0.917f, 0.00433f, 0.0299f, 6.05f}},
    {"sptile__Float16_p1_r1k4w16u4", {0.218f, 2.65f, 0, 0.0534f, 0.245f, 0.798f, 0.00341f, 0.0217f, 2.76f}},
    {"sptile__Float16_p1_r1k8w16u4", {0.265f, 2.83f, 0, 0.054f, 0.229f, 0.731f, 0.00207f, 0.0222f, 1.81f}},
    {"sptile__Float16_p2_r1k1w16u4", {8.88f, 0.522f, 0, 0.0605f, 0.326f, 1.18f, 0.00449f, 0.0402f, 0}},
    {"sptile__Float16_p2_r1k2w16u4", {7.11f, 2.6f, 0, 0.0611f, 0.286f, 1.14f, 0.00641f, 0.0242f, 0.0517f}},
    {"sptile__Float16_p2_r1k4w16u4", {0, 2.74f, 0.266f, 0.0602f, 0.258f, 1.08f, 0.00662f, 0.0147f, 3.36f}},
    {"sptile__Float16_p2_r1k8w16u4", {0.213f, 2.59f, 0.75f, 0.0579f, 0.235f, 1.01f, 0.00975f, 0, 2.07f}},
    {"sptile__Float16_v2_r4k1w16u4", {10.9f, 0, 0, 0.0518f, 0.35f, 1.44f, 0.00497f, 0.0896f, 0}},
    {"sptile_float_p1_r1k1w16u4", {8.55f, 0, 0, 0.0487f, 0.154f, 0.723f, 0.00219f, 0.00281f, 0}},
    {"sptile_float_p1_r1k2w16u4", {0, 1.99f, 0.474f, 0.0523f, 0.103f, 0.733f, 0.00445f, 0.0239f, 6.02f}},
    {"sptile_float_p1_r1k4w16u4", {5.61f, 2.41f, 0.476f, 0.0528f, 0.0939f, 0.591f, 0.00386f, 0.026f, 0}},
    {"sptile_float_p1_r1k8w16u4", {5.58f, 2.39f, 0.502f, 0.0528f, 0.0962f, 0.494f, 0.00318f, 0.0242f, 0.00893f}},
    {"sptile_float_p1_r1k8w8u4", {6.48f, 1.72f, 0, 0.032f, 0.0685f, 0.501f, 0.00808f, 0.0182f, 0.0108f}},
    {"sptile_float_p2_r1k16w16u4", {7.19f, 1.52f, 0.621f, 0.0469f, 0.0954f, 0, 0.013f, 0.0261f, 0.00486f}},
    {"sptile_float_p2_r1k1w16u4", {9.4f, 0, 0, 0.0604f, 0.158f, 0.7f, 0.0033f, 0.021f, 0}},
    {"sptile_float_p2_r1k2w16u4", {8.89f, 0, 0.218f, 0.0609f, 0.128f, 0.649f, 0.00341f, 0.028f, 0.0417f}},
    {"sptile_float_p2_r1k4w16u4", {8.04f, 0.563f, 0.281f, 0.0619f, 0.12f, 0.651f, 0, 0.0211f, 0}},
    {"sptile_float_p2_r1k8w16u4", {7.31f, 1.32f, 0.698f, 0.0527f, 0.0925f, 0, 0.0105f, 0.0278f, 0.0148f}},
    {"sptile_float_v2_r1k1w16u4", {9.01f, 0, 0.124f, 0.0578f, 0.13f, 0.688f, 0.00317f, 0.0342f, 0}},
    {"sptile_float_v2_r2k1w16u4", {9.86f, 0, 0, 0.0562f, 0.152f, 1.1f, 0.00276f, 0.0466f, 0}},
    {"sptile_float_v2_r4k1w16u4", {10.3f, 0, 0, 0.0499f, 0.216f, 1.08f, 0.00576f, 0.0675f, 0}},
    {"sptile_float_v4_r1k2w16u4", {2.06f, 3.45f, 0.548f, 0.0909f, 0.0503f, 1.19f, 0.00891f, 0.012f, 4.32f}},
    {"sptile_float_v4_r1k4w16u4", {0.31f, 3.97f, 0.621f, 0.0907f, 0.0455f, 0.995f, 0.00901f, 0.0112f, 2.73f}},
    {"squad__Float16_r2k8g1b16", {0.0258f, 0, 0, 0, 0, 0.0145f, 0.00759f, 2.28f, 0}},
    {"squad_float_r4k2g2b8", {2.41f, 4.22f, 0.148f, 0, 1.22f, 0.0264f, 0.214f, 0.144f, 0}},
    {"stile__Float16_k3x3s1_t16p4_w8g2c8f0", {6.4f, 0.405f, 1.33f, 0.0593f, 0.000166f, 1.25f, 0.0312f, 0.0176f, 0.0117f}},
    {"stile__Float16_k3x3s1_t32p4_w8g8c8f1", {0.0651f, 1.28f, 0, 0.04f, 0.0427f, 2.18f, 0.0233f, 0.019f, 2.71f}},
    {"stile__Float16_k3x3s1_t8p1_w16g16c4f1", {6.44f, 1.84f, 2.37f, 0.0289f, 0.0018f, 1.01f, 0.00508f, 0, 0}},
    {"stile__Float16_k3x3s2_t32p2_w8g8c4f1", {1.16f, 0, 0, 0.0287f, 0.0622f, 1.34f, 0.015f, 0.0326f, 2.0f}},
    {"stile__Float16_k7x7s2_t32p4_w4g4c1f1", {9.68f, 0, 0.955f, 0.0318f, 0.00509f, 0.384f, 0.0187f, 0.021f, 0}},
    {"stile_float_k1x1s2_t32p2_w8g8c16f1", {2.27f, 0.512f, 0.121f, 0.0315f, 0.0132f, 0.293f, 0.0128f, 0.00567f, 1.15f}},
    {"stile_float_k3x3s1_t16p4_w8g1c8f0", {4.87f, 0, 1.43f, 0.0401f, 0.00435f, 1.05f, 0.0229f, 0.0213f, 0.335f}},
    {"stile_float_k3x3s1_t16p4_w8g2c8f0", {0.0707f, 0.596f, 1.16f, 0.055f, 0, 1.38f, 0.028f, 0.017f, 2.04f}},
    {"stile_float_k3x3s1_t8p1_w16g16c4f1", {0.722f, 1.93f, 0, 0.0289f, 0.327f, 1.03f, 0.00507f, 0, 1.3f}},
    {"stile_float_k3x3s1_t8p1_w8g4c16f0", {5.43f, 0.696f, 0, 0.0259f, 0.0396f, 1.34f, 0.014f, 0.0231f, 0.338f}},
    {"stile_float_k3x3s2_t32p2_w8g8c4f1", {0, 1.37f, 1.57f, 0.0255f, 0.00836f, 1.48f, 0.0146f, 0.0284f, 1.95f}},
    {"stile_float_k3x3s2_t8p1_w8g2c8f0", {5.63f, 0, 0, 0.0156f, 0.0559f, 0.621f, 0.012f, 0.033f, 0.00911f}},
    {"stile_float_k7x7s2_t32p4_w4g4c1f1", {1.23f, 0, 0.00818f, 0.0313f, 0.0457f, 0.991f, 0.0154f, 0.0208f, 4.18f}},
    {"swide__Float16_f4_r1w16", {6.86f, 1.12f, 0.852f, 0.0509f, 0.0941f, 0.325f, 0.00169f, 0.0336f, 0}},
    {"swide__Float16_f4_r2w16", {7.2f, 1.4f, 1.44f, 0.0487f, 0.087f, 1.28f, 0.00311f, 0.025f, 0}},
    {"swide__Float16_f4_r4w16", {8.46f, 0.571f, 2.48f, 0.0387f, 0.0713f, 1.65f, 0.00857f, 0.0331f, 0}},
    {"swide__Float16_g4_r1w16l16", {7.09f, 0, 0.389f, 0.0616f, 0.124f, 0.812f, 0.00457f, 0.0314f, 0}},
    {"swide__Float16_g4_r1w16l4", {6.62f, 0, 0.455f, 0.0494f, 0.129f, 0.735f, 0.00504f, 0.0271f, 0}},
    {"swide__Float16_g4_r1w16l8", {7.17f, 0, 0.209f, 0.0618f, 0.14f, 0.83f, 0.00249f, 0.0274f, 0}},
    {"swide__Float16_g4_r1w8l16", {6.85f, 0, 1.15f, 0.0355f, 0.0594f, 0.38f, 0.0111f, 0.0347f, 0}},
    {"swide__Float16_g4_r1w8l4", {6.64f, 0, 1.11f, 0.033f, 0.064f, 0.253f, 0.00978f, 0.0335f, 0}},
    {"swide__Float16_g4_r2w16l16", {7.73f, 0, 0.842f, 0.0584f, 0.12f, 1.09f, 0.00676f, 0.0428f, 0}},
    {"swide__Float16_g4_r2w16l4", {7.29f, 0, 0.869f, 0.0461f, 0.125f, 0.774f, 0.00796f, 0.0337f, 0}},
    {"swide__Float16_g4_r2w16l8", {8.01f, 0, 0.232f, 0.0585f, 0.14f, 0.91f, 0.00564f, 0.0429f, 0}},
    {"swide__Float16_g4_r4w16l4", {8.53f, 0, 1.01f, 0.0342f, 0.157f, 0.94f, 0.0126f, 0.0355f, 0}},
    {"swide_float_f4_r2w16", {6.78f, 1.54f, 1.54f, 0.0437f, 0.0665f, 1.1f, 0.0019f, 0.0421f, 0}},
    {"swide_float_f4_r8w8", {11.0f, 0, 2.48f, 0.0316f, 0.0529f, 3.12f, 0.0104f, 0.0522f, 0}},
    {"swide_float_g4_r1w16l16", {7.01f, 0, 0, 0.0618f, 0.117f, 0.765f, 0.00462f, 0.0313f, 0}},
    {"swide_float_g4_r1w16l4", {6.23f, 0, 0.331f, 0.05f, 0.109f, 0.589f, 0.00392f, 0.0288f, 0}},
    {"swide_float_g4_r1w16l8", {6.9f, 0, 0, 0.0611f, 0.124f, 0.703f, 0.00317f, 0.0284f, 0}},
    {"swide_float_g4_r1w8l16", {6.48f, 0, 1.14f, 0.0367f, 0.0314f, 0.361f, 0.00973f, 0.0328f, 0}},
    {"swide_float_g4_r1w8l4", {6.35f, 0, 1.21f, 0.0333f, 0.0322f, 0.184f, 0.00921f, 0.0294f, 0}},
    {"swide_float_g4_r1w8l8", {6.64f, 0, 0.96f, 0.0366f, 0.0464f, 0.264f, 0.0102f, 0.0306f, 0}},
    {"swide_float_g4_r2w16l16", {7.6f, 0, 0.21f, 0.0575f, 0.128f, 1.09f, 0.00761f, 0.0364f, 0}},
    {"swide_float_g4_r2w16l4", {6.86f, 0, 0.636f, 0.0451f, 0.116f, 0.576f, 0.00704f, 0.0371f, 0}},
    {"swide_float_g4_r2w16l8", {7.6f, 0, 0, 0.057f, 0.134f, 0.759f, 0.00716f, 0.0397f, 0}},
    {"swide_float_g4_r4w16l4", {7.66f, 0, 0.666f, 0.0347f, 0.184f, 0.809f, 0.0117f, 0.034f, 0}},
    {"swide_float_g4_r4w16l8", {7.79f, 0, 1.14f, 0.045f, 0.16f, 1.19f, 0.0135f, 0.0266f, 0}},
};

// Layers with something fused into them, or around de-interleaved tensors: the sum of all terms, with constants per
// family and pixels per lane (fitted to 230 layers, and on the nets' layers 1.08 times the best).
struct FamilyCost { int family, p, kind, f16; float c[9]; };
constexpr FamilyCost kFamilyCosts[] = {
    {FAM_DENSE, 1, 1, 1, {11.8f, 0.846f, 0.474f, 0.0656f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f}},
    {FAM_LINEAR, 1, 0, 0, {5.93f, 0.0f, 0.0156f, 0.0183f, 0.117f, 0.0f, 0.222f, 0.0173f, 0.0f}},
    {FAM_LINEAR, 1, 0, 1, {5.76f, 0.0f, 0.0f, 0.0343f, 0.143f, 0.0f, 0.03f, 0.0f, 0.0f}},
    {FAM_LINEAR, 2, 0, 0, {5.99f, 0.0f, 0.0204f, 0.0295f, 0.136f, 0.0f, 0.237f, 0.0f, 0.0f}},
    {FAM_LINEAR, 2, 0, 1, {5.5f, 0.493f, 0.0569f, 0.0237f, 0.0f, 0.0f, 0.167f, 0.0f, 0.0f}},
    {FAM_LINEAR, 2, 1, 0, {5.91f, 0.0f, 0.0119f, 0.0228f, 0.144f, 0.0183f, 0.0f, 0.0f, 0.0f}},
    {FAM_LINEAR, 2, 1, 1, {5.75f, 0.0f, 0.0147f, 0.0319f, 0.157f, 0.00247f, 0.0f, 0.0f, 0.0f}},
    {FAM_LINEAR, 4, 0, 0, {7.44f, 0.0873f, 0.0935f, 0.00873f, 0.611f, 0.0f, 0.219f, 0.0f, 0.0f}},
    {FAM_LINEAR, 4, 0, 1, {6.71f, 0.18f, 0.127f, 0.0f, 0.733f, 0.0f, 0.272f, 0.0f, 0.0f}},
    {FAM_LINEAR, 4, 1, 0, {6.22f, 0.0f, 0.0159f, 0.0245f, 0.26f, 0.0188f, 0.0f, 0.0f, 0.0f}},
    {FAM_LINEAR, 4, 1, 1, {6.08f, 0.0f, 0.0f, 0.0844f, 0.191f, 0.0143f, 0.0f, 0.0708f, 0.0f}},
    {FAM_LINEAR, 2, 2, 0, {5.85f, 0.517f, 0.0f, 0.0218f, 0.541f, 0.0217f, 0.0f, 0.0f, 0.0f}},
    {FAM_LINEAR, 4, 2, 0, {5.54f, 0.7f, 0.0f, 0.0354f, 0.286f, 0.0163f, 0.0287f, 0.342f, 0.0f}},
    {FAM_WTILE, 4, 16, 0, {8.59f, 0.0f, 1.18f, 0.0245f, 0.0662f, 0.526f, 0.00741f, 0.0f, 0.0f}},
    {FAM_WTILE, 4, 4, 0, {8.32f, 0.0f, 1.22f, 0.0204f, 0.0805f, 0.293f, 0.00506f, 0.0f, 0.0f}},
    {FAM_WTILE, 4, 64, 0, {7.92f, 0.307f, 0.717f, 0.0456f, 0.0614f, 0.592f, 0.0f, 0.0f, 0.0f}},
    {FAM_WTILE, 4, 8, 0, {8.78f, 0.0f, 1.15f, 0.0239f, 0.0765f, 0.345f, 0.00688f, 0.0f, 0.0f}},
    {FAM_WTILE, 4, 16, 1, {8.69f, 0.87f, 0.975f, 0.0175f, 0.113f, 0.0f, 0.00935f, 0.0f, 0.0f}},
    {FAM_WTILE, 4, 4, 1, {8.0f, 0.687f, 1.78f, 0.0154f, 0.0849f, 0.0f, 0.0071f, 0.0f, 0.0f}},
    {FAM_WTILE, 4, 64, 1, {8.9f, 0.0f, 1.5f, 0.0367f, 0.035f, 0.341f, 0.0f, 0.00752f, 0.0f}},
    {FAM_WTILE, 4, 8, 1, {9.29f, 0.267f, 1.57f, 0.0164f, 0.0964f, 0.0f, 0.00959f, 0.0f, 0.0f}},
};

static const VariantCost* modelled_alone(const ConvVariant* v) {
    static const std::map<const ConvVariant*, const VariantCost*> rows = [] {
        std::map<const ConvVariant*, const VariantCost*> m;
        for (const std::vector<ConvVariant>* all : {&all_linear_variants(), &all_quad_variants(), &all_direct_variants(), &all_tile_variants(),
                                                    &all_dense_variants(), &all_dense_wide_variants(), &all_stile_variants(),
                                                    &all_ptile_variants(), &all_wtile_variants()})
            for (const ConvVariant& u : *all)
                for (const VariantCost& c : kVariantCosts)
                    if (std::strcmp(u.name, c.name) == 0) m[&u] = &c;
        return m;
    }();
    auto it = rows.find(v);
    return it == rows.end() ? nullptr : it->second;
}

static double variant_cost(const cadnn_weights* w, const ConvGeom& g, const ConvVariant* v) {
    auto up = [](int64_t a, int64_t b) { return (a + b - 1) / b; };
    const int taps = w->kh * w->kw, S = g.stride;
    const bool dense = v->family == FAM_DENSE, free = v->family == FAM_LINEAR || v->family == FAM_DIRECT;
    // for a pruned layer (whose zeros would meet every activation), and for K split over workgroups, the measured
    // selection decides on the matrix cores
    if (dense && ((double)w->nnz < 0.25 * (double)w->cout * w->cin * taps || v->splitk > 1)) return -1.0;
    const bool alone = !g.ex && !g.xd.s2d && !g.out_s2d;
    const float* m = nullptr;
    if (alone) {
        if (const VariantCost* c = modelled_alone(v)) m = c->c;
    } else {
        const int kind = dense ? v->tw == 128 : v->family == FAM_WTILE ? v->rw : v->family == FAM_LINEAR ? (v->quad ? 2 : v->adjacent != 0) : 0;
        for (const FamilyCost& c : kFamilyCosts)
            if (c.family == v->family && (dense || c.p == v->p) && c.kind == kind && (c.f16 != 0) == v->is_f16) m = c.c;
    }
    if (!m) return -1.0;
    double x[9] = {1.0};
    if (dense) {
        const bool wide = v->tw == 128;
        const int tm = wide ? v->rows_per_block() : 64, tn = wide ? 64 * v->p : 64;
        const int64_t pixels = (int64_t)g.hout * g.wout;
        const double blocks = (double)((wide ? up(pixels * g.n, tn) : up(pixels, tn) * g.n) * up(w->cout, tm));
        const double steps = (double)(wide && w->cin % 32 == 0 ? (int64_t)w->cin / 32 * taps : up((int64_t)w->cin * taps, 32));
        x[3] = blocks / 256.0 * steps * (tm * tn / 4096.0);
        if (alone) {
            x[1] = blocks / 256.0;
            x[2] = steps;
            x[4] = w->cin % 32 ? steps : 0.0;
            x[5] = w->cin % 32 ? x[3] : 0.0;
        } else {
            x[1] = std::max(1.0, blocks / 512.0);
            x[2] = x[1] * steps;
        }
    } else {
        const double nnz_row = (double)w->nnz / w->cout;
        double iters = (v->quad ? 1 : v->rpw) * nnz_row / v->ks;
        const int64_t groups = up(w->cout, v->rows_per_block());
        int64_t tiles, resident, chunks = 0;
        double words = 0.0;                       // 64-word staging steps of a wave
        if (free) {
            const int64_t row = v->adjacent ? up(g.wout, v->p) * v->p : g.wout;
            tiles = (v->quad ? 1 : up(g.hout * row, 64 * v->p)) * g.n;
            resident = 12 / v->nw;
        } else if (v->family == FAM_PTILE) {
            const PtileGeom t = ptile_geom(*v, w->cin, w->kh, w->kw, S, g.pad, g.wout);
            tiles = up(g.wout, t.tile_w) * up(g.hout, t.tile_h) * g.n;
            chunks = t.nchunks;
            words = (double)w->cin * t.nstp / v->nw;
            resident = std::min<int64_t>((int64_t)(kLdsBytesPerCU / std::max<size_t>(t.lds_bytes, 1)), 24 / v->nw);
            iters += 2.0 * v->rpw * (double)chunks;         // (parts are padded)
        } else if (v->family == FAM_WTILE) {
            const WtileGeom t = wtile_geom(*v, w->cin, w->kh, w->kw, S);
            tiles = t.flat ? up((int64_t)g.hout * g.wout * g.n, t.tile_w) : up(g.wout, t.tile_w) * up(g.hout, t.tile_h) * g.n;
            chunks = t.nchunks;
            words = (double)w->cin * t.nstp / v->nw;
            resident = std::min<int64_t>((int64_t)(kLdsBytesPerCU / std::max<size_t>(t.lds_bytes, 1)), 24 / v->nw);
            iters += 2.0 * v->rpw * (double)chunks;
        } else {
            const int th = 64 / v->tw * v->p;
            tiles = up(g.wout, v->tw) * up(g.hout, th) * g.n;
            const double plane = (double)((th - 1) * S + w->kh) * ((v->tw - 1) * S + w->kw);
            const bool split = v->family == FAM_STILE;        // every wave stages its own channels
            chunks = up(w->cin, (int64_t)v->cch * (split ? v->nw : 1));
            words = (split ? (double)chunks * v->cch : (double)w->cin / v->nw) * plane / 64.0;
            resident = 16 / v->nw;
        }
        const int64_t blocks = tiles * groups;
        const double rounds = (double)up(up(blocks, 256), std::max<int64_t>(1, resident)), waves = (double)blocks * v->nw;
        if (free) {
            const double line_bytes = 256.0 * v->p * ((S == 2 && !g.xd.s2d) ? 2.0 : 1.0);
            x[1] = rounds;
            x[2] = rounds * iters / std::sqrt(v->family == FAM_DIRECT ? 4.0 : v->quad ? 16.0 : (double)v->unroll);
            x[3] = rounds * iters;
            x[4] = waves / 1024.0;
            x[5] = waves / 1024.0 * iters;
            x[6] = waves * iters * line_bytes / 32.0 / 256.0 / 1000.0;
            x[7] = std::log2((double)v->ks);
        } else {
            x[1] = rounds;
            x[2] = rounds * (double)chunks;
            x[3] = rounds * iters;
            x[4] = rounds * words;
            x[5] = waves / 1024.0;
            x[6] = waves / 1024.0 * iters;
            x[7] = waves / 1024.0 * words;
            x[8] = std::log2((double)v->ks);
        }
    }
    double us = 0.0, t[9];
    for (int i = 0; i < 9; ++i) us += t[i] = (double)m[i] * x[i];
    if (!alone) return us;
    const double chain = dense ? t[2] + t[4] : t[1] + t[2] + t[3] + (free ? 0.0 : t[4]);
    const double issue = dense ? t[1] + t[3] + t[5] : free ? t[4] + t[5] + t[6] : t[5] + t[6] + t[7];
    return us - chain - issue + std::cbrt(chain * chain * chain + issue * issue * issue);
}

// Layers launched together (FAM_LINEAR only): the variants of one launch are compared by the slowest member in
// cycles, each priced as the largest of a wave's own latency chain times the rounds of waves, the issue slots all waves
// consume, and the L1 cache-line traffic -- fitted to single layers' timings on ResNet-50, VGG-16,
// MobileNet-V1 and Inception-V3.  The model above, its chains' maximum plus what all waves issue, picks worse
// here (Inception-V3 fp32 batch 1: 591 us against 577).
static double group_member_cost(const cadnn_weights* w, const ConvGeom& g, const ConvVariant* v) {
    const double nnz_row = w->cout ? (double)w->nnz / w->cout : 0.0;
    const int P = v->p;
    const double walked = v->adjacent == 2 ? (double)g.hout * ((g.wout + P - 1) / P * P) : (double)g.hout * g.wout;
    const double tiles = std::ceil(walked / (64.0 * P)) * g.n;
    const double waves = tiles * std::ceil((double)w->cout / v->rows_per_block()) * v->nw;
    const double iters = v->rpw * nnz_row / v->ks;
    const double line_bytes = 256.0 * P * ((g.stride == 2 && !g.xd.s2d) ? 2.0 : 1.0);
    const double t_l1 = waves * iters * line_bytes / 32.0 / 256.0;
    const double instrs = v->adjacent ? 3.0 + P : 2.0 + 2.0 * P;
    const double t_issue = waves * (1787.0 + iters * instrs * 1.21) / 1024.0;
    const double per_nz = 77.4 * (1.0 + 0.51 * (P - 1)) / (1.0 + 0.079 * std::log2(v->unroll / 4.0));
    const double t_wave = 382.0 + iters * per_nz + (v->ks > 1 ? 338.0 * std::log2((double)v->ks) : 0.0);
    return std::max(std::max(t_wave * std::ceil(waves / (1024.0 * 2.3)), t_issue), 0.078 * t_l1);
}

static const ConvVariant* heuristic_variant(const cadnn_weights* w, const ConvGeom& g) {
    const std::vector<const ConvVariant*> cand = candidates(w, g);
    if (cand.empty()) return nullptr;
    const double nnz_row = w->cout ? (double)w->nnz / w->cout : 0.0;
    const ConvVariant* best = nullptr;
    double best_cost = 0.0;
    for (const ConvVariant* v : cand) {
        const double cost = variant_cost(w, g, v);
        if (cost < 0.0) continue;   // not modelled: chosen by tuning only
        if (!best || cost < best_cost) { best = v; best_cost = cost; }
    }
    if (!best) {
        // nothing modelled serves the layer (a sparse layer of a geometry that only the matrix cores take): the one
        // whose waves walk the fewest nonzeros each
        for (const ConvVariant* v : cand) {
            const double cost = v->rpw * nnz_row / std::max(v->ks, 1);
            if (!best || cost < best_cost) { best = v; best_cost = cost; }
        }
    }
    return best;
}

// The model runs over some two hundred instantiations, which takes the host longer than a small
// layer takes the GPU: its pick is kept on the handle, per geometry and distance between images (a slice of a wide
// region can be too far apart for kernels that hold a batch behind one 32-bit offset; a pinned
// variant is passed over there for the same reason).  A fused shortcut's own geometry is not part of the key, so
// those picks are not kept.
static const ConvVariant* pick_variant(const cadnn_weights* w, const ConvGeom& g) {
    const GeomKey key = g.key();
    const std::pair<GeomKey, int64_t> spaced(key, g.xd.image);
    const bool keep = !(g.ex && g.ex->w);
    {
        std::lock_guard<std::mutex> lock(w->mu);
        auto it = w->chosen.find(key);
        if (it != w->chosen.end() && variant_fits(*it->second, w, g, true)) return it->second;
        auto kept = w->modelled.find(spaced);
        if (keep && kept != w->modelled.end()) return kept->second;
    }
    const ConvVariant* v = heuristic_variant(w, g);
    if (keep && v) {
        std::lock_guard<std::mutex> lock(w->mu);
        w->modelled[spaced] = v;
    }
    return v;
}

// The launch record of variant v on the layer (builds and uploads the variant's plan on first use).
static cadnn_status make_launch(const cadnn_weights* w, const ConvVariant* v, const ConvGeom& g,
                                const void* x, void* y, const TensorDesc& yd, const void* residual,
                                const TensorDesc& rd, const void* bias, int relu, ConvLaunch* out,
                                std::shared_ptr<ConvPlan>* keep = nullptr) {
    const ConvPlan* plan = nullptr;
    cadnn_status st = get_conv_plan(w, v, g.xd, g.stride, g.pad, g.wout, &plan, g.ex, keep);
    if (st != CADNN_OK) return st;
    ConvLaunch a{};
    a.x = x;
    a.y = y;
    a.bias = (const float*)bias;
    a.residual = residual;
    a.nz = (const uint2*)plan->nz.p;
    a.nz_off = (const uint16_t*)plan->nz_off.p;
    a.seg_ptr = (const int32_t*)plan->seg_ptr.p;
    a.perm = (const int32_t*)plan->perm.p;
    a.xd = g.xd; a.yd = yd; a.rd = rd;
    a.n = g.n; a.cout = w->cout; a.stride = g.stride; a.pad = g.pad; a.relu = relu ? 1 : 0;
    if (g.ex && g.ex->pool_y) {
        a.pool_y = g.ex->pool_y;
        a.pool_scale = 1.0f / (float)(g.hout * g.wout);
    }
    if (g.ex && g.ex->dw) {
        if (!g.ex->dw->dw_ready) return fail(CADNN_EINVAL, "fused depthwise filters were not prepared");
        a.dw_y = g.ex->dw_y;
        a.dw_w = (const float*)g.ex->dw->d_dw.p;
        a.dw_bias = (const float*)g.ex->dw_bias;
        a.dw_yd = g.ex->dw_yd;
        a.dw_stride = g.ex->dw_stride;
        a.dw_relu = g.ex->dw_relu;
    }
    if (g.ex && g.ex->w) {
        // the shortcut's input as a plain view walked with one stride from pixel (0, 0)
        a.x2 = g.ex->x;
        a.bias2 = (const float*)g.ex->bias;
        a.x2d = g.ex->xd;
        a.stride2 = g.ex->stride;
        if (g.ex->xd.s2d) {
            a.x2d.origin = tensor_off(g.ex->xd, 0, 0);
            a.x2d.s2d = 0;
            a.stride2 = 1;
        }
        a.image2_bytes = (uint32_t)(g.ex->xd.image * (int64_t)w->elem());
    }
    if (g.xd.s2d && g.stride == 2 && v->family != FAM_DENSE) {
        // plain view for the kernel: unit stride over the rows of one phase, starting at the
        // position of tap (0, 0) of output pixel (0, 0); the plan's tap offsets pick the phase
        a.xd.origin = tensor_off(g.xd, -g.pad, -g.pad);
        a.xd.s2d = 0;
        a.stride = 1;
        a.pad = 0;
    }
    a.nchunks = plan->nchunks;
    a.kh = w->kh; a.kw = w->kw; a.is_f16 = w->dtype == CADNN_F16;
    a.hwout = g.hout * g.wout;
    a.image_bytes = (uint32_t)(g.xd.image * (int64_t)w->elem());
    if (v->family == FAM_PTILE) {
        const PtileGeom pg = ptile_geom(*v, w->cin, w->kh, w->kw, g.stride, g.pad, g.wout);
        a.tiles_x = (g.wout + pg.tile_w - 1) / pg.tile_w;
        a.tiles_y = (g.hout + pg.tile_h - 1) / pg.tile_h;
        a.pt_pitch = pg.pitch; a.pt_sub = pg.sub; a.pt_plane = pg.plane; a.pt_nphc = pg.nphc;
        a.pt_nph = pg.nphr * pg.nphc; a.pt_in_rows = pg.in_rows; a.pt_in_cols = pg.alias ? pg.in_cols - 1 : pg.in_cols;
        a.pt_cch = pg.cch; a.pt_nstp = pg.nstp; a.pt_nchunks = pg.nchunks;
        a.pt_lds_bytes = (uint32_t)pg.lds_bytes;
        a.pt_nbuf = pg.nbuf;
    } else if (v->family == FAM_WTILE) {
        const WtileGeom wg = wtile_geom(*v, w->cin, w->kh, w->kw, g.stride);
        if (wg.flat) {
            a.tiles_x = (int)(((int64_t)g.n * g.hout * g.wout + wg.tile_w - 1) / wg.tile_w);
            a.tiles_y = 1;
        } else {
            a.tiles_x = (g.wout + wg.tile_w - 1) / wg.tile_w;
            a.tiles_y = (g.hout + wg.tile_h - 1) / wg.tile_h;
        }
        a.wt_tiles = a.tiles_x * a.tiles_y;
        a.wt_lc = wg.lc; a.wt_ns = wg.ns; a.wt_pitch = wg.pitch; a.wt_sub = wg.sub; a.wt_plane = wg.plane;
        a.wt_nphc = wg.nphc; a.wt_nph = wg.nphr * wg.nphc; a.wt_cch = wg.cch; a.wt_nstp = wg.nstp;
        a.wt_nchunks = wg.nchunks; a.wt_nbuf = wg.nbuf;
        a.wt_lds_bytes = (uint32_t)wg.lds_bytes;
        auto magic = [](int d) { return (uint32_t)((((uint64_t)1 << 32) + (uint64_t)d - 1) / (uint64_t)d); };
        a.wt_m_sub = magic(wg.sub); a.wt_m_pitch = magic(wg.pitch); a.wt_m_nphc = magic(wg.nphc);
    } else if (v->family == FAM_TILE || v->family == FAM_STILE) {
        a.tiles_x = (g.wout + v->tw - 1) / v->tw;
        a.tiles_y = (g.hout + v->th - 1) / v->th;
    } else {
        a.wq = (v->family == FAM_LINEAR && v->adjacent == 2) ? (g.wout + v->p - 1) / v->p * v->p : g.wout;
        a.hwq = g.hout * a.wq;
        a.tiles_x = (a.hwq + 64 * v->p - 1) / (64 * v->p);
        if (v->family == FAM_LINEAR && v->dw == 2) a.tiles_x = 1;    // the workgroup's waves are the tiles
        a.tiles_y = 1;
    }
    a.row_groups = plan->rows_padded / v->rows_per_block();
    a.sk = 1;
    if (v->family == FAM_DENSE && v->splitk > 1 && (st = ensure_sk_scratch(w, v, g, &a)) != CADNN_OK) return st;
    *out = a;
    return CADNN_OK;
}

static cadnn_status launch_variant(const cadnn_weights* w, const ConvVariant* v, const ConvGeom& g,
                                   const void* x, void* y, const TensorDesc& yd, const void* residual,
                                   const TensorDesc& rd, const void* bias, int relu, hipStream_t s) {
    ConvLaunch a;
    cadnn_status st = make_launch(w, v, g, x, y, yd, residual, rd, bias, relu, &a);
    if (st != CADNN_OK) return st;
    CADNN_HIP(v->launch(a, s));
    return CADNN_OK;
}

// ---- independent layers in one launch ---------------------------------------------
static cadnn_status check_io(const char* who, const cadnn_weights* w, const ConvGeom& g, const void* x,
                             void* y, const TensorDesc& yd, const void* residual, const TensorDesc& rd);
static cadnn_status member_geom(const ConvMember& m, int n, ConvGeom* g) {
    if (m.pool_kind != 0) {
        // a window pool: only its tensors are checked, it constrains no variant
        if (!m.x || !m.y || m.x == m.y || m.pool_k <= 0 || m.stride <= 0 || m.pad < 0 || m.xd.s2d || m.yd.s2d ||
            m.yd.c != m.xd.c || m.yd.h != conv_out(m.xd.h, m.pool_k, m.stride, m.pad) ||
            m.yd.w != conv_out(m.xd.w, m.pool_k, m.stride, m.pad) || m.yd.h <= 0 || m.yd.w <= 0 || n <= 0)
            return fail(CADNN_EINVAL, "cadnn_net (co-launched layers): bad pool member");
        *g = ConvGeom{};
        return CADNN_OK;
    }
    cadnn_status st = check_conv("cadnn_net (co-launched layers)", m.w, m.xd, n, m.stride, m.pad, g,
                                 m.yd.s2d || (m.residual && m.rd.s2d), nullptr);
    if (st != CADNN_OK) return st;
    return check_io("cadnn_net (co-launched layers)", m.w, *g, m.x, m.y, m.yd, m.residual, m.rd);
}

cadnn_status conv2d_group_candidates(const std::vector<ConvMember>& members, int n,
                                     std::vector<const ConvVariant*>* out, const ConvVariant** pick) {
    out->clear();
    if (pick) *pick = nullptr;
    std::vector<ConvGeom> geoms(members.size());
    for (size_t k = 0; k < members.size(); ++k) {
        cadnn_status st = member_geom(members[k], n, &geoms[k]);
        if (st != CADNN_OK) return st;
    }
    if (members.empty()) return CADNN_OK;
    for (const ConvVariant& v : all_linear_variants()) {   // (the only family that offers it)
        if (!v.launch_multi) continue;
        bool all = true, any = false;
        for (size_t k = 0; k < members.size() && all; ++k) {
            if (members[k].pool_kind != 0) continue;
            any = true;
            all = variant_fits(v, members[k].w, geoms[k]);
        }
        if (all && any) out->push_back(&v);
    }
    // untuned pick: the layers run side by side, so the slowest of them decides
    double best = 0.0;
    for (const ConvVariant* v : *out) {
        double worst = 0.0;
        for (size_t k = 0; k < members.size(); ++k)
            if (members[k].pool_kind == 0) worst = std::max(worst, group_member_cost(members[k].w, geoms[k], v));
        if (pick && (!*pick || worst < best)) { *pick = v; best = worst; }
    }
    return CADNN_OK;
}

cadnn_status conv2d_group_records(const std::vector<ConvMember>& members, int n, const ConvVariant* v,
                                  std::vector<ConvLaunch>* records, std::vector<std::shared_ptr<ConvPlan>>* keep) {
    records->resize(members.size());
    if (keep) keep->assign(members.size(), nullptr);
    if (members.size() > (size_t)kMaxCoLaunch) return fail(CADNN_EINVAL, "cadnn_net: more than %d layers in one launch", kMaxCoLaunch);
    int64_t total = 0;
    if (!v || !v->launch_multi) return fail(CADNN_EINVAL, "cadnn_net: variant cannot launch several layers");
    for (size_t k = 0; k < members.size(); ++k) {
        const ConvMember& m = members[k];
        ConvGeom g;
        cadnn_status st = member_geom(m, n, &g);
        if (st != CADNN_OK) return st;
        if (m.pool_kind != 0) {
            ConvLaunch a{};
            a.x = m.x; a.y = m.y; a.xd = m.xd; a.yd = m.yd; a.n = n; a.stride = m.stride; a.pad = m.pad;
            a.op_type = m.pool_kind; a.pool_k = m.pool_k;
            // the output elements of an image dealt round robin to the threads of at most 256
            // workgroups (one per compute unit)
            const int64_t threads = (int64_t)v->nw * 64;
            a.tiles_x = 1;
            a.tiles_y = 1;
            a.row_groups = (int)std::min<int64_t>(((int64_t)m.yd.c * m.yd.h * m.yd.w + threads - 1) / threads, 256);
            (*records)[k] = a;
            total += (int64_t)a.tiles_x * a.row_groups;
            continue;
        }
        if (!variant_fits(*v, m.w, g)) return fail(CADNN_EINVAL, "cadnn_net: '%s' does not serve every co-launched layer", v->name);
        if ((st = make_launch(m.w, v, g, m.x, m.y, m.yd, m.residual, m.rd, m.bias, m.relu, &(*records)[k],
                              keep ? &(*keep)[k] : nullptr)) != CADNN_OK) return st;
        total += (int64_t)(*records)[k].tiles_x * (*records)[k].row_groups;
    }
    if (n > 65535 || total > 0x7fffffffll)
        return fail(CADNN_EUNSUPPORTED, "cadnn_net: co-launched layers exceed the grid limits");
    return CADNN_OK;
}

// Times every variant that serves all members in one launch, the way conv2d_tune_impl times a
// single layer (caches swept, `before` launched, one event-timed launch per repeat).
cadnn_status conv2d_group_tune(const std::vector<ConvMember>& members, int n, hipStream_t s, int reps,
                               const std::function<cadnn_status()>* before, const ConvVariant** best_v,
                               float* best_us) {
    *best_v = nullptr;
    if (reps <= 0) return fail(CADNN_EINVAL, "cadnn_net: reps must be positive");
    std::vector<const ConvVariant*> cand;
    cadnn_status st = conv2d_group_candidates(members, n, &cand, nullptr);
    if (st != CADNN_OK) return st;
    if (cand.empty()) return CADNN_OK;
    DevBuf sweep;
    const size_t sweep_bytes = (size_t)64 << 20;
    if (hipMalloc(&sweep.p, 2 * sweep_bytes) != hipSuccess) {
        sweep.p = nullptr;
        return fail(CADNN_ENOMEM, "cadnn_net: no memory for the cache sweep buffer");
    }
    sweep.bytes = 2 * sweep_bytes;
    if (hipMemsetAsync(sweep.p, 0, 2 * sweep_bytes, s) != hipSuccess) return fail(CADNN_EHIP, "hipMemsetAsync failed");
    hipEvent_t e0 = nullptr, e1 = nullptr;
    CADNN_HIP(hipEventCreate(&e0));
    if (hipEventCreate(&e1) != hipSuccess) { (void)hipEventDestroy(e0); return fail(CADNN_EHIP, "hipEventCreate failed"); }
    float best_ms = 0.0f;
    std::vector<ConvLaunch> recs;
    const TrialPlans trial;
    for (const ConvVariant* v : cand) {
        if (conv2d_group_records(members, n, v, &recs) != CADNN_OK) continue;   // does not fit these weights
        DevBuf table;
        if ((st = table.upload(recs.data(), recs.size() * sizeof(ConvLaunch))) != CADNN_OK) break;
        const ConvLaunch* tab = (const ConvLaunch*)table.p;
        if (v->launch_multi(tab, recs.data(), (int)recs.size(), n, s) != hipSuccess) { st = fail(CADNN_EHIP, "co-launch failed"); break; }
        float total_ms = 0.0f;
        for (int i = 0; i < reps && st == CADNN_OK; ++i) {
            st = launch_copy(sweep.p, (char*)sweep.p + sweep_bytes, sweep_bytes, s);
            if (st != CADNN_OK) break;
            if (before && (st = (*before)()) != CADNN_OK) break;
            if (hipEventRecord(e0, s) != hipSuccess) { st = fail(CADNN_EHIP, "hipEventRecord failed"); break; }
            if (v->launch_multi(tab, recs.data(), (int)recs.size(), n, s) != hipSuccess) { st = fail(CADNN_EHIP, "co-launch failed"); break; }
            if (hipEventRecord(e1, s) != hipSuccess || hipEventSynchronize(e1) != hipSuccess) { st = fail(CADNN_EHIP, "event wait failed"); break; }
            float ms = 0.0f;
            if (hipEventElapsedTime(&ms, e0, e1) != hipSuccess) { st = fail(CADNN_EHIP, "hipEventElapsedTime failed"); break; }
            total_ms += ms;
        }
        if (st != CADNN_OK) break;
        if (hipStreamSynchronize(s) != hipSuccess) { st = fail(CADNN_EHIP, "hipStreamSynchronize failed"); break; }   // before the table goes
        if (std::getenv("CADNN_TUNE_LOG"))
            std::fprintf(stderr, "[cadnn tune] %zu layers at once %-44s %8.2f us\n", members.size(), v->name, total_ms * 1e3f / reps);
        if (!*best_v || total_ms < best_ms) { *best_v = v; best_ms = total_ms; }
    }
    (void)hipEventDestroy(e0);
    (void)hipEventDestroy(e1);
    if (st != CADNN_OK) return st;
    for (const ConvMember& m : members) if (m.w) drop_unpinned_plans(m.w);
    if (best_us) *best_us = best_ms * 1e3f / reps;
    return CADNN_OK;
}

static cadnn_status check_io(const char* who, const cadnn_weights* w, const ConvGeom& g, const void* x,
                             void* y, const TensorDesc& yd, const void* residual, const TensorDesc& rd) {
    if (!x || !y) return fail(CADNN_EINVAL, "%s: NULL tensor", who);
    if (x == y) return fail(CADNN_EINVAL, "%s: y aliases x", who);
    if (yd.c != w->cout || yd.h != g.hout || yd.w != g.wout) return fail(CADNN_EINVAL, "%s: output layout does not match the layer", who);
    if (residual && (rd.c != w->cout || rd.h != g.hout || rd.w != g.wout))
        return fail(CADNN_EINVAL, "%s: residual layout does not match the output", who);
    return CADNN_OK;
}

cadnn_status conv2d_impl(const cadnn_weights* w, const void* x, const TensorDesc& xd, void* y,
                         const TensorDesc& yd, const void* residual, const TensorDesc& rd, int n,
                         int stride, int pad, const void* bias, int relu, hipStream_t s, const ConvExtra* ex) {
    ConvGeom g;
    cadnn_status st = check_conv("cadnn_sparse_conv2d", w, xd, n, stride, pad, &g, yd.s2d || (residual && rd.s2d), ex);
    if (st != CADNN_OK) return st;
    if ((st = check_io("cadnn_sparse_conv2d", w, g, x, y, yd, residual, rd)) != CADNN_OK) return st;
    const ConvVariant* v = pick_variant(w, g);
    if (!v)
        return fail(CADNN_EUNSUPPORTED, "cadnn_sparse_conv2d: no kernel for %dx%d filters with stride %d",
                    w->kh, w->kw, stride);
    return launch_variant(w, v, g, x, y, yd, residual, rd, bias, relu, s);
}

cadnn_status conv2d_prepare_impl(const cadnn_weights* w, const TensorDesc& xd, int n, int stride, int pad,
                                 int out_s2d, const ConvExtra* ex) {
    ConvGeom g;
    cadnn_status st = check_conv("cadnn_conv2d_prepare", w, xd, n, stride, pad, &g, out_s2d, ex);
    if (st != CADNN_OK) return st;
    const ConvVariant* v = pick_variant(w, g);
    if (!v)
        return fail(CADNN_EUNSUPPORTED, "cadnn_conv2d_prepare: no kernel for %dx%d filters with stride %d",
                    w->kh, w->kw, stride);
    const ConvPlan* plan = nullptr;
    if ((st = get_conv_plan(w, v, xd, g.stride, g.pad, g.wout, &plan, g.ex)) != CADNN_OK) return st;
    return ensure_sk_scratch(w, v, g, nullptr);
}

const char* conv2d_variant_name_impl(const cadnn_weights* w, const TensorDesc& xd, int n, int stride, int pad,
                                     int out_s2d, const ConvExtra* ex) {
    ConvGeom g;
    if (check_conv("cadnn_net_op_variant", w, xd, n, stride, pad, &g, out_s2d, ex) != CADNN_OK) return nullptr;
    const ConvVariant* v = pick_variant(w, g);
    if (!v) {
        (void)fail(CADNN_EUNSUPPORTED, "no kernel for %dx%d filters with stride %d", w->kh, w->kw, stride);
        return nullptr;
    }
    return v->name;
}

cadnn_status conv2d_list_variants_impl(const cadnn_weights* w, const TensorDesc& xd, int n, int stride, int pad,
                                       char* buf, size_t len, int out_s2d, const ConvExtra* ex) {
    if (!buf || len == 0) return fail(CADNN_EINVAL, "cadnn_conv2d_list_variants: NULL buffer");
    ConvGeom g;
    cadnn_status st = check_conv("cadnn_conv2d_list_variants", w, xd, n, stride, pad, &g, out_s2d, ex);
    if (st != CADNN_OK) return st;
    std::string all;
    for (const ConvVariant* v : candidates(w, g)) {
        if (!all.empty()) all += "\n";
        all += v->name;
    }
    if (all.size() + 1 > len) return fail(CADNN_EINVAL, "cadnn_conv2d_list_variants: buffer of %zu bytes, %zu needed", len, all.size() + 1);
    std::memcpy(buf, all.c_str(), all.size() + 1);
    return CADNN_OK;
}

cadnn_status conv2d_set_variant_impl(const cadnn_weights* w, const TensorDesc& xd, int n, int stride, int pad,
                                     const char* name, int out_s2d, const ConvExtra* ex) {
    ConvGeom g;
    cadnn_status st = check_conv("cadnn_conv2d_set_variant", w, xd, n, stride, pad, &g, out_s2d, ex);
    if (st != CADNN_OK) return st;
    std::lock_guard<std::mutex> lock(w->mu);
    if (!name || !*name) {
        w->chosen.erase(g.key());
        return CADNN_OK;
    }
    for (const ConvVariant* v : candidates(w, g)) {
        if (std::strcmp(v->name, name) == 0) {
            w->chosen[g.key()] = v;
            return CADNN_OK;
        }
    }
    return fail(CADNN_EINVAL, "cadnn_conv2d_set_variant: '%s' does not serve this layer", name);
}

cadnn_status conv2d_tune_impl(const cadnn_weights* w, const void* x, const TensorDesc& xd, void* y,
                              const TensorDesc& yd, const void* residual, const TensorDesc& rd, int n,
                              int stride, int pad, const void* bias, int relu, hipStream_t s, int reps,
                              float* best_us, const std::function<cadnn_status()>* before, const ConvExtra* ex) {
    ConvGeom g;
    cadnn_status st = check_conv("cadnn_conv2d_tune", w, xd, n, stride, pad, &g, yd.s2d || (residual && rd.s2d), ex);
    if (st != CADNN_OK) return st;
    if ((st = check_io("cadnn_conv2d_tune", w, g, x, y, yd, residual, rd)) != CADNN_OK) return st;
    if (reps <= 0) return fail(CADNN_EINVAL, "cadnn_conv2d_tune: reps must be positive");
    const std::vector<const ConvVariant*> cand = candidates(w, g);
    if (cand.empty())
        return fail(CADNN_EUNSUPPORTED, "cadnn_conv2d_tune: no kernel for %dx%d filters with stride %d",
                    w->kh, w->kw, stride);
    // Inside a network a layer starts with cold L2 caches: its input was just written by
    // another kernel and its weights were last touched a whole forward pass ago.  Timing
    // back-to-back repeats would reward variants that only do well on cached data, so the
    // L2s are swept with a 64 MiB copy before every timed launch.
    DevBuf sweep;
    const size_t sweep_bytes = (size_t)64 << 20;
    if (hipMalloc(&sweep.p, 2 * sweep_bytes) != hipSuccess) {
        sweep.p = nullptr;
        return fail(CADNN_ENOMEM, "cadnn_conv2d_tune: no memory for the cache sweep buffer");
    }
    sweep.bytes = 2 * sweep_bytes;
    if (hipMemsetAsync(sweep.p, 0, 2 * sweep_bytes, s) != hipSuccess) return fail(CADNN_EHIP, "hipMemsetAsync failed");
    hipEvent_t e0 = nullptr, e1 = nullptr;
    CADNN_HIP(hipEventCreate(&e0));
    if (hipEventCreate(&e1) != hipSuccess) { (void)hipEventDestroy(e0); return fail(CADNN_EHIP, "hipEventCreate failed"); }
    const ConvVariant* best = nullptr;
    float best_ms = 0.0f;
    const TrialPlans trial;
    for (const ConvVariant* v : cand) {
        {
            const ConvPlan* probe = nullptr;
            if (get_conv_plan(w, v, g.xd, g.stride, g.pad, g.wout, &probe, g.ex) == CADNN_EUNSUPPORTED) continue;   // does not fit these weights
        }
        st = launch_variant(w, v, g, x, y, yd, residual, rd, bias, relu, s);
        float total_ms = 0.0f;
        for (int i = 0; i < reps && st == CADNN_OK; ++i) {
            st = launch_copy(sweep.p, (char*)sweep.p + sweep_bytes, sweep_bytes, s);
            if (st != CADNN_OK) break;
            // inside a net: the producer of the input runs right before, as it will
            if (before && (st = (*before)()) != CADNN_OK) break;
            if (hipEventRecord(e0, s) != hipSuccess) { st = fail(CADNN_EHIP, "hipEventRecord failed"); break; }
            st = launch_variant(w, v, g, x, y, yd, residual, rd, bias, relu, s);
            if (st != CADNN_OK) break;
            if (hipEventRecord(e1, s) != hipSuccess || hipEventSynchronize(e1) != hipSuccess) { st = fail(CADNN_EHIP, "event wait failed"); break; }
            float ms = 0.0f;
            if (hipEventElapsedTime(&ms, e0, e1) != hipSuccess) { st = fail(CADNN_EHIP, "hipEventElapsedTime failed"); break; }
            total_ms += ms;
        }
        if (st != CADNN_OK) break;
        const float ms = total_ms;
        if (std::getenv("CADNN_TUNE_LOG"))
            std::fprintf(stderr, "[cadnn tune] cin=%d cout=%d k=%d s=%d hw=%dx%d nnz=%lld %-44s %8.2f us\n", w->cin,
                         w->cout, w->kh, stride, xd.h, xd.w, (long long)w->nnz, v->name, ms * 1e3f / reps);
        if (!best || ms < best_ms) { best = v; best_ms = ms; }
    }
    (void)hipEventDestroy(e0);
    (void)hipEventDestroy(e1);
    if (st != CADNN_OK) return st;
    {
        std::lock_guard<std::mutex> lock(w->mu);
        w->chosen[g.key()] = best;
    }
    drop_unpinned_plans(w);
    if (best_us) *best_us = best_ms * 1e3f / reps;
    return CADNN_OK;
}

}  // namespace cadnn

static TensorDesc out_desc(const cadnn_weights* w, int h, int wdt, int stride, int pad) {
    if (stride <= 0 || pad < 0) return make_desc(0, 0, 0);   // rejected by the argument checks
    return make_desc(w ? w->cout : 0, w ? conv_out(h, w->kh, stride, pad) : 0, w ? conv_out(wdt, w->kw, stride, pad) : 0);
}

extern "C" cadnn_status cadnn_sparse_conv2d(const cadnn_weights* w, const void* x, void* y, int n,
                                            int h, int wdt, int stride, int pad, const void* bias,
                                            const void* residual, int relu, void* stream) {
    const TensorDesc yd = out_desc(w, h, wdt, stride, pad);
    return conv2d_impl(w, x, make_desc(w ? w->cin : 0, h, wdt), y, yd, residual, yd, n, stride, pad, bias,
                       relu, (hipStream_t)stream);
}

extern "C" cadnn_status cadnn_conv2d_tune(const cadnn_weights* w, const void* x, void* y, int n, int h,
                                          int wdt, int stride, int pad, const void* bias,
                                          const void* residual, int relu, void* stream, int reps,
                                          float* best_us) {
    const TensorDesc yd = out_desc(w, h, wdt, stride, pad);
    return conv2d_tune_impl(w, x, make_desc(w ? w->cin : 0, h, wdt), y, yd, residual, yd, n, stride, pad,
                            bias, relu, (hipStream_t)stream, reps, best_us);
}

extern "C" cadnn_status cadnn_conv2d_prepare(const cadnn_weights* w, int n, int h, int wdt,
                                             int stride, int pad) {
    return conv2d_prepare_impl(w, make_desc(w ? w->cin : 0, h, wdt), n, stride, pad);
}

extern "C" cadnn_status cadnn_conv2d_variant_name(const cadnn_weights* w, int n, int h, int wdt,
                                                  int stride, int pad, char* buf, size_t len) {
    if (!buf || len == 0) return fail(CADNN_EINVAL, "cadnn_conv2d_variant_name: NULL buffer");
    ConvGeom g;
    cadnn_status st = check_conv("cadnn_conv2d_variant_name", w, make_desc(w ? w->cin : 0, h, wdt), n, stride, pad, &g);
    if (st != CADNN_OK) return st;
    const ConvVariant* v = pick_variant(w, g);
    if (!v)
        return fail(CADNN_EUNSUPPORTED, "cadnn_conv2d_variant_name: no kernel for %dx%d filters with stride %d",
                    w->kh, w->kw, stride);
    std::strncpy(buf, v->name, len - 1);
    buf[len - 1] = '\0';
    return CADNN_OK;
}

extern "C" cadnn_status cadnn_conv2d_list_variants(const cadnn_weights* w, int n, int h, int wdt,
                                                   int stride, int pad, char* buf, size_t len) {
    return conv2d_list_variants_impl(w, make_desc(w ? w->cin : 0, h, wdt), n, stride, pad, buf, len);
}

extern "C" cadnn_status cadnn_conv2d_set_variant(const cadnn_weights* w, int n, int h, int wdt,
                                                 int stride, int pad, const char* name) {
    return conv2d_set_variant_impl(w, make_desc(w ? w->cin : 0, h, wdt), n, stride, pad, name);
}

// The variant `name` among those that serve the layer (NULL / "": the one that would be launched).
static cadnn_status named_variant(const char* who, const cadnn_weights* w, const ConvGeom& g, const char* name,
                                  const ConvVariant** out) {
    *out = nullptr;
    if (!name || !*name) {
        *out = pick_variant(w, g);
        if (!*out) return fail(CADNN_EUNSUPPORTED, "%s: no kernel for %dx%d filters with stride %d", who, w->kh, w->kw, g.stride);
        return CADNN_OK;
    }
    for (const ConvVariant* v : candidates(w, g))
        if (std::strcmp(v->name, name) == 0) { *out = v; return CADNN_OK; }
    return fail(CADNN_EINVAL, "%s: '%s' does not serve this layer", who, name);
}

extern "C" cadnn_status cadnn_conv2d_plan_info(const cadnn_weights* w, int n, int h, int wdt, int stride, int pad,
                                               const char* variant, cadnn_plan_info* out) {
    if (!out) return fail(CADNN_EINVAL, "cadnn_conv2d_plan_info: NULL pointer");
    ConvGeom g;
    cadnn_status st = check_conv("cadnn_conv2d_plan_info", w, make_desc(w ? w->cin : 0, h, wdt), n, stride, pad, &g);
    if (st != CADNN_OK) return st;
    const ConvVariant* v = nullptr;
    if ((st = named_variant("cadnn_conv2d_plan_info", w, g, variant, &v)) != CADNN_OK) return st;
    ConvPlan plan;
    if ((st = build_host_plan(w, v, g.xd, g.stride, g.pad, g.wout, &plan)) != CADNN_OK) return st;
    cadnn_plan_info info{};
    info.entries = plan.walked;
    info.stream_bytes = plan.walked * plan.entry_bytes;
    info.alloc_bytes = (int64_t)plan.nz.bytes + (int64_t)plan.nz_off.bytes;
    info.table_bytes = (int64_t)plan.seg_ptr.bytes + (int64_t)plan.perm.bytes;
    info.bytes_per_nonzero = w->nnz ? (double)info.stream_bytes / (double)w->nnz : 0.0;
    info.chunks = 1;
    info.lds_bytes = (int)v->lds_bytes;
    if (v->family == FAM_WTILE) {
        const WtileGeom wg = wtile_geom(*v, w->cin, w->kh, w->kw, g.stride);
        info.chunks = wg.nchunks;
        info.lds_bytes = (int)wg.lds_bytes;
    } else if (v->family == FAM_PTILE) {
        const PtileGeom pg = ptile_geom(*v, w->cin, w->kh, w->kw, g.stride, g.pad, g.wout);
        info.chunks = pg.nchunks;
        info.lds_bytes = (int)pg.lds_bytes;
    } else if (v->family == FAM_TILE || v->family == FAM_STILE) {
        info.chunks = plan.nchunks;
    }
    *out = info;
    return CADNN_OK;
}

extern "C" cadnn_status cadnn_conv2d_plan_unpack(const cadnn_weights* w, int n, int h, int wdt, int stride, int pad,
                                                 const char* variant, float* w_host_out) {
    if (!w_host_out) return fail(CADNN_EINVAL, "cadnn_conv2d_plan_unpack: NULL pointer");
    ConvGeom g;
    cadnn_status st = check_conv("cadnn_conv2d_plan_unpack", w, make_desc(w ? w->cin : 0, h, wdt), n, stride, pad, &g);
    if (st != CADNN_OK) return st;
    const ConvVariant* v = nullptr;
    if ((st = named_variant("cadnn_conv2d_plan_unpack", w, g, variant, &v)) != CADNN_OK) return st;
    if (v->family != FAM_WTILE) return fail(CADNN_EUNSUPPORTED, "cadnn_conv2d_plan_unpack: '%s' has no compact tile-offset stream", v->name);
    ConvPlan plan;
    if ((st = build_host_plan(w, v, g.xd, g.stride, g.pad, g.wout, &plan)) != CADNN_OK) return st;
    return wtile_plan_unpack(w, v, g.stride, plan, w_host_out);
}

extern "C" cadnn_status cadnn_sparse_fc(const cadnn_weights* w, const void* x, void* y, int n,
                                        const void* bias, int relu, void* stream) {
    if (!w || !x || !y) return fail(CADNN_EINVAL, "cadnn_sparse_fc: NULL pointer");
    if (n <= 0) return fail(CADNN_EINVAL, "cadnn_sparse_fc: non-positive batch");
    if (w->kh != 1 || w->kw != 1)
        return fail(CADNN_EINVAL, "cadnn_sparse_fc: weights are a %dx%d filter bank", w->kh, w->kw);
    if (n > 8 * 65535) return fail(CADNN_EUNSUPPORTED, "cadnn_sparse_fc: batch too large");
    cadnn_status st = ensure_fc_device(w);
    if (st != CADNN_OK) return st;
    return launch_fc(w, x, y, n, (const float*)bias, relu ? 1 : 0, (hipStream_t)stream);
}

extern "C" cadnn_status cadnn_fc_prepare(const cadnn_weights* w) {
    if (!w) return fail(CADNN_EINVAL, "cadnn_fc_prepare: NULL handle");
    if (w->kh != 1 || w->kw != 1) return fail(CADNN_EINVAL, "cadnn_fc_prepare: weights are not a matrix");
    return ensure_fc_device(w);
}

static cadnn_status check_depthwise(const char* who, const cadnn_weights* w, int n, int h, int wdt, int stride,
                                    int pad) {
    if (!w) return fail(CADNN_EINVAL, "%s: NULL handle", who);
    if (w->cin != 1) return fail(CADNN_EINVAL, "%s: weights have %d input channels per filter, a depthwise filter bank has 1", who, w->cin);
    if (n <= 0 || h <= 0 || wdt <= 0 || stride <= 0 || pad < 0) return fail(CADNN_EINVAL, "%s: bad size", who);
    if (conv_out(h, w->kh, stride, pad) <= 0 || conv_out(wdt, w->kw, stride, pad) <= 0)
        return fail(CADNN_EINVAL, "%s: empty output", who);
    if (desc_too_large(make_desc(1, h, wdt)) || desc_too_large(make_desc(1, conv_out(h, w->kh, stride, pad), conv_out(wdt, w->kw, stride, pad))))
        return fail(CADNN_EUNSUPPORTED, "%s: a channel plane of 2^30 elements or more", who);
    return CADNN_OK;
}

extern "C" cadnn_status cadnn_depthwise_conv2d(const cadnn_weights* w, const void* x, void* y, int n, int h,
                                               int wdt, int stride, int pad, const void* bias, int relu,
                                               void* stream) {
    if (!x || !y) return fail(CADNN_EINVAL, "cadnn_depthwise_conv2d: NULL tensor");
    cadnn_status st = check_depthwise("cadnn_depthwise_conv2d", w, n, h, wdt, stride, pad);
    if (st != CADNN_OK) return st;
    if ((st = ensure_dw_device(w)) != CADNN_OK) return st;
    const TensorDesc xd = make_desc(w->cout, h, wdt);
    const TensorDesc yd = make_desc(w->cout, conv_out(h, w->kh, stride, pad), conv_out(wdt, w->kw, stride, pad));
    return launch_depthwise(w, x, xd, y, yd, n, stride, pad, (const float*)bias, relu ? 1 : 0, (hipStream_t)stream);
}

extern "C" cadnn_status cadnn_depthwise_prepare(const cadnn_weights* w) {
    if (!w) return fail(CADNN_EINVAL, "cadnn_depthwise_prepare: NULL handle");
    if (w->cin != 1) return fail(CADNN_EINVAL, "cadnn_depthwise_prepare: not a depthwise filter bank");
    return ensure_dw_device(w);
}

extern "C" cadnn_status cadnn_device_copy(const void* src, void* dst, size_t bytes, void* stream) {
    if (!src || !dst) return fail(CADNN_EINVAL, "cadnn_device_copy: NULL pointer");
    if (bytes % 16) return fail(CADNN_EINVAL, "cadnn_device_copy: size must be a multiple of 16 bytes");
    return launch_copy(src, dst, bytes, (hipStream_t)stream);
}

// Measurement aid: what one kernel boundary costs inside a replayed HIP graph.  `launches`
// dependent 16-byte copies (the smallest kernel of the library) are captured into one graph,
// which is replayed `reps` times between two events.
extern "C" cadnn_status cadnn_graph_launch_floor(void* scratch32, int launches, int reps, void* stream,
                                                 float* us_per_launch) {
    if (!scratch32 || !us_per_launch) return fail(CADNN_EINVAL, "cadnn_graph_launch_floor: NULL pointer");
    if (launches <= 0 || launches > 4096 || reps <= 0) return fail(CADNN_EINVAL, "cadnn_graph_launch_floor: bad count");
    hipStream_t s = (hipStream_t)stream;
    hipStream_t cs = nullptr;
    CADNN_HIP(hipStreamCreateWithFlags(&cs, hipStreamNonBlocking));
    hipGraph_t graph = nullptr;
    hipGraphExec_t exec = nullptr;
    hipEvent_t e0 = nullptr, e1 = nullptr;
    cadnn_status st = CADNN_OK;
    hipError_t e = hipStreamBeginCapture(cs, hipStreamCaptureModeThreadLocal);
    if (e != hipSuccess) st = fail(CADNN_EHIP, "hipStreamBeginCapture failed: %s", hipGetErrorString(e));
    if (st == CADNN_OK) {
        for (int i = 0; i < launches && st == CADNN_OK; ++i) st = launch_copy(scratch32, (char*)scratch32 + 16, 16, cs);
        e = hipStreamEndCapture(cs, &graph);
        if (st == CADNN_OK && e != hipSuccess) st = fail(CADNN_EHIP, "hipStreamEndCapture failed: %s", hipGetErrorString(e));
    }
    if (st == CADNN_OK && hipGraphInstantiate(&exec, graph, nullptr, nullptr, 0) != hipSuccess) st = fail(CADNN_EHIP, "hipGraphInstantiate failed");
    if (st == CADNN_OK && (hipEventCreate(&e0) != hipSuccess || hipEventCreate(&e1) != hipSuccess)) st = fail(CADNN_EHIP, "hipEventCreate failed");
    if (st == CADNN_OK) {
        bool ok = hipGraphLaunch(exec, s) == hipSuccess && hipEventRecord(e0, s) == hipSuccess;
        for (int r = 0; r < reps && ok; ++r) ok = hipGraphLaunch(exec, s) == hipSuccess;
        ok = ok && hipEventRecord(e1, s) == hipSuccess && hipEventSynchronize(e1) == hipSuccess;
        float ms = 0.0f;
        ok = ok && hipEventElapsedTime(&ms, e0, e1) == hipSuccess;
        if (!ok) st = fail(CADNN_EHIP, "cadnn_graph_launch_floor: replay failed");
        else *us_per_launch = ms * 1e3f / (float)reps / (float)launches;
    }
    if (e0) (void)hipEventDestroy(e0);
    if (e1) (void)hipEventDestroy(e1);
    if (exec) (void)hipGraphExecDestroy(exec);
    if (graph) (void)hipGraphDestroy(graph);
    (void)hipStreamDestroy(cs);
    return st;
}

extern "C" cadnn_status cadnn_maxpool2d(const void* x, void* y, int n, int c, int h, int wdt, int k,
                                        int stride, int pad, cadnn_dtype dtype, void* stream) {
    if (!x || !y) return fail(CADNN_EINVAL, "cadnn_maxpool2d: NULL tensor");
    if (n <= 0 || c <= 0 || h <= 0 || wdt <= 0 || k <= 0 || stride <= 0 || pad < 0)
        return fail(CADNN_EINVAL, "cadnn_maxpool2d: bad size");
    if (dtype != CADNN_F32 && dtype != CADNN_F16) return fail(CADNN_EINVAL, "cadnn_maxpool2d: dtype");
    if (conv_out(h, k, stride, pad) <= 0 || conv_out(wdt, k, stride, pad) <= 0)
        return fail(CADNN_EINVAL, "cadnn_maxpool2d: empty output");
    if (desc_too_large(make_desc(c, h, wdt)) || desc_too_large(make_desc(c, conv_out(h, k, stride, pad), conv_out(wdt, k, stride, pad))))
        return fail(CADNN_EUNSUPPORTED, "cadnn_maxpool2d: a channel plane of 2^30 elements or more");
    return launch_maxpool(x, make_desc(c, h, wdt), y,
                          make_desc(c, conv_out(h, k, stride, pad), conv_out(wdt, k, stride, pad)), n, k, stride,
                          pad, dtype, (hipStream_t)stream);
}

extern "C" cadnn_status cadnn_avgpool2d(const void* x, void* y, int n, int c, int h, int wdt, int k,
                                        int stride, int pad, cadnn_dtype dtype, void* stream) {
    if (!x || !y) return fail(CADNN_EINVAL, "cadnn_avgpool2d: NULL tensor");
    if (n <= 0 || c <= 0 || h <= 0 || wdt <= 0 || k <= 0 || stride <= 0 || pad < 0)
        return fail(CADNN_EINVAL, "cadnn_avgpool2d: bad size");
    if (dtype != CADNN_F32 && dtype != CADNN_F16) return fail(CADNN_EINVAL, "cadnn_avgpool2d: dtype");
    if (conv_out(h, k, stride, pad) <= 0 || conv_out(wdt, k, stride, pad) <= 0)
        return fail(CADNN_EINVAL, "cadnn_avgpool2d: empty output");
    if (desc_too_large(make_desc(c, h, wdt)) || desc_too_large(make_desc(c, conv_out(h, k, stride, pad), conv_out(wdt, k, stride, pad))))
        return fail(CADNN_EUNSUPPORTED, "cadnn_avgpool2d: a channel plane of 2^30 elements or more");
    return launch_avgpool2d(x, make_desc(c, h, wdt), y,
                            make_desc(c, conv_out(h, k, stride, pad), conv_out(wdt, k, stride, pad)), n, k, stride,
                            pad, dtype, (hipStream_t)stream);
}

extern "C" cadnn_status cadnn_global_avgpool(const void* x, void* y, int n, int c, int h, int wdt,
                                             cadnn_dtype dtype, void* stream) {
    if (!x || !y) return fail(CADNN_EINVAL, "cadnn_global_avgpool: NULL tensor");
    if (n <= 0 || c <= 0 || h <= 0 || wdt <= 0) return fail(CADNN_EINVAL, "cadnn_global_avgpool: bad size");
    if (dtype != CADNN_F32 && dtype != CADNN_F16) return fail(CADNN_EINVAL, "cadnn_global_avgpool: dtype");
    if (desc_too_large(make_desc(c, h, wdt))) return fail(CADNN_EUNSUPPORTED, "cadnn_global_avgpool: a channel plane of 2^30 elements or more");
    return launch_avgpool(x, make_desc(c, h, wdt), y, n, dtype, (hipStream_t)stream);
}
