// Matrix-core path: dispatch and the BMM instantiations (kernels are in bnn_mfma_kernel.h and
// bnn_mfma_staged.h).
#include <stdio.h>

#include "bnn_mfma_staged.h"

namespace bnn {

namespace {

// The LDS-staged kernel covers every BMM (rows are padded to 128 bits) and the convolutions whose
// pixels are 8 bytes or a multiple of 16 bytes with -1 padding; the smallest tile, exclude
// padding and other channel counts use the direct kernel.
bool staged_ok(const Geom& g, int tile) {
    if (tile == 3) return false;
    if (!g.conv) return true;
    if (tile == 1 && g.tw == 2) return false;    // 512 loader rows of 8-byte pixels: too many registers
    return mfma::conv_stages_through_lds(g);
}

}  // namespace

// Bits only, on the unrolled 3x3 forms of the direct kernel: what the other kernels serve keeps its own row order, and so do excluded
// padding, whose sums may need a correction by pixel, and odd sizes, whose last row or column lies in no window.  Small batches
// gain a launch and a kernel of 3 us; VGG for 32x32 images, batch 8: 49 -> 41 us with three pooling layers stored this way.  Layers of the band kernel too:
// in bands, with a pooling launch, a chain of first layer, convolution and pooling runs at 0.85 to 1.08 of the speed (38 layers, median 0.99).
bool mfma_conv_pools(const Geom& g, const Epi& e) {
    return g.conv && !g.excl && g.k == 3 && (g.tw == 2 || g.tw == 4 || g.tw == 8 || g.tw == 16) && (g.P & 1) == 0 && (g.Q & 1) == 0 && g.A2 == nullptr && mfma::epilogue_kind(e, true, false) == mfma::EPI_BITS &&
           !mfma_conv_patch_takes(g, e) && mfma_conv_xlds_tile(g, e) == 0 && !staged_ok(g, mfma::pick_tile(g, &e)) && mfma::offsets_fit(g);
}

int launch_mfma(const uint32_t* A, const uint32_t* B, const Geom& g, const Epi& e, hipStream_t s) {
    if (mfma_skinny_takes(g)) return launch_mfma_skinny(A, B, g, e, s);
    const int tile = mfma::pick_tile(g, &e);
    if (const BitsChoice bt = mfma_bits_choice(g, e, tile)) return launch_mfma_bits(bt, A, B, g, e, s);
    if (!g.conv) {
        if (!g.b_tiled && staged_ok(g, tile)) {
            switch (tile) {
                case 0: return mfma::launch_staged_tile<mfma::TileBig, 16, false>(A, B, g, e, s);
                case 1: return mfma::launch_staged_tile<mfma::TileTall, 16, false>(A, B, g, e, s);
                default: return mfma::launch_staged_tile<mfma::TileMid, 16, false>(A, B, g, e, s);
            }
        }
        // tw is a multiple of 4 words; a chunk is 8 words, so an odd number of 4-word groups
        // leaves the upper half-wave without data in the last chunk -> guarded variant
        if (!mfma::offsets_fit(g)) {     // leading dimensions beyond the direct kernel's 32-bit offsets
            if (g.b_tiled) return BNN_ERR_UNSUPPORTED;
            return mfma::launch_staged_tile<mfma::TileMid, 16, false>(A, B, g, e, s);
        }
        if (g.tw % 8 == 0) return mfma::launch_shape<4, false, false>(A, B, g, e, s);
        return mfma::launch_shape<4, false, true>(A, B, g, e, s);
    }
    if (mfma_conv_band_takes(g, e)) return launch_mfma_conv_band(A, B, g, e, s);
    if (mfma_conv_patch_takes(g, e)) return launch_mfma_conv_patch(A, B, g, e, s);
    if (const int xt = mfma_conv_xlds_tile(g, e)) return launch_mfma_conv_xlds(xt, A, B, g, e, s);
    // (blocked 16-bit sums are implemented by the band, patch, wave-per-tap and direct kernels)
    if (!e.sums_tiled && staged_ok(g, tile)) return launch_mfma_conv_staged(A, B, g, e, s);
    if (tile == 3 && mfma_conv_taps_takes(g, e, g.pool2 != 0)) return launch_mfma_conv_taps(A, B, g, e, s);
    if (!mfma::offsets_fit(g)) return BNN_ERR_UNSUPPORTED;
    const bool stream = mfma::streams_residual(g, e);
    switch (mfma::conv_load_words(g)) {
        case 4: return stream ? launch_mfma_conv_v4_stream(A, B, g, e, s) : launch_mfma_conv_v4(A, B, g, e, s);
        case 2: return stream ? launch_mfma_conv_v2_stream(A, B, g, e, s) : launch_mfma_conv_v2(A, B, g, e, s);
        default: return stream ? launch_mfma_conv_v1_stream(A, B, g, e, s) : launch_mfma_conv_v1(A, B, g, e, s);
    }
}

const char* describe_mfma(const Geom& g, bool int32_out, int flags) {
    const bool program = (flags & NAME_PROGRAM) != 0;
    if (mfma_skinny_takes(g)) return describe_mfma_skinny(g, program);
    static int32_t some_output;
    static uint32_t some_bits;
    Epi e = {};                                   // the choice only asks which outputs there are, never touches them
    e.out = int32_out ? &some_output : nullptr;
    e.bits = int32_out ? nullptr : &some_bits;
    e.ldbits_w = (g.cols + 31) / 32;
    e.ldc = g.cols;
    static int16_t some_sums;
    if (flags & BNN_CONV_RESIDUAL) e.resid16 = &some_sums;
    if (flags & BNN_CONV_KEEP_SUM) e.out16 = &some_sums;
    if (flags & BNN_CONV_RESIDUAL32) e.resid = &some_output;
    static thread_local char name[64];
    auto with_suffix = [](const char* base, const char* suffix) {
        snprintf(name, sizeof(name), "%s%s", base, suffix);
        return (const char*)name;
    };
    e.sums_tiled = (flags & (BNN_CONV_RESIDUAL | BNN_CONV_KEEP_SUM)) && g.cols % 32 == 0 ? 1 : 0;
    const int tile = mfma::pick_tile(g, &e);
    if (const BitsChoice bt = mfma_bits_choice(g, e, tile)) return describe_mfma_bits(bt, program);
    const bool pools = (flags & BNN_CONV_POOL2) && mfma_conv_pools(g, e);
    if (!pools && mfma_conv_band_takes(g, e)) return "mfma_fp4_conv3x3_band_wg64";
    if (mfma_conv_patch_takes(g, e)) return describe_mfma_conv_patch(g);
    if (const int xt = mfma_conv_xlds_tile(g, e))         // (its streamed form needs whole lines only)
        return with_suffix(describe_mfma_conv_xlds(xt), e.resid != nullptr && (e.ldc & 31) == 0 ? "_stream" : "");
    const char* suffix = pools ? "_pool2" : mfma::streams_residual(g, e) ? "_stream" : "";
    if (tile == 3 && mfma_conv_taps_takes(g, e, pools)) return with_suffix("mfma_fp4_conv_taps_wg32x32", suffix);
    const bool st = !g.b_tiled && !e.sums_tiled && staged_ok(g, tile);
    auto product = [&](const char* base) { return program ? with_suffix(base, "_signs") : base; };
    switch (tile) {
        case 0: return g.conv ? with_suffix(st ? "mfma_fp4_conv_lds_wg256x128" : "mfma_fp4_conv_wg256x128", suffix)
                              : product(st ? "mfma_fp4_bmm_lds_wg256x128" : "mfma_fp4_bmm_wg256x128");
        case 1: return g.conv ? with_suffix(st ? "mfma_fp4_conv_lds_wg512x64" : "mfma_fp4_conv_wg512x64", suffix)
                              : product(st ? "mfma_fp4_bmm_lds_wg512x64" : "mfma_fp4_bmm_wg512x64");
        case 2: return g.conv ? with_suffix(st ? "mfma_fp4_conv_lds_wg128x128" : "mfma_fp4_conv_wg128x128", suffix)
                              : product(st ? "mfma_fp4_bmm_lds_wg128x128" : "mfma_fp4_bmm_wg128x128");
        default: return g.conv ? with_suffix("mfma_fp4_conv_wg64x64", suffix) : product("mfma_fp4_bmm_wg64x64");
    }
}

}  // namespace bnn
