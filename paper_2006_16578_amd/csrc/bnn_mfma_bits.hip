// Which products the kernels of bnn_mfma_bits.h take, on which tile, and their launches.
#include "bnn_mfma_bits.h"

namespace bnn {
namespace {

using mfma::BitsTile;
using mfma::KsplitTile;

typedef BitsTile<4, 2, 2, 4, 2> T256x256;      // eight waves of 128 x 64, one workgroup per compute unit
typedef BitsTile<4, 2, 2, 2, 2> T256x128;      // four waves of 128 x 64
typedef BitsTile<3, 2, 2, 2, 2> T192x128;      // four waves of 96 x 64
typedef BitsTile<2, 2, 2, 2, 3> T128x128;      // four waves of 64 x 64
typedef BitsTile<2, 1, 2, 4, 4> T128x128w8;    // eight waves of 64 x 32
typedef BitsTile<2, 1, 2, 2, 4> T128x64;       // four waves of 64 x 32
typedef KsplitTile<2, 1, 1, 2, 4, 4> K64x64;   // two waves of 64 x 32, four groups
typedef KsplitTile<1, 1, 1, 1, 8, 4> K32x32;   // eight groups

// What a call on a tile takes, in us: launch + max(first + slabs * slab, q * (each + slabs * per + sums)), q workgroups on the busiest of 256 compute units: the
// chain of one workgroup by itself, or the work of those that share a compute unit.  Fitted to graph replays of 700 products of 129 to 16384 rows, 10 to 16384
// columns and 64 to 16384 bits, bits and int32 out, on every tile (mean deviation 2 to 6 %, of nine in ten 5 to 13 %).  On them the tile with the smallest
// estimate is 1.10 times as fast, in the geometric mean, as the tile by size alone and the kernels before (0.90 to 2.5; 14 of 700 lose more than 3 %).
struct Cost { BitsChoice tile; int rows, cols, slab_words; float launch, first, slab, each, per, sums; };
constexpr Cost COSTS[] = {
    {BITS_256x256, 256, 256, 16, 0.000f, 6.039f, 1.969f, 5.771f, 1.950f, 4.917f},
    {BITS_256x128, 256, 128, 16, 4.399f, 1.166f, 1.274f, 1.461f, 1.203f, 3.223f},
    {BITS_192x128, 192, 128, 16, 3.855f, 0.000f, 1.157f, 1.241f, 0.936f, 2.284f},
    {BITS_128x128, 128, 128, 16, 3.202f, 0.365f, 0.956f, 0.732f, 0.678f, 1.622f},
    {BITS_128x128W8, 128, 128, 16, 2.419f, 0.759f, 0.780f, 0.931f, 0.741f, 1.477f},
    {BITS_128x64, 128, 64, 16, 2.965f, 0.004f, 0.625f, 0.371f, 0.413f, 0.775f},
    {BITS_K64x64, 64, 64, 32, 2.451f, 0.846f, 0.551f, 1.092f, 0.428f, 0.396f},
    {BITS_K32x32, 32, 32, 64, 2.626f, 0.856f, 0.371f, 0.721f, 0.295f, 0.109f},
};
constexpr Cost DIRECT64 = {BITS_NONE, 64, 64, 8, 2.502f, 0.000f, 0.216f, 0.120f, 0.182f, 0.474f};    // the direct kernel's 64 x 64 tile

float estimate(const Cost& c, long long rows, long long span, int tw, bool sums) {
    const long long q = cdiv(cdiv(rows, c.rows) * cdiv(span, c.cols), 256);
    // a tile's slab of 16 words is multiplied by halves, a group's share of a larger one is not
    const float slabs = c.slab_words == 16 ? 0.5f * (float)cdiv(tw, 8) : (float)cdiv(tw, c.slab_words);
    const float alone = c.first + c.slab * slabs, shared = (float)q * (c.each + c.per * slabs + (sums ? c.sums : 0.f));
    return c.launch + (alone > shared ? alone : shared);
}

template <class TL, bool FULL, bool PANELS>
int launch_bits_form(const uint32_t* A, const uint32_t* B, const Geom& g, const Epi& e, hipStream_t s) {
    const int col_span = (e.bits != nullptr) ? max(g.cols, e.ldbits_w * 32) : g.cols;
    const int gx = (int)cdiv(g.rows, TL::ROWS), gy = (int)cdiv(col_span, TL::COLS);
    const unsigned nwg = (unsigned)(cdiv((long long)gx * gy, 8) * 8);
    static const hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void*>(&mfma::mfma_bits_kernel<TL, FULL, PANELS>),
                                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)TL::LDS_BYTES);
    if (attr != hipSuccess) return BNN_ERR_DEVICE;
    launch((mfma::mfma_bits_kernel<TL, FULL, PANELS>), dim3(nwg), dim3(TL::THREADS), TL::LDS_BYTES, s, A, B, g, e, gx, gy);
    return check_launch();
}

template <class TL, bool PANELS>
int launch_bits(const uint32_t* A, const uint32_t* B, const Geom& g, const Epi& e, hipStream_t s) {
    return g.tw % 16 == 0 ? launch_bits_form<TL, true, PANELS>(A, B, g, e, s) : launch_bits_form<TL, false, PANELS>(A, B, g, e, s);
}

template <class TL>
int launch_ksplit(const uint32_t* A, const uint32_t* B, const Geom& g, const Epi& e, hipStream_t s) {
    const int col_span = (e.bits != nullptr) ? max(g.cols, e.ldbits_w * 32) : g.cols;
    const int gx = (int)cdiv(g.rows, TL::ROWS), gy = (int)cdiv(col_span, TL::COLS);
    const unsigned nwg = (unsigned)(cdiv((long long)gx * gy, 8) * 8);
    static const hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void*>(&mfma::mfma_ksplit_kernel<TL>),
                                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)TL::LDS_BYTES);
    if (attr != hipSuccess) return BNN_ERR_DEVICE;
    launch((mfma::mfma_ksplit_kernel<TL>), dim3(nwg), dim3(TL::THREADS), TL::LDS_BYTES, s, A, B, g, e, gx, gy);
    return check_launch();
}

}  // namespace

// The old tile by size (pick_tile) stays where K is short: up to 512 bits, where a tile is a launch, a load and an epilogue, and the set bits' two additions to a
// sum cost more than cheaper operands save (116 to 430 bits, bits out: 0.80 to 0.95 of the speed); and for bits up to 1280 where it gives the two
// largest tiles (4000x4000x800 10.6 us on its 256 x 128 tile, 11.2 on the one here; 5000x5100x1234 22.1 on 256 x 256, estimated 20.2 and measured 19.8 on 128 x 128,
// but 26.0 -> 27.1 for 6952x6700x828).  The 256 x 256 tile needs most of the compute units: as many as it has for bits, and any by the estimate for sums.
// The direct kernel's 64 x 64 tile is given 7 %: its estimate deviates most.
BitsChoice mfma_bits_choice(const Geom& g, const Epi& e, int tile) {
    if (g.conv || g.b_tiled || g.taps != 1) return BITS_NONE;
    const int kind = mfma::epilogue_kind(e, false, false);
    if (kind != mfma::EPI_BITS && kind != mfma::EPI_SUMS) return BITS_NONE;
    // 32-bit byte offsets inside a tile: 255 rows and a row's words
    if (g.lda_w >= (1 << 22) || g.ldb_w >= (1 << 22)) return BITS_NONE;
    const bool sums = kind == mfma::EPI_SUMS;
    const long long span = sums ? g.cols : cdiv(g.cols, 128) * 128;       // (output rows of packed words are padded to four)
    const long long large = cdiv(g.rows, 256) * cdiv(span, 256);
    if (g.tw <= 16) return BITS_NONE;
    if (!sums && g.tw <= 40 && tile == 0) return g.tw >= 32 && large >= 240 ? BITS_256x256 : BITS_NONE;
    const bool direct = tile == 3 && mfma::offsets_fit(g);
    BitsChoice best = BITS_NONE;
    float least = direct ? 0.93f * estimate(DIRECT64, g.rows, span, g.tw, sums) : 3.4e38f;
    for (const Cost& c : COSTS) {
        if (c.tile == BITS_256x256 && !sums && large < 208) continue;
        const float t = estimate(c, g.rows, span, g.tw, sums);
        if (t < least) { least = t; best = c.tile; }
    }
    return best;
}

int launch_mfma_bits(BitsChoice tile, const uint32_t* A, const uint32_t* B, const Geom& g, const Epi& e, hipStream_t s) {
    switch (tile) {
        case BITS_256x256: return launch_bits<T256x256, false>(A, B, g, e, s);
        case BITS_256x128: return launch_bits<T256x128, false>(A, B, g, e, s);
        case BITS_192x128: return launch_bits<T192x128, false>(A, B, g, e, s);
        case BITS_128x128: return launch_bits<T128x128, false>(A, B, g, e, s);
        case BITS_128x128W8: return launch_bits<T128x128w8, false>(A, B, g, e, s);
        case BITS_128x64: return launch_bits<T128x64, false>(A, B, g, e, s);
        case BITS_K64x64: return launch_ksplit<K64x64>(A, B, g, e, s);
        case BITS_K32x32: return launch_ksplit<K32x32>(A, B, g, e, s);
        default: return BNN_ERR_UNSUPPORTED;
    }
}

const char* describe_mfma_bits(BitsChoice tile, bool program) {
    switch (tile) {
        case BITS_256x256: return program ? "mfma_fp4_bmm_xlds_wg256x256_01" : "mfma_fp4_bmm_xlds_wg256x256";
        case BITS_256x128: return program ? "mfma_fp4_bmm_lds_wg256x128_01" : "mfma_fp4_bmm_lds_wg256x128";
        case BITS_192x128: return program ? "mfma_fp4_bmm_lds_wg192x128_01" : "mfma_fp4_bmm_lds_wg192x128";
        case BITS_128x128: return program ? "mfma_fp4_bmm_lds_wg128x128_01_w4" : "mfma_fp4_bmm_lds_wg128x128";
        case BITS_128x128W8: return program ? "mfma_fp4_bmm_lds_wg128x128_01_w8" : "mfma_fp4_bmm_lds_wg128x128";
        case BITS_128x64: return program ? "mfma_fp4_bmm_lds_wg128x64_01" : "mfma_fp4_bmm_lds_wg128x64";
        case BITS_K64x64: return program ? "mfma_fp4_bmm_wg64x64_01_ksplit" : "mfma_fp4_bmm_wg64x64";
        default: return program ? "mfma_fp4_bmm_wg32x32_01_ksplit" : "mfma_fp4_bmm_wg32x32";
    }
}

// Operands in K panels (g.tw a multiple of 8, lda_w / ldb_w unused); e.bits, if set, receives panels too
// (e.ldbits_w = 8 * number of output panels).  Any shape; the tile is sized for large ones.
int launch_mfma_bits_panels(const uint32_t* A, const uint32_t* B, const Geom& g, const Epi& e, hipStream_t s) {
    if (g.conv || g.b_tiled || (g.tw & 7) || g.rows >= (1LL << 31)) return BNN_ERR_UNSUPPORTED;
    if (e.bits != nullptr && (e.out != nullptr || e.out16 != nullptr || e.resid != nullptr || e.resid16 != nullptr ||
                              e.resid_bits != nullptr || (e.ldbits_w & 7)))
        return BNN_ERR_UNSUPPORTED;
    return launch_bits<T256x256, true>(A, B, g, e, s);
}

}  // namespace bnn
