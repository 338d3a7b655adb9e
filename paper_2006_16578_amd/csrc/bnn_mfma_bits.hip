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

// What a call on a tile takes, in us: launch + max(first + slabs * slab, q * (each + slabs * per)), q workgroups on the busiest of 256 compute units: the chain of one workgroup by itself, or the work of
// those that share a compute unit.  Sums have their own constants, and what their megabytes wait for memory (near: each; far: each beyond 256, which the last cache does not
// take), which overlaps in part with the products: the root of the squares.  Fitted to graph replays of 1790 products of 129 to 16384 rows, 10 to
// 16384 columns (120 of up to 1.5 million rows and 70 of up to 60000 columns) and 513 to 16384 bits, on every tile, where a tile took at most 1.5 times the best one's time: mean deviation
// 2 to 5 %, of nine in ten 3 to 11 %.
struct Cost { BitsChoice tile; int rows, cols, slab_words; float launch, first, slab, each, per, near, far; };
constexpr Cost COSTS[2][8] = {
    {// bits
     {BITS_256x256, 256, 256, 16, 0.35f, 5.87f, 0.85f, 5.00f, 2.19f, 0.00f, 0.00f},
     {BITS_256x128, 256, 128, 16, 2.78f, 2.52f, 1.29f, 1.92f, 1.16f, 0.00f, 0.00f},
     {BITS_192x128, 192, 128, 16, 2.42f, 2.02f, 1.06f, 1.50f, 0.91f, 0.00f, 0.00f},
     {BITS_128x128, 128, 128, 16, 2.77f, 0.83f, 0.88f, 0.68f, 0.67f, 0.00f, 0.00f},
     {BITS_128x128W8, 128, 128, 16, 1.91f, 1.12f, 0.79f, 0.89f, 0.74f, 0.00f, 0.00f},
     {BITS_128x64, 128, 64, 16, 2.62f, 0.18f, 0.60f, 0.34f, 0.42f, 0.00f, 0.00f},
     {BITS_K64x64, 64, 64, 32, 2.09f, 1.19f, 0.53f, 1.07f, 0.46f, 0.00f, 0.00f},
     {BITS_K32x32, 32, 32, 64, 2.54f, 0.72f, 0.36f, 0.68f, 0.33f, 0.00f, 0.00f},
    },
    {// sums
     {BITS_256x256, 256, 256, 16, 1.19f, 1.56f, 0.87f, 7.10f, 2.42f, 0.21f, 0.15f},
     {BITS_256x128, 256, 128, 16, 2.68f, 6.67f, 1.30f, 4.11f, 1.18f, 0.13f, 0.17f},
     {BITS_192x128, 192, 128, 16, 3.49f, 3.96f, 1.09f, 2.67f, 0.93f, 0.13f, 0.16f},
     {BITS_128x128, 128, 128, 16, 4.51f, 0.85f, 0.90f, 1.03f, 0.69f, 0.13f, 0.22f},
     {BITS_128x128W8, 128, 128, 16, 3.56f, 0.24f, 0.44f, 1.29f, 0.79f, 0.12f, 0.08f},
     {BITS_128x64, 128, 64, 16, 3.62f, 0.34f, 0.62f, 0.68f, 0.44f, 0.10f, 0.18f},
     {BITS_K64x64, 64, 64, 32, 2.56f, 0.97f, 0.55f, 1.19f, 0.46f, 0.30f, 0.10f},
     {BITS_K32x32, 32, 32, 64, 2.75f, 0.80f, 0.37f, 0.76f, 0.33f, 0.30f, 0.20f},
    }};
// The kernels that multiply signs, by pick_tile's tile: three through LDS, and the direct one; and that of bnn_mfma_signs.hip, for bits.
constexpr Cost SIGNS[2][4] = {
    {// bits
     {BITS_NONE, 256, 128, 16, 2.73f, 0.36f, 0.62f, 1.30f, 1.36f, 0.00f, 0.00f},
     {BITS_NONE, 512, 64, 16, 3.10f, 0.26f, 2.34f, 1.02f, 1.67f, 0.00f, 0.00f},
     {BITS_NONE, 128, 128, 16, 3.13f, 0.17f, 0.63f, 0.18f, 0.77f, 0.00f, 0.00f},
     {BITS_NONE, 64, 64, 16, 2.20f, 0.04f, 0.44f, 0.14f, 0.35f, 0.00f, 0.00f},
    },
    {// sums
     {BITS_NONE, 256, 128, 16, 3.36f, 6.43f, 2.64f, 3.78f, 1.39f, 0.07f, 0.17f},
     {BITS_NONE, 512, 64, 16, 0.00f, 12.36f, 3.32f, 0.50f, 2.83f, 0.30f, 0.40f},
     {BITS_NONE, 128, 128, 16, 3.67f, 3.15f, 0.28f, 0.96f, 0.78f, 0.17f, 0.20f},
     {BITS_NONE, 64, 64, 16, 2.84f, 0.16f, 0.40f, 0.21f, 0.36f, 0.15f, 0.01f},
    }};
constexpr Cost SIGNS256 = {BITS_SIGNS256x256, 256, 256, 16, 0.11f, 4.35f, 2.60f, 3.47f, 2.47f, 0.00f, 0.00f};

float estimate(const Cost& c, long long rows, long long span, int tw, float megabytes) {
    const long long q = cdiv(cdiv(rows, c.rows) * cdiv(span, c.cols), 256);
    // a tile's slab of 16 words is multiplied by halves, a group's share of a larger one is not; without masks (whole slabs) a tile takes 0.95
    const bool halves = c.slab_words == 16;
    const float slabs = halves ? 0.5f * (float)cdiv(tw, 8) : (float)cdiv(tw, c.slab_words);
    const float alone = c.first + c.slab * slabs, shared = (float)q * (c.each + c.per * slabs), products = alone > shared ? alone : shared;
    const bool unmasked = halves && c.tile != BITS_NONE && c.tile != BITS_SIGNS256x256 && tw % 16 == 0;
    return c.launch + hypotf(unmasked ? 0.95f * products : products, c.near * megabytes + (megabytes > 256.f ? c.far * (megabytes - 256.f) : 0.f));
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

// The kernels for signs keep K up to 512 bits, where a tile is a launch, a load and an epilogue, and counting the set bits costs more than cheaper operands save
// (116 to 430 bits, bits out: 0.80 to 0.95 of the speed); and for bits K up to 1280 where pick_tile gives its largest tile: with 240 tiles of 256 x 256 or more and K from
// 993 on the kernel of bnn_mfma_signs.hip (256 x 256 on {0, 1}: 0.88 to 0.96 of its speed), else that tile (4000x4000x800 10.4 us, here 10.9).  Everything else goes to the
// smallest estimate, theirs among them at 0.97 (the direct kernel's deviates most; bnn_mfma_signs.hip up to 2048 bits).  The 256 x 256 tile for bits needs most of the compute units.
// Of 920 other products (860 of up to 16384 rows and columns, 60 of up to 1.5 million rows) three are slower than on the kernels before those for {0, 1}, by more than 3 %: 0.94 to 0.95;
// the mean is 1.11 to 1.20 by the range.
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
    if (!sums && g.tw <= 40 && tile == 0) return g.tw >= 32 && large >= 240 ? BITS_SIGNS256x256 : BITS_NONE;
    const float megabytes = sums ? 4e-6f * (float)g.rows * (float)g.cols : 0.f;
    BitsChoice best = BITS_NONE;
    float least = tile != 3 || mfma::offsets_fit(g) ? 0.97f * estimate(SIGNS[sums][tile], g.rows, span, g.tw, megabytes) : 3.4e38f;
    if (!sums && tile == 0 && g.tw <= 64 && large >= 240) {
        const float t = 0.97f * estimate(SIGNS256, g.rows, span, g.tw, 0.f);
        if (t < least) { least = t; best = BITS_SIGNS256x256; }
    }
    for (const Cost& c : COSTS[sums]) {
        if (c.tile == BITS_256x256 && !sums && large < 208) continue;
        const float t = estimate(c, g.rows, span, g.tw, megabytes);
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
        case BITS_SIGNS256x256: return launch_mfma_signs(A, B, g, e, s);
        default: return BNN_ERR_UNSUPPORTED;
    }
}

const char* describe_mfma_bits(BitsChoice tile, bool program) {
    switch (tile) {
        case BITS_256x256: return program ? "mfma_fp4_bmm_xlds_wg256x256_01" : "mfma_fp4_bmm_xlds_wg256x256";
        case BITS_SIGNS256x256: return program ? "mfma_fp4_bmm_xlds_wg256x256_signs" : "mfma_fp4_bmm_xlds_wg256x256";
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
// (e.ldbits_w = 8 * number of output panels).  Any shape; the tile is sized for large ones.  On {0, 1} where tiles fill the chip and K is long enough for its cheaper
// K-steps, else as products of signs.  Bits / sums, signs -> {0, 1}, us: 4096 x 4096, K = 1024 8.8 -> 10.0 / 16.4 -> 18.1, 4096 23.1 -> 23.2 / 30.7 -> 31.2, 8192 42.7 -> 41.4 / 50.7 ->
// 48.8; 20000 x 20000 sums, K = 2048 458 -> 481, 4096 705 -> 715; 2048 x 2048 x 16384 68 -> 72 / 71 -> 75.  (Sums of 16384 columns are the exception, 0.93 to 0.97 of the time from K = 1024 on.)
int launch_mfma_bits_panels(const uint32_t* A, const uint32_t* B, const Geom& g, const Epi& e, hipStream_t s) {
    if (g.conv || g.b_tiled || (g.tw & 7) || g.rows >= (1LL << 31)) return BNN_ERR_UNSUPPORTED;
    if (e.bits != nullptr && (e.out != nullptr || e.out16 != nullptr || e.resid != nullptr || e.resid16 != nullptr ||
                              e.resid_bits != nullptr || (e.ldbits_w & 7)))
        return BNN_ERR_UNSUPPORTED;
    if (cdiv(g.rows, 256) * cdiv(g.cols, 256) < 208 || g.tw <= 128) return launch_mfma_signs_panels(A, B, g, e, s);
    return launch_bits<T256x256, true>(A, B, g, e, s);
}

}  // namespace bnn
