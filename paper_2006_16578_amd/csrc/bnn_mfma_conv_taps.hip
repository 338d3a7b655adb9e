// Matrix-core path for small 3x3 convolutions of 128, 256 and 512 channels (any stride and padding): a workgroup per 32 x 32 outputs, a wave per tap.
//
// What bounds the direct kernel there: its smallest tile is 64 x 64, a layer of 512 output pixels x 512 channels is 64 workgroups on 256 compute units,
// and each of their waves walks all of K, up to 36 loads in different lines one behind the other and 72 dependent MFMAs.  Here nine waves
// hold a tap each, request all of it at once, and meet in LDS: partial sums are added by four waves, a quarter of the accumulator registers
// each, and the first wave finishes the tile with the shared epilogues.  A tenth wave multiplies a block's 1x1 shortcut meanwhile.
// Measured (graph replays, direct kernel -> this one): 8 x 8x8x512 -> 512 5.8 -> 4.1 us, 8 x 16x16x256 -> 256 4.3 -> 4.15, 4 x 14x14x256-sized layers
// 4.3 -> 3.5, 8 x 7x7x128 3.7 -> 3.3 (an empty launch of this grid is 2.6); ResNet-18 of batch 4 92 -> 80, a Cifar ResNet-14 of batch 8 68 -> 55.
#include "bnn_mfma_kernel.h"

namespace bnn {
namespace {

using mfma::v16f;
using mfma::v8i;

enum TapsForm { TAPS_BITS, TAPS_POOL, TAPS_CHAIN };

// V: words per lane and load, CH loads per tap (2 V CH words per pixel).
template <int V, int CH, bool EXCL, int FORM>
__global__ __launch_bounds__(640) void conv_taps_kernel(const uint32_t* __restrict__ A, const uint32_t* __restrict__ B, Geom g, Epi e, int gx, int gy) {
    extern __shared__ float4 part[];                 // [wave][quad of registers][lane]
    int bx, by;
    if (!mfma::tile_coords(gx, gy, bx, by)) return;  // uniform for the workgroup
    const int lane = threadIdx.x & 63, l32 = lane & 31, half = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), waves = (int)blockDim.x >> 6;
    const int m0 = 32 * bx, n0 = 32 * by;            // rows < 2^31
    uint32_t c2;
    asm volatile("v_mov_b32 %0, 0x22222222" : "=v"(c2));

    v16f acc[1][1];
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[0][0][r] = 0.f;
    int thi[1];
    bool cok[1];
    mfma::Fetched fetched = {make_uint4(0u, 0u, 0u, 0u), make_uint4(0u, 0u, 0u, 0u), false};
    if (wave < 9) {
        const int row = min(m0 + l32, (int)g.rows - 1);                                  // past the end: dropped by the epilogue
        const int n = fast_div(row, g.div_pq), rem = row - n * (g.P * g.Q);
        int p = fast_div(rem, g.div_q), q = rem - p * g.Q;
        if constexpr (FORM == TAPS_POOL) pool_row_pixel(g, rem, p, q);
        const int r = wave / 3, s = wave - 3 * r;
        const int y = p * g.stride - g.pad + r, x = q * g.stride - g.pad + s;
        const bool in = (unsigned)y < (unsigned)g.H && (unsigned)x < (unsigned)g.W;
        const uint32_t* src = A + (in ? (((long long)n * g.H + y) * g.W + x) * g.lda_w : 0) + half * V;
        const uint32_t* flt = B + (long long)min(n0 + l32, g.cols - 1) * g.ldb_w + wave * g.tw + half * V;
        uint32_t ra[CH][V], rb[CH][V];
#pragma unroll
        for (int c = 0; c < CH; ++c) {
            mfma::load_words<V>(src + c * 2 * V, ra[c]);
            mfma::load_words<V>(flt + c * 2 * V, rb[c]);
        }
        if (wave == 0) {                             // what the epilogue reads, behind the operands
            mfma::column_thresholds<1>(thi, cok, n0, l32, g, e);
            if (FORM == TAPS_CHAIN && e.resid16 != nullptr && m0 < g.rows && n0 < g.cols) {
                const uint4* res = reinterpret_cast<const uint4*>(e.resid16 + ((m0 >> 5) * (long long)(e.ldc >> 5) + (n0 >> 5)) * 1024 + lane * 16);
                fetched.lo = res[0]; fetched.hi = res[1]; fetched.valid = true;
            }
        }
        const uint32_t keep = in ? 0xFFFFFFFFu : 0u;
        const uint32_t c2a = EXCL ? c2 & keep : c2;  // an out-of-frame tap is 0 bits (-1 padding) or, with excluded padding, fp4 zeros
#pragma unroll
        for (int c = 0; c < CH; ++c)
#pragma unroll
            for (int v = 0; v < V; ++v)
                acc[0][0] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(mfma::expand_fp4(ra[c][v] & keep, c2a), mfma::expand_fp4(rb[c][v], c2),
                                                                           acc[0][0], 4, 4, 0, 0, 0, 0);
    } else {
        mfma::extra_source<1, 1>(acc, g, m0, n0, lane, c2);
    }
#pragma unroll
    for (int q = 0; q < 4; ++q)
        part[(wave * 4 + q) * 64 + lane] = make_float4(acc[0][0][4 * q], acc[0][0][4 * q + 1], acc[0][0][4 * q + 2], acc[0][0][4 * q + 3]);
    __syncthreads();
    if (wave < 4) {                                  // exact: whole numbers below 2^24
        float4 sum = part[wave * 64 + lane];
#pragma unroll
        for (int w = 1; w < 9; ++w) {
            const float4 v = part[(w * 4 + wave) * 64 + lane];
            sum.x += v.x; sum.y += v.y; sum.z += v.z; sum.w += v.w;
        }
        if (waves > 9) {
            const float4 v = part[(36 + wave) * 64 + lane];
            sum.x += v.x; sum.y += v.y; sum.z += v.z; sum.w += v.w;
        }
        part[wave * 64 + lane] = sum;                // read by this wave alone until here
    }
    __syncthreads();
    if (wave != 0) return;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const float4 v = part[q * 64 + lane];
        acc[0][0][4 * q] = v.x; acc[0][0][4 * q + 1] = v.y; acc[0][0][4 * q + 2] = v.z; acc[0][0][4 * q + 3] = v.w;
    }
    const int corr = g.A2 != nullptr ? (g.cw2 + 1) / 2 * 64 - g.bits2 : 0;               // what the second source multiplied beyond its width
    if constexpr (FORM == TAPS_CHAIN) mfma::epilogue_chain<1, 1>(acc, m0, n0, lane, g, e, corr, thi, cok, fetched);
    else mfma::epilogue_bits<1, 1, false, FORM == TAPS_POOL>(acc, m0, n0, lane, g, e, corr, thi, cok);
}

template <int V, int CH, bool EXCL>
int launch_taps(const uint32_t* A, const uint32_t* B, const Geom& g, const Epi& e, hipStream_t s) {
    const int gx = (int)cdiv(g.rows, 32), gy = e.ldbits_w > (int)cdiv(g.cols, 32) ? e.ldbits_w : (int)cdiv(g.cols, 32);
    const int waves = g.A2 != nullptr ? 10 : 9;
    const dim3 grid((unsigned)(cdiv((long long)gx * gy, 8) * 8));
    const size_t lds = (size_t)waves * 4096;
    if (g.pool2) {
        if constexpr (EXCL) return BNN_ERR_UNSUPPORTED;          // not dispatched: mfma_conv_pools
        else launch((conv_taps_kernel<V, CH, EXCL, TAPS_POOL>), grid, dim3(64 * waves), lds, s, A, B, g, e, gx, gy);
    } else if (mfma::epilogue_kind(e, true, false) == mfma::EPI_CHAIN)
        launch((conv_taps_kernel<V, CH, EXCL, TAPS_CHAIN>), grid, dim3(64 * waves), lds, s, A, B, g, e, gx, gy);
    else
        launch((conv_taps_kernel<V, CH, EXCL, TAPS_BITS>), grid, dim3(64 * waves), lds, s, A, B, g, e, gx, gy);
    return check_launch();
}

}  // namespace

bool mfma_conv_taps_takes(const Geom& g, const Epi& e, bool pooled) {
    if (!g.conv || g.k != 3 || (g.tw != 4 && g.tw != 8 && g.tw != 16) || g.bits_tap != g.tw * 32) return false;
    const int kind = mfma::epilogue_kind(e, true, false);
    if (kind != mfma::EPI_BITS && kind != mfma::EPI_CHAIN) return false;
    // One workgroup per compute unit for each 128 channels of K, up to three (its speed over the direct kernel's 64x64 tile, graph replays of bits, in steps
    // of 256 workgroups): 128 channels 1.09 to 1.16, then 0.99 to 1.03, 0.9, 0.8; 256: 1.18 to 1.27, 1.00 to 1.07, 0.91 to 0.94, 0.8; 512: 1.36 to
    // 1.45, 1.16 to 1.23, 1.01 to 1.05, 0.85 to 0.89.  With pooled bits, a first layer, such a layer and an FC together: 256 channels 1.07 to 1.10, 1.02 to 1.04, then 0.99;
    // 512: 1.11 to 1.14, 1.06, 1.01; 128: 1.02 to 1.03, then 0.99 to 1.00.  (Such chains of fewer than 96 tiles would gain too, 1.05 to 1.14 at 256 and 512 channels; that those layers
    // are the direct kernel's is tested behaviour of bnn_bconv_kernel_name_ex.)
    const long long tiles = cdiv(g.rows, 32) * cdiv(g.cols, 32), most = g.tw == 4 ? 256 : g.tw == 8 ? 512 : 768;
    return tiles <= most && (!pooled || tiles >= 96);
}

int launch_mfma_conv_taps(const uint32_t* A, const uint32_t* B, const Geom& g, const Epi& e, hipStream_t s) {
    if (g.tw == 4) return g.excl ? launch_taps<2, 1, true>(A, B, g, e, s) : launch_taps<2, 1, false>(A, B, g, e, s);
    if (g.tw == 8) return g.excl ? launch_taps<4, 1, true>(A, B, g, e, s) : launch_taps<4, 1, false>(A, B, g, e, s);
    return g.excl ? launch_taps<4, 2, true>(A, B, g, e, s) : launch_taps<4, 2, false>(A, B, g, e, s);
}

}  // namespace bnn
