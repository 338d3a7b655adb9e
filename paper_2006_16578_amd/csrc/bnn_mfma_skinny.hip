// Matrix-core path for skinny matrix products (at most 128 rows of A: fully-connected layers at small batch).
//
// Such a product is bound by streaming the weights: M = 8, K = N = 4096 is 2 MB of B for 0.13 G bit-products.
// The tiled kernels give it one workgroup per 64 x 64 outputs, each walking all of K serially -- 64 workgroups on
// 256 compute units, a handful of loads in flight each.  Here a workgroup owns 32 output columns and ALL rows, and
// its waves (eight for up to 32 rows, else four) split K between them (the occupancy argument of Sec. 5.2, Design-1, turned around: with few rows
// the parallelism has to come from K and N).  Every wave requests all of its share of B and A up front (four
// 256-bit chunks in flight per lane), multiplies, and leaves its partial 32 x 32 sums in LDS; after one barrier
// wave i adds the partials of row tile i and runs the ordinary epilogue (threshold -> packed bits, or int32).
// N / 32 workgroups, each with its whole 16 KB of weights in flight at once: the kernel for more than 4096 columns and more than 16 rows.  The rest runs 16 columns to a
// workgroup (mfma_skinny16_kernel, below).
#include "bnn_mfma_kernel.h"

namespace bnn {
namespace {

using mfma::v16f;
using mfma::v8i;

constexpr int DEPTH = 4;      // chunks (256 bits of K per row) a wave keeps in flight

// WAVES: 8 for a single row tile (the partial sums of 8 waves are 32 KB of LDS), 4 otherwise
template <int MT, int WAVES>
__global__ __launch_bounds__(64 * WAVES) void mfma_skinny_kernel(const uint32_t* __restrict__ A, const uint32_t* __restrict__ B,
                                                                 Geom g, Epi e) {
    __shared__ float part[WAVES][MT][16][64];
    const int lane = threadIdx.x & 63, l32 = lane & 31, half = lane >> 5;
    const int wave = threadIdx.x >> 6;
    const int n0 = (int)blockIdx.x * 32;

    uint32_t c2;
    asm volatile("v_mov_b32 %0, 0x22222222" : "=v"(c2));

    const uint32_t* ap[MT];
#pragma unroll
    for (int i = 0; i < MT; ++i) ap[i] = A + (long long)min((long long)(32 * i + l32), g.rows - 1) * g.lda_w + half * 4;
    const uint32_t* bp = B + (long long)min(n0 + l32, g.cols - 1) * g.ldb_w + half * 4;

    v16f acc[MT];
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[i][r] = 0.f;

    // chunk c covers words 8c .. 8c+7 of a row (lower half-wave the first four, upper the last four); wave w
    // takes chunks w, w + 4, ...  tw is a multiple of 4, so only the upper half of the last chunk can lie past
    // the row's end: it is read from the row's start instead and masked to zero bits when multiplied.
    const int T = (g.tw + 7) / 8;
    const int mine = (T - wave + WAVES - 1) / WAVES;
    uint4 ra[DEPTH][MT], rb[DEPTH];
    uint32_t keep[DEPTH];
    auto request = [&](int buf, int t) {
        if (t < mine) {
            const int wo = (wave + WAVES * t) * 8;
            const bool ok = wo + half * 4 < g.tw;
            const int off = ok ? wo : -half * 4;
            rb[buf] = *reinterpret_cast<const uint4*>(bp + off);
#pragma unroll
            for (int i = 0; i < MT; ++i) ra[buf][i] = *reinterpret_cast<const uint4*>(ap[i] + off);
            keep[buf] = ok ? 0xFFFFFFFFu : 0u;
        }
    };
    auto multiply = [&](int buf) {
        const uint32_t km = keep[buf];
        const uint32_t bw[4] = {rb[buf].x & km, rb[buf].y & km, rb[buf].z & km, rb[buf].w & km};
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const v8i eb = mfma::expand_fp4(bw[v], c2);
#pragma unroll
            for (int i = 0; i < MT; ++i) {
                const uint4 a4 = ra[buf][i];
                const uint32_t aw = (v == 0 ? a4.x : v == 1 ? a4.y : v == 2 ? a4.z : a4.w) & km;
                acc[i] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(mfma::expand_fp4(aw, c2), eb, acc[i], 4, 4, 0, 0, 0, 0);
            }
        }
    };
#pragma unroll
    for (int d = 0; d < DEPTH; ++d) request(d, d);
    for (int t = 0; t < mine; t += DEPTH) {
#pragma unroll
        for (int d = 0; d < DEPTH; ++d) {
            if (t + d < mine) multiply(d);
            request(d, t + d + DEPTH);
        }
    }

#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int r = 0; r < 16; ++r) part[wave][i][r][lane] = acc[i][r];
    __syncthreads();
    if (wave < MT) {                      // wave i finishes row tile i
        v16f sum[1][1];
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            float v = 0.f;                // exact: every partial is an integer below 2^24 in magnitude
#pragma unroll
            for (int w = 0; w < WAVES; ++w) v += part[w][wave][r][lane];
            sum[0][0][r] = v;
        }
        // every chunk multiplied 256 bit positions per row; those past K are 0 bits in both operands (+1 each)
        mfma::epilogue<1, 1, false, false>(sum, 32LL * wave, n0, lane, g, e, T * 256 - g.bits_tap, 0);
    }
}

// 16 columns to a workgroup (v_mfma_f32_16x16x128_f8f6f4, the weights as row operand), twice as many workgroups, and a load takes 64 neighbouring bytes of 16 rows
// instead of 32 of 32 (the address side works line by line: of the 4.8 us of 8 x 1024 x 8192 two were its).  A lane ends up with four channels of one row of A.
// Measured (graph replays of bits, 32 columns -> this one): 8 x 1024 x 8192 4.84 -> 3.85 us, 8 x 1024 x 1024 3.34 -> 2.93, 8 x 4096 x 4096 3.78 -> 2.85, 8 x 4096 x 25088
// 7.86 -> 4.97, 16 x 16384 x 16384 12.0 -> 10.4 (11.0 on the kernel for 32 rows), 16 x 16384 x 1024 3.08 (3.76); 32 x 4096 x 4096 3.96 -> 3.55, 32 x 1024 x 8192 5.04 -> 4.18; 64 x 4096 x 4096 4.87 -> 4.15, 64 x 1000 x 8192 (int32) 6.55 -> 5.45;
// 128 x 4096 x 4096 6.87 -> 5.41, 128 x 10 x 4096 (int32) 6.49 -> 4.57, 128 x 4096 x 16384 13.7 -> 13.4.
typedef float v4f __attribute__((ext_vector_type(4)));
constexpr int WAVES16 = 8;

// What the kernel needs of a call, and no more: a launch takes 2.1 us of host time with 16 bytes of arguments, 2.9 with the 384 of Geom and Epi.
struct Skinny {
    const int32_t* thr;
    uint32_t* bits;
    int32_t* out;
    int rows, cols, tw, lda, ldb, ldc, ldbits, K, out_f32;
};

// RT row tiles of 16; part: RT * WAVES16 * 64
template <int RT>
__device__ __forceinline__ void skinny16(const uint32_t* __restrict__ A, const uint32_t* __restrict__ B, const Skinny& g, float4* part) {
    const int lane = threadIdx.x & 63, l16 = lane & 15, grp = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int n0 = (int)blockIdx.x * 16;

    uint32_t c2;
    asm volatile("v_mov_b32 %0, 0x22222222" : "=v"(c2));
    const uint32_t* ap[RT];
#pragma unroll
    for (int i = 0; i < RT; ++i) ap[i] = A + (long long)min(16 * i + l16, g.rows - 1) * g.lda;
    const uint32_t* bp = B + (long long)min(n0 + l16, g.cols - 1) * g.ldb;

    // chunk c: words 16 c + 4 grp .. + 3 of a row; tw is a multiple of 4, groups past the row's end are zero bits
    const int T = (g.tw + 15) / 16;
    const int mine = (T - wave + WAVES16 - 1) / WAVES16;
    uint4 ra[DEPTH][RT], rb[DEPTH];
    uint32_t keep[DEPTH];
    auto request = [&](int buf, int t) {
        if (t < mine) {
            const int wo = (wave + WAVES16 * t) * 16 + 4 * grp;
            const bool ok = wo < g.tw;
            rb[buf] = *reinterpret_cast<const uint4*>(bp + (ok ? wo : 0));
#pragma unroll
            for (int i = 0; i < RT; ++i) ra[buf][i] = *reinterpret_cast<const uint4*>(ap[i] + (ok ? wo : 0));
            keep[buf] = ok ? 0xFFFFFFFFu : 0u;
        }
    };
    v4f acc[RT];
#pragma unroll
    for (int i = 0; i < RT; ++i) acc[i] = v4f{0.f, 0.f, 0.f, 0.f};
    auto multiply = [&](int buf) {
        const uint32_t km = keep[buf];
        const uint32_t bw[4] = {rb[buf].x & km, rb[buf].y & km, rb[buf].z & km, rb[buf].w & km};
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const v8i eb = mfma::expand_fp4(bw[v], c2);
#pragma unroll
            for (int i = 0; i < RT; ++i) {
                const uint4& a4 = ra[buf][i];
                const uint32_t aw = (v == 0 ? a4.x : v == 1 ? a4.y : v == 2 ? a4.z : a4.w) & km;
                acc[i] = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(eb, mfma::expand_fp4(aw, c2), acc[i], 4, 4, 0, 0, 0, 0);
            }
        }
    };
#pragma unroll
    for (int d = 0; d < DEPTH; ++d) request(d, d);
    int thr[4] = {0, 0, 0, 0};                          // behind the operands, ahead of the barrier
    if (g.bits != nullptr)
#pragma unroll
        for (int r = 0; r < 4; ++r) thr[r] = g.thr[min(n0 + 4 * grp + r, g.cols - 1)];
    for (int t = 0; t < mine; t += DEPTH) {
#pragma unroll
        for (int d = 0; d < DEPTH; ++d) {
            if (t + d < mine) multiply(d);
            request(d, t + d + DEPTH);
        }
    }
#pragma unroll
    for (int i = 0; i < RT; ++i) part[(i * WAVES16 + wave) * 64 + lane] = make_float4(acc[i][0], acc[i][1], acc[i][2], acc[i][3]);
    __syncthreads();
    const int row = 16 * wave + l16;                    // wave i finishes row tile i
    if (wave >= RT || 16 * wave >= g.rows) return;
    float4 sum = part[wave * WAVES16 * 64 + lane];                   // exact: whole numbers below 2^24
#pragma unroll
    for (int w = 1; w < WAVES16; ++w) {
        const float4 v = part[(wave * WAVES16 + w) * 64 + lane];
        sum.x += v.x; sum.y += v.y; sum.z += v.z; sum.w += v.w;
    }
    const int corr = T * 512 - g.K;                     // positions past K: 0 bits in both operands (+1 each)
    const int v[4] = {(int)sum.x - corr, (int)sum.y - corr, (int)sum.z - corr, (int)sum.w - corr};
    const int ch = n0 + 4 * grp;
    if (g.out != nullptr && row < g.rows)
#pragma unroll
        for (int r = 0; r < 4; ++r)
            if (ch + r < g.cols) g.out[(long long)row * g.ldc + ch + r] = g.out_f32 ? __float_as_int((float)v[r]) : v[r];
    if (g.bits != nullptr) {                            // uniform: the four groups of a row meet in a half-word
        uint32_t b = 0u;
#pragma unroll
        for (int r = 0; r < 4; ++r) b |= (ch + r < g.cols && v[r] >= thr[r]) ? 1u << (4 * grp + r) : 0u;
        b |= (uint32_t)__shfl_xor((int)b, 16);
        b |= (uint32_t)__shfl_xor((int)b, 32);
        if (grp == 0 && row < g.rows && (int)blockIdx.x < 2 * g.ldbits)
            reinterpret_cast<uint16_t*>(g.bits)[2LL * row * g.ldbits + blockIdx.x] = (uint16_t)b;
    }
}

// At most 16 * RT rows.
template <int RT>
__global__ __launch_bounds__(64 * WAVES16) void mfma_skinny16_kernel(const uint32_t* __restrict__ A, const uint32_t* __restrict__ B, Skinny g) {
    __shared__ float4 part[RT * WAVES16 * 64];
    skinny16<RT>(A, B, g, part);
}

template <int RT>
int launch_skinny16(const uint32_t* A, const uint32_t* B, const Geom& g, const Epi& e, int col_span, hipStream_t s) {
    const Skinny a = {e.thr, e.bits, e.out, (int)g.rows, g.cols, g.tw, g.lda_w, g.ldb_w, e.ldc, e.ldbits_w, g.bits_tap, e.out_f32};
    launch(mfma_skinny16_kernel<RT>, dim3((unsigned)cdiv(col_span, 16)), dim3(64 * WAVES16), 0, s, A, B, a);
    return check_launch();
}

// 16 columns to a workgroup: with up to 16 rows always, beyond while there is a workgroup for each compute unit at most.  Past that every further one reads all rows of A
// again: 32 rows 5000 x 4096 4.05 -> 4.29, 5000 x 16384 7.3 -> 8.7 (but 10000 x 16384 13.4 -> 11.8), 64 rows 5000 x 4096 5.05 -> 6.23, 128 rows 6.95 -> 9.06.
bool columns16(const Geom& g, int col_span) { return g.rows <= 16 || cdiv(col_span, 16) <= 256; }

}  // namespace

bool mfma_skinny_takes(const Geom& g) { return !g.conv && !g.b_tiled && g.rows <= 128; }

// The names without the program keep the classes that reports know: from 4096 columns on there is none for 16 rows.
const char* describe_mfma_skinny(const Geom& g, bool program) {
    if (g.rows <= 16) return program ? "mfma_fp4_bmm_skinny_m16_c16" : g.cols < 4096 ? "mfma_fp4_bmm_skinny_m16" : "mfma_fp4_bmm_skinny_m32";
    const bool c16 = program && columns16(g, (int)cdiv(g.cols, 128) * 128), c32 = program && !c16;       // (output rows of packed words are padded to four)
    if (g.rows <= 32) return c16 ? "mfma_fp4_bmm_skinny_m32_c16" : c32 ? "mfma_fp4_bmm_skinny_m32_c32" : "mfma_fp4_bmm_skinny_m32";
    if (g.rows <= 64) return c16 ? "mfma_fp4_bmm_skinny_m64_c16" : c32 ? "mfma_fp4_bmm_skinny_m64_c32" : "mfma_fp4_bmm_skinny_m64";
    return c16 ? "mfma_fp4_bmm_skinny_m128_c16" : c32 ? "mfma_fp4_bmm_skinny_m128_c32" : "mfma_fp4_bmm_skinny_m128";
}

int launch_mfma_skinny(const uint32_t* A, const uint32_t* B, const Geom& g, const Epi& e, hipStream_t s) {
    const int col_span = (e.bits != nullptr) ? max(g.cols, e.ldbits_w * 32) : g.cols;
    if (columns16(g, col_span) && e.resid == nullptr && e.out16 == nullptr) {
        if (g.rows <= 16) return launch_skinny16<1>(A, B, g, e, col_span, s);
        if (g.rows <= 32) return launch_skinny16<2>(A, B, g, e, col_span, s);
        return g.rows <= 64 ? launch_skinny16<4>(A, B, g, e, col_span, s) : launch_skinny16<8>(A, B, g, e, col_span, s);
    }
    const dim3 grid((unsigned)cdiv(col_span, 32));
    if (g.rows <= 32) launch((mfma_skinny_kernel<1, 8>), grid, dim3(64 * 8), 0, s, A, B, g, e);
    else if (g.rows <= 64) launch((mfma_skinny_kernel<2, 4>), grid, dim3(64 * 4), 0, s, A, B, g, e);
    else launch((mfma_skinny_kernel<4, 4>), grid, dim3(64 * 4), 0, s, A, B, g, e);
    return check_launch();
}

}  // namespace bnn
