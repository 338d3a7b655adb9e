// First layer with binarized weights for large strided windows (11x11 stride 4, 7x7 stride 2 and 4) of 3-channel images: a rectangle of
// output pixels and up to 128 channels per wave, input patch in the wave's own LDS, weights as sign bits in registers.
//
// Same arithmetic as the kernels of bnn_bwn.hip: an fp32 value is the exact sum of three bf16 terms, a +1/-1 weight is exact in bf16,
// the products are accumulated in fp32 by v_mfma_f32_32x32x16_bf16 (smallest terms first) and compared with the fp32 threshold.
//
// What bounded these layers before was everything beside the matrix pipe.  Expanded weights of 64 channels (56 KB for 11x11) left LDS for six
// patches, so two of the four SIMDs had one wave; the weights were read from LDS beside the pixels for every rectangle; a
// layer of 128 channels staged and split every patch twice; and each of 40 loads of a lane fetched one tap of one channel, 64
// lines at a time.  Small calls took a kernel that loads, masks and splits its runs in the K loop.  Here:
//  * a lane keeps the signs of its columns (one of every 32 channels) for the whole launch, 32 bits for four K-steps of a column
//    (28 registers for 128 channels and 28 steps), and makes a bf16 operand register of them by a shift and a bit select, 2.7
//    vector instructions beside each 32-cycle MFMA;
//  * LDS holds nothing but eight patches, two waves for every SIMD; a K-step reads 3 KB for 3 NT MFMAs;
//  * the weights reach the lanes by way of LDS (the patches' space, idle until the first is staged): whole lines once per
//    workgroup, rows of bits, then the words.
// The patch of the wave's next rectangle is requested before the K loop and split after the epilogue; no barrier after the prologue.
// Measured, before -> now (weights included): 11x11, n x 224x224x3 -> 128: n = 1 31.7 -> 9.0 us, 16 33.5 -> 18.8, 64 61 -> 53.8, 128 107 -> 92;
// 7x7 stride 4 -> 64: n = 1 20.1 -> 5.8, 16 21.1 -> 7.7, 128 64 -> 33.5; stride 2 -> 64: n = 1 13.5 -> 5.7, 32 47 -> 29, 128 157 -> 94
// (two workgroups a compute unit there, which its patches and 114 registers allow: 88, but 8 x 112x112x3 5.7 -> 6.9).  The MFMAs of the 128-image 11x11 layer take 60 us (K slots 82 % full); the two
// waves of a SIMD overlap the rest of each other in part (another wave priority for one of them changes nothing).
#include <type_traits>

#include "bnn_bwn_wave.h"

namespace bnn {
namespace {

using wave::v16f;
using wave::v8bf;

template <int KS_, int STRIDE_, int FQ_>
struct RectGeom : wave::PatchGeom<KS_, STRIDE_, FQ_> {
    typedef wave::PatchGeom<KS_, STRIDE_, FQ_> B;
    static constexpr int TAPS = B::KS * B::KS;
    static constexpr int WQ = (B::NSTEPS + 3) / 4;                           // sign words of a column
    static constexpr size_t LDS = (size_t)B::WAVES * 3 * B::PLANE;
    static_assert(B::SEG <= 64 && LDS <= 160 * 1024, "a filter row of signs in two words; eight patches in LDS");
};

// bits 0, 2, 4, ... of a word, packed
__device__ __forceinline__ uint32_t even_bits(uint32_t v) {
    v &= 0x55555555u;
    v = (v | (v >> 1)) & 0x33333333u;
    v = (v | (v >> 2)) & 0x0F0F0F0Fu;
    v = (v | (v >> 4)) & 0x00FF00FFu;
    return (v | (v >> 8)) & 0x0000FFFFu;
}

template <class G, int NT, bool WANT_Y>
__global__ __launch_bounds__(G::WAVES * 64, 1) void bwn_rect_kernel(const float* __restrict__ x, const uint32_t* __restrict__ wbits,
                                                                   const float* __restrict__ thr, float* __restrict__ y,
                                                                   uint32_t* __restrict__ bits, wave::Args g) {
    constexpr int COLS = 32 * NT, NTHR = G::WAVES * 64;
    extern __shared__ uint4 smem[];
    const int tid = (int)threadIdx.x;
    const int lane = tid & 63, l32 = lane & 31, half = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);        // scalar: everything derived from the rectangle index stays scalar
    char* patch = reinterpret_cast<char*>(smem) + wave * (3 * G::PLANE);      // this wave's three planes
    const int n0 = (int)blockIdx.y * COLS;

    // this lane's output pixel inside a rectangle (rows vary fastest over the lanes: fewer bank conflicts of the 8-byte reads)
    const int dp = l32 % G::FP, dq = l32 / G::FP;
    const char* abase = patch + dp * (G::STRIDE * G::PITCH) + dq * (G::STRIDE * G::CIN * 2);
    const char* a_same = abase + half * 16;                                   // upper half-wave's run follows in the same filter row
    const char* a_next = abase + half * (G::PITCH - (G::RPR - 1) * 16);       // ... begins the next row

    wave::float2_ub pre[G::PR];                // the patch of the next rectangle, on its way
    const int ow = (g.O + 31) / 32;
    const int whole = g.ntiles / ((int)gridDim.x * G::WAVES);
    int t = wave::tile_of<G>(g, whole, 0, wave);
    if (t < g.ntiles) wave::request<G>(g, x, t, lane, pre);            // the first one while the weights are prepared
    else wave::no_request<G>(pre);

    float th[NT];
    bool cok[NT];
    wave::load_thresholds<NT, WANT_Y>(thr, bits, n0, l32, g.O, th, cok);
    uint32_t sw[G::WQ][NT];                    // step 4q + s, register i: element 2i at bit 4s + i, element 2i + 1 at bit 16 + 4s + i; set: -1
    {
        constexpr int RAW = COLS * G::TAPS, PER = (RAW + NTHR - 1) / NTHR;
        constexpr int ROWS = COLS * G::KS, WORDS = COLS * 2 * G::WQ;
        static_assert((size_t)(RAW + 2 * ROWS + WORDS) * 4 <= G::LDS, "the patches' space holds the weights first");
        uint32_t* raw = reinterpret_cast<uint32_t*>(smem);             // [column][tap]
        uint32_t* rows = raw + RAW;                                    // [column][filter row][2]: the row's values as bits, set: -1
        uint32_t* words = rows + 2 * ROWS;                             // [q][half][column]
        const uint32_t* src = wbits + (long long)n0 * G::TAPS;
        const int last = min(COLS, g.O - n0) * G::TAPS - 1;
        uint32_t v[PER];
#pragma unroll
        for (int i = 0; i < PER; ++i) v[i] = src[min(tid + i * NTHR, last)];
#pragma unroll
        for (int i = 0; i < PER; ++i)
            if (tid + i * NTHR < RAW) raw[tid + i * NTHR] = v[i];
        __syncthreads();
        for (int e = tid; e < ROWS; e += NTHR) {
            unsigned long long row = 0u;
#pragma unroll
            for (int tap = 0; tap < G::KS; ++tap) row |= (unsigned long long)(~raw[e * G::KS + tap] & 7u) << (3 * tap);
            rows[2 * e] = (uint32_t)row;
            rows[2 * e + 1] = (uint32_t)(row >> 32);
        }
        __syncthreads();
        for (int e = tid; e < WORDS; e += NTHR) {
            const int col = e % COLS, h = (e / COLS) & 1, q = e / (2 * COLS);
            uint32_t four = 0u;                                        // the runs of steps 4q .. 4q + 3, a byte each
#pragma unroll
            for (int s = 0; s < 4; ++s) {
                const int rho = 2 * (4 * q + s) + h;
                if (rho < G::NRUNS) {
                    const int r = rho / G::RPR, j = rho - r * G::RPR;
                    four |= ((rows[2 * (col * G::KS + r) + (j >> 2)] >> (8 * (j & 3))) & 0xFFu) << (8 * s);
                }
            }
            words[e] = even_bits(four) | (even_bits(four >> 1) << 16);
        }
        __syncthreads();
#pragma unroll
        for (int q = 0; q < G::WQ; ++q)
#pragma unroll
            for (int j = 0; j < NT; ++j) sw[q][j] = words[(2 * q + half) * COLS + 32 * j + l32];
        __syncthreads();                       // the last barrier: the patches' space is free
    }

    for (int r = 0; t < g.ntiles; ++r) {
        const int t_next = wave::tile_of<G>(g, whole, r + 1, wave);
        wave::stage<G>(g, t, lane, pre, patch);
        if (t_next < g.ntiles) wave::request<G>(g, x, t_next, lane, pre);

        v16f acc[NT];
#pragma unroll
        for (int j = 0; j < NT; ++j)
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[j][i] = 0.f;
        // the words are read anew for every rectangle: otherwise the compiler keeps expanded operands of all steps (and spills)
#pragma unroll
        for (int q = 0; q < G::WQ; ++q)
#pragma unroll
            for (int j = 0; j < NT; ++j) asm volatile("" : "+v"(sw[q][j]));
        // two operand sets: the reads and the expansion of step st + 1 run between the MFMAs of step st
        uint4 oa[2][3], ob[2][NT];
        auto fetch = [&](auto st_tag) {
            constexpr int st = decltype(st_tag)::value;
            constexpr int rho0 = 2 * st, rho1 = 2 * st + 1;
            constexpr bool upper = rho1 < G::NRUNS;                    // false: there is no run for the upper half-wave
            constexpr bool wraps = rho0 % G::RPR == G::RPR - 1;
            constexpr int off = (rho0 / G::RPR) * G::PITCH + (rho0 % G::RPR) * 16;
            const char* asrc = !upper ? abase : wraps ? a_next : a_same;
#pragma unroll
            for (int pl = 0; pl < 3; ++pl) oa[st & 1][pl] = wave::read_run<G>(asrc + off + pl * G::PLANE);
#pragma unroll
            for (int j = 0; j < NT; ++j) {
                uint32_t reg[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) reg[i] = ((sw[st / 4][j] << (15 - 4 * (st % 4) - i)) & 0x80008000u) | 0x3F803F80u;
                ob[st & 1][j] = make_uint4(reg[0], reg[1], reg[2], reg[3]);
            }
        };
        auto multiply = [&](auto st_tag) {
            constexpr int st = decltype(st_tag)::value;
            wave::clear_past_row<G, st>(oa[st & 1], half);             // (2 to 4 % of the time; as the values arrive 3 to 9)
#pragma unroll
            for (int pl = 2; pl >= 0; --pl)                            // smallest terms first
#pragma unroll
                for (int j = 0; j < NT; ++j)
                    acc[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(v8bf, oa[st & 1][pl]),
                                                                     __builtin_bit_cast(v8bf, ob[st & 1][j]), acc[j], 0, 0, 0);
        };
        fetch(std::integral_constant<int, 0>{});
        __builtin_amdgcn_sched_barrier(0);
        static_for<G::NSTEPS>([&](auto st_tag) {
            constexpr int st = decltype(st_tag)::value;
            if constexpr (st + 1 < G::NSTEPS) fetch(std::integral_constant<int, st + 1>{});
            multiply(st_tag);
            // keeps the reads and the expansion of the next step between this step's MFMAs
#pragma unroll
            for (int q = 0; q < 3 * NT; ++q) {
                __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);     // an MFMA
                __builtin_amdgcn_sched_group_barrier(0x002, 3, 0);     // vector instructions
                if (q % 2 == 0 || NT < 4) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);     // an LDS read
            }
            __builtin_amdgcn_sched_barrier(0);
        });

        wave::store<G, NT, WANT_Y>(g, t, acc, th, cok, y, bits, n0, ow, lane);
        t = t_next;                            // every read of this rectangle's patch has been consumed by its MFMAs
    }
}

struct RectCall {
    const float* x; const uint32_t* wbits; const float* thr; float* y; uint32_t* bits;
    double other;                              // what the caller's own kernel would take (launch_rect)
    int cus;
    hipStream_t s;
};

template <class G, int NT, bool WANT_Y>
int launch_rect_v(const RectCall& c, const wave::Args& g) {
    static const hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void*>(&bwn_rect_kernel<G, NT, WANT_Y>),
                                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)G::LDS);
    if (attr != hipSuccess) return BNN_ERR_DEVICE;
    const int col_tiles = (int)cdiv(g.O, 32 * NT);
    const int wgs = min(g.ntiles, max(1, c.cus / col_tiles));          // one workgroup per compute unit (LDS), resident for the whole call
    launch(bwn_rect_kernel<G, NT, WANT_Y>, dim3((unsigned)wgs, (unsigned)col_tiles), dim3(G::WAVES * 64), G::LDS, c.s, c.x, c.wbits, c.thr, c.y,
           c.bits, g);
    return check_launch();
}

template <class G, int NT>
int launch_rect_nt(const RectCall& c, const wave::Args& g) {
    return c.y != nullptr ? launch_rect_v<G, NT, true>(c, g) : launch_rect_v<G, NT, false>(c, g);
}

// false: the caller's own kernel is the faster one.
template <class G>
bool launch_rect(const RectCall& c, wave::Args g, int N, int* rc) {
    wave::set_tiles<G>(g, N);
    // Channels of a wave (32 NT): the least work for the SIMD with the most waves, the patch of a rectangle costing about as much as the
    // products of 16 channels and a wave that has its SIMD to itself, with nothing to overlap, a little more.  Measured, NT = 2 / 3 / 4, us:
    // n x 224x224x3 -> 128, 11x11: n = 4 8.6 / 10.5 / 12.1, 8 11.8 / 15.0 / 12.8, 12 15.2 / 19.7 / 18.2, 16 19.9 / 25.7 / 18.4, 64 53.7 / 69.5 / 51.5,
    // 128 99 / 130 / 91; -> 96: n = 4 8.6 / 10.1 / 12.0, 8 11.7 / 10.8 / 12.8, 64 53.2 / 41.9 / 50.7; 7x7 windows alike.
    int nt = 2;
    double best = 0.;
    for (int n = 2; n <= 4; ++n) {
        const long long per_simd = cdiv((long long)g.ntiles * cdiv(g.O, 32 * n), 4LL * c.cus);
        const double cost = (double)per_simd * (n + 0.5) + (per_simd == 1 ? 0.7 : 0.);
        if (n == 2 || cost < best) { best = cost; nt = n; }
    }
    // Many rectangles that the image leaves mostly empty: the direct kernel packs 32 consecutive outputs.  16977 images of 6 x 1 outputs -> 64, 7x7 stride 4, 76 us
    // here, 21 there; 16668 of 1 x 3 -> 128 58 and 18; 1642 of 41 x 3 -> 128 63 and 53; of 26 x 5 51 and 54.
    if (best > c.other) return false;
    *rc = nt == 4 ? launch_rect_nt<G, 4>(c, g) : nt == 3 ? launch_rect_nt<G, 3>(c, g) : launch_rect_nt<G, 2>(c, g);
    return true;
}

}  // namespace

bool try_bwn_rect(const float* x, const uint32_t* wbits, const float* thr, float* y, uint32_t* bits, int N, int H, int W, int C, int O,
                  int k, int stride, int pad, int P, int Q, double other, hipStream_t s, int* rc) {
    if (C != 3 || !(k == 7 ? stride == 2 || stride == 4 : k == 11 && stride == 4)) return false;
    if ((long long)H * W * C >= (1LL << 31)) return false;
    if ((long long)N * cdiv(P, 2) * cdiv(Q, 8) >= (1LL << 31) - 65536) return false;
    int dev = 0, cus = 0;
    if (hipGetDevice(&dev) != hipSuccess || hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus < 1) {
        *rc = BNN_ERR_DEVICE;
        return true;
    }
    wave::Args g = {};
    g.H = H; g.W = W; g.O = O; g.pad = pad; g.P = P; g.Q = Q;
    const RectCall c = {x, wbits, thr, y, bits, other, cus, s};
    if (k == 11) return launch_rect<RectGeom<11, 4, 8>>(c, g, N, rc);
    if (stride == 4) return launch_rect<RectGeom<7, 4, 8>>(c, g, N, rc);
    // 2 x 16 outputs, or 4 x 8 where the busiest SIMD then has fewer rectangles: 491 images of 79 x 3 outputs -> 192 99 -> 56 us (the kernel for staged patches 86), 426 of
    // 90 x 8 -> 64 37 -> 24 (34).  With as many it is the slower one by 3 to 5 %, four patch rows more: 12 images of 94 x 38 -> 32 6.6 -> 6.95.
    const long long col_tiles = cdiv(O, 64), wide = N * cdiv(P, 2) * cdiv(Q, 16), tall = N * cdiv(P, 4) * cdiv(Q, 8);
    if (cdiv(tall * col_tiles, 4LL * cus) < cdiv(wide * col_tiles, 4LL * cus)) return launch_rect<RectGeom<7, 2, 8>>(c, g, N, rc);
    return launch_rect<RectGeom<7, 2, 16>>(c, g, N, rc);
}

}  // namespace bnn
