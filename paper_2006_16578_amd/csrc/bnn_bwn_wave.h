// What the first-layer kernels with wave-private patches share (conv_f32_wave_kernel of bnn_bwn.hip, bwn_rect_kernel of bnn_bwn_rect.hip): a wave owns a rectangle of
// FP x FQ = 32 output pixels, keeps the input patch under it in its own slice of LDS as three bf16 planes (fp32 values split exactly), walks the K loop from LDS
// only and stores bits (and sums).  Window, stride and channels are fixed at compile time, so every LDS address of the loop is a lane base plus an immediate.
#ifndef BNN_BWN_WAVE_H
#define BNN_BWN_WAVE_H

#include "bnn_internal.h"

namespace bnn {
namespace wave {

typedef float v16f __attribute__((ext_vector_type(16)));
typedef __bf16 v8bf __attribute__((ext_vector_type(8)));
typedef float float2_ub __attribute__((ext_vector_type(2), aligned(4)));       // 8-byte load, 4-byte aligned
extern "C" __device__ int bnn_wave_writelane_i32(int val, int lane, int old) __asm("llvm.amdgcn.writelane.i32");

template <int KS_, int STRIDE_, int FQ_>
struct PatchGeom {
    static constexpr int KS = KS_, STRIDE = STRIDE_, CIN = 3, FQ = FQ_, FP = 32 / FQ_, WAVES = 8;
    static constexpr int PR = (FP - 1) * STRIDE + KS;                        // patch rows
    static constexpr int ROW_ELEMS = ((FQ - 1) * STRIDE + KS) * CIN;         // input values of a patch row
    static constexpr int SEG = KS * CIN;                                     // values of one filter row
    static constexpr int RPR = (SEG + 7) / 8;                                // runs of 8 per filter row
    static constexpr int LAST = SEG - 8 * (RPR - 1);                         // values of a row's last run
    static constexpr int NRUNS = KS * RPR;
    static constexpr int NSTEPS = (NRUNS + 1) / 2;                           // MFMA K-steps (two runs each, one per half-wave)
    static constexpr int REACH = (FQ - 1) * STRIDE * CIN + 8 * RPR;          // farthest element a run reads from a patch row, + 1
    static constexpr int PITCH = (2 * (REACH > ROW_ELEMS ? REACH : ROW_ELEMS) + 7) / 8 * 8;    // bytes between patch rows
    static constexpr int PAIRS = PITCH / 4;                                  // 2-element units written per patch row (data + zeroed slack)
    static constexpr int PLANE = PR * PITCH;                                 // bytes of one bf16 plane of a patch
    static constexpr bool ALIGNED8 = (STRIDE * CIN * 2) % 8 == 0;            // of every run, else 4 bytes
    static_assert(FP * FQ == 32 && PAIRS <= 64 && (STRIDE * CIN * 2) % 4 == 0, "one lane per pair; aligned runs");
    static_assert(2 * (PAIRS - 1) >= ROW_ELEMS, "the last pair is slack: the lanes past it repeat its stores of zeros");
};

struct Args {
    int H, W, O, pad, P, Q;
    int tiles_p, tiles_q;
    int ntiles;              // images * tiles_p * tiles_q
    FastDiv div_tiles, div_tq;
};

template <class G>
inline void set_tiles(Args& g, int N) {
    g.tiles_p = (int)cdiv(g.P, G::FP); g.tiles_q = (int)cdiv(g.Q, G::FQ);
    g.ntiles = N * g.tiles_p * g.tiles_q;
    g.div_tiles = make_fastdiv((uint32_t)(g.tiles_p * g.tiles_q));
    g.div_tq = make_fastdiv((uint32_t)g.tiles_q);
}

template <class G>
__device__ __forceinline__ void tile_origin(const Args& g, int t, int& n, int& p0, int& q0) {
    n = fast_div(t, g.div_tiles);
    const int rem = t - n * (g.tiles_p * g.tiles_q);
    const int tp = fast_div(rem, g.div_tq);
    p0 = tp * G::FP;
    q0 = (rem - tp * g.tiles_q) * G::FQ;
}

// Rectangle of a wave in round r: whole rounds give a workgroup's waves consecutive rectangles; the last, partial round is dealt across the
// workgroups (wave 0 of each first), so that no compute unit runs a full extra round.  whole: g.ntiles / (gridDim.x * WAVES); g.ntiles: none.
template <class G>
__device__ __forceinline__ int tile_of(const Args& g, int whole, int r, int wave) {
    const int step = (int)gridDim.x * G::WAVES;
    if (r < whole) return r * step + (int)blockIdx.x * G::WAVES + wave;
    return r == whole ? whole * step + wave * (int)gridDim.x + (int)blockIdx.x : g.ntiles;
}

// No rectangle: the registers of its patch hold anything (without this the compiler clears them all).
template <class G>
__device__ __forceinline__ void no_request(float2_ub (&pre)[G::PR]) {
#pragma unroll
    for (int r = 0; r < G::PR; ++r) asm volatile("" : "=v"(pre[r]));
}

// Issues the loads of rectangle t's patch; nothing waits here.  Lane l holds elements 2l, 2l + 1 of every patch row.  A pair may hang over the left or right edge
// of the image row by one element (the padding is not a multiple of 2 elements): it is then loaded one element further in, and stage() picks the element that is data.
template <class G>
__device__ __forceinline__ void request(const Args& g, const float* __restrict__ x, int t, int lane, float2_ub (&pre)[G::PR]) {
    int n, p0, q0;
    tile_origin<G>(g, t, n, p0, q0);
    const int rowlen = g.W * G::CIN;                                                    // values per image row, >= 2 (H * W * C < 2^31: both checked on the host)
    const int y0 = p0 * G::STRIDE - g.pad;
    const int e0 = (q0 * G::STRIDE - g.pad) * G::CIN + 2 * lane;                        // first element of this lane's pair in the image row
    const uint32_t lane_bytes = (uint32_t)min(max(e0, 0), rowlen - 2) * 4u;
    const float* img = x + (long long)n * g.H * rowlen;                                 // uniform
#pragma unroll
    for (int r = 0; r < G::PR; ++r) {
        const int yy = min(max(y0 + r, 0), g.H - 1);                                    // uniform: rows outside the image are zeroed in stage()
        const char* rowp = reinterpret_cast<const char*>(img + yy * rowlen);            // uniform: scalar base + lane offset
        pre[r] = *reinterpret_cast<const float2_ub*>(rowp + lane_bytes);
    }
}

// Splits the requested patch of rectangle t into the wave's three planes.
template <class G>
__device__ __forceinline__ void stage(const Args& g, int t, int lane, const float2_ub (&pre)[G::PR], char* patch) {
    int n, p0, q0;
    tile_origin<G>(g, t, n, p0, q0);
    const int rowlen = g.W * G::CIN;
    const int y0 = p0 * G::STRIDE - g.pad;
    const int e0 = (q0 * G::STRIDE - g.pad) * G::CIN + 2 * lane;
    const bool shifted = min(max(e0, 0), rowlen - 2) != e0;
    // element validity as bit masks: inside the image row and inside the patch row's data (beyond it the row's slack is zeroed); rows above / below
    // the image are zeroed through a wave-uniform mask -- no branch in the loop
    const uint32_t m0 = (e0 >= 0 && e0 < rowlen && 2 * lane < G::ROW_ELEMS) ? 0xFFFFFFFFu : 0u;
    const uint32_t m1 = (e0 + 1 >= 0 && e0 + 1 < rowlen && 2 * lane + 1 < G::ROW_ELEMS) ? 0xFFFFFFFFu : 0u;
    char* dst = patch + 4 * min(lane, G::PAIRS - 1);
#pragma unroll
    for (int r = 0; r < G::PR; ++r) {
        const uint32_t ym = (unsigned)(y0 + r) < (unsigned)g.H ? 0xFFFFFFFFu : 0u;     // uniform
        // shifted by one element: the left-edge pair holds its second element first, the right-edge pair its first element second
        const uint32_t ua = __float_as_uint(shifted ? pre[r][1] : pre[r][0]) & m0 & ym;
        const uint32_t ub = __float_as_uint(shifted ? pre[r][0] : pre[r][1]) & m1 & ym;
        const float a = __uint_as_float(ua), b = __uint_as_float(ub);
        const float ra = a - __uint_as_float(ua & 0xffff0000u), rb = b - __uint_as_float(ub & 0xffff0000u);
        const uint32_t va = __float_as_uint(ra), vb = __float_as_uint(rb);
        const float la = ra - __uint_as_float(va & 0xffff0000u), lb = rb - __uint_as_float(vb & 0xffff0000u);
        *reinterpret_cast<uint32_t*>(dst + r * G::PITCH) = __builtin_amdgcn_perm(ub, ua, 0x07060302u);
        *reinterpret_cast<uint32_t*>(dst + r * G::PITCH + G::PLANE) = __builtin_amdgcn_perm(vb, va, 0x07060302u);
        *reinterpret_cast<uint32_t*>(dst + r * G::PITCH + 2 * G::PLANE) =
            __builtin_amdgcn_perm(__float_as_uint(lb), __float_as_uint(la), 0x07060302u);
    }
}

// A run of 8 values of one plane.
template <class G>
__device__ __forceinline__ uint4 read_run(const char* run) {
    if constexpr (G::ALIGNED8) {
        const uint2 lo = *reinterpret_cast<const uint2*>(run), hi = *reinterpret_cast<const uint2*>(run + 8);
        return make_uint4(lo.x, lo.y, hi.x, hi.y);
    } else {
        const uint32_t* w = reinterpret_cast<const uint32_t*>(run);
        return make_uint4(w[0], w[1], w[2], w[3]);
    }
}

// What a row's last run reads past the filter becomes zero in the values of K-step ST, not only in weights: a pixel that is not finite then touches no
// output whose window does not cover it.  To be called as the step is multiplied: as the values arrive, the masks wait for LDS a step early.
template <class G, int ST>
__device__ __forceinline__ void clear_past_row(uint4 (&a)[3], int half) {
    constexpr int v0 = (2 * ST) % G::RPR == G::RPR - 1 ? G::LAST : 8;                  // values of the run each half-wave multiplies
    constexpr int v1 = 2 * ST + 1 >= G::NRUNS ? 0 : (2 * ST + 1) % G::RPR == G::RPR - 1 ? G::LAST : 8;
    auto keep = [&](uint32_t v, int i) {
        const uint32_t m0 = (2 * i < v0 ? 0xFFFFu : 0u) | (2 * i + 1 < v0 ? 0xFFFF0000u : 0u);
        const uint32_t m1 = (2 * i < v1 ? 0xFFFFu : 0u) | (2 * i + 1 < v1 ? 0xFFFF0000u : 0u);
        return m0 == 0xFFFFFFFFu && m1 == 0xFFFFFFFFu ? v : v & (half ? m1 : m0);
    };
    if constexpr (v0 < 8 || v1 < 8)
#pragma unroll
        for (int pl = 0; pl < 3; ++pl) a[pl] = make_uint4(keep(a[pl].x, 0), keep(a[pl].y, 1), keep(a[pl].z, 2), keep(a[pl].w, 3));
}

// Thresholds of a lane's columns n0 + 32 j + l32: those past the last channel are never reached (NaN).
template <int NT, bool WANT_Y>
__device__ __forceinline__ void load_thresholds(const float* __restrict__ thr, const uint32_t* bits, int n0, int l32, int O, float (&th)[NT], bool (&cok)[NT]) {
#pragma unroll
    for (int j = 0; j < NT; ++j) {
        const int col = n0 + 32 * j + l32;
        cok[j] = col < O;
        th[j] = __builtin_nanf("");
        if (!WANT_Y || bits != nullptr) {
            const float v = thr[min(col, O - 1)];
            th[j] = cok[j] ? v : th[j];
        }
    }
}

// Threshold -> packed bits (and / or the fp32 sums) of rectangle t; without sums bits are always wanted.  ow: words of a pixel.
template <class G, int NT, bool WANT_Y>
__device__ __forceinline__ void store(const Args& g, int t, const v16f (&acc)[NT], const float (&th)[NT], const bool (&cok)[NT], float* __restrict__ y,
                                      uint32_t* __restrict__ bits, int n0, int ow, int lane) {
    const int l32 = lane & 31, half = lane >> 5;
    int n, p0, q0;
    tile_origin<G>(g, t, n, p0, q0);
    const long long img_pix = (long long)n * g.P * g.Q;
    uint32_t wout[NT];
#pragma unroll
    for (int j = 0; j < NT; ++j) wout[j] = 0u;
#pragma unroll
    for (int i = 0; i < 16; ++i) {
        const int lo_row = 8 * (i >> 2) + (i & 3);
#pragma unroll
        for (int j = 0; j < NT; ++j) {
            const float v = acc[j][i];
            if (WANT_Y) {
                const int m = lo_row + 4 * half;                   // rectangle pixel of this register in this lane
                const int mp = m % G::FP, mq = m / G::FP;
                if (p0 + mp < g.P && q0 + mq < g.Q && cok[j])
                    y[(img_pix + (long long)(p0 + mp) * g.Q + q0 + mq) * g.O + n0 + 32 * j + l32] = v;
            }
            if (!WANT_Y || bits != nullptr) {
                const unsigned long long ball = __builtin_amdgcn_ballot_w64(v >= th[j]);
                wout[j] = (uint32_t)bnn_wave_writelane_i32((int)(uint32_t)ball, lo_row, (int)wout[j]);
                wout[j] = (uint32_t)bnn_wave_writelane_i32((int)(uint32_t)(ball >> 32), lo_row + 4, (int)wout[j]);
            }
        }
    }
    const int dp = l32 % G::FP, dq = l32 / G::FP;                  // lane m < 32 holds the words of pixel m
    if ((!WANT_Y || bits != nullptr) && lane < 32 && p0 + dp < g.P && q0 + dq < g.Q) {
        const long long pix = img_pix + (long long)(p0 + dp) * g.Q + q0 + dq;
#pragma unroll
        for (int j = 0; j < NT; ++j) {
            const int wi = (n0 >> 5) + j;
            if (wi < ow) bits[pix * ow + wi] = wout[j];
        }
    }
}

}  // namespace wave
}  // namespace bnn
#endif
