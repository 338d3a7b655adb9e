// First layer with binarized weights for small windows (3x3, 5x5) of 3-channel images: one LDS record per input pixel,
// weights resident in registers.
//
// Same arithmetic as the kernels of bnn_bwn.hip: an fp32 value is the exact sum of three bf16 terms h + m + l, a +1/-1 weight is
// exact in bf16, the sums are accumulated in fp32 by v_mfma_f32_32x32x16_bf16 and compared with the fp32 threshold.
//
// What bounded the staged kernel of bnn_bwn.hip at these windows was everything beside the matrix pipe (33 % busy): K slots
// spent on padding (a filter row of 9 values took 16 slots in each of the three planes: 18 MFMAs per 32 pixels x 64 channels),
// 8-byte operand reads with bank conflicts, three 2-byte LDS stores for every input value, three vector instructions per
// accumulator register to pack its bits, and a patch that was loaded, multiplied and dropped with nothing overlapped.  Here:
//  * A pixel's nine terms are one 16-byte record (h0 h1 | h2 m0 | m1 m2 | l0 l1) plus l2 apart.  A K run (the 8 slots of a
//    half-wave) is ONE aligned 16-byte read, consecutive lanes consecutive records: a tap's record; the l2 terms of a filter row, kept as 8-byte units
//    (l2 of four consecutive pixels) beside the records, fill one more run per filter row.  K^2 + K runs in all -- 12 for
//    3x3, 12 MFMAs per 32 pixels x 64 channels, what the 81 products per output need at 16 slots an instruction.
//  * The weights are the MFMA's row operand and stay in registers for the whole launch (the workgroups are persistent), expanded
//    from their bits by each wave: no expansion launch, no weight traffic in the loop.
//  * Accumulator registers then hold 16 channels of one pixel.  With channels dealt to rows so that a half-wave owns 32
//    consecutive ones (row m of tile j: channel 32 * ((m >> 2) & 1) + 16 * j + 4 * (m >> 3) + m % 4), packing is a compare and
//    an add-with-carry per register (w = 2 w + bit), and a lane stores the finished word of its pixel.
//  * Two patch buffers: the next tile's pixels are requested before this tile is multiplied and split into the other buffer
//    after it; one barrier per tile.  The packed words leave only after that staging: memory operations retire in order, and
//    stores issued earlier put their latency in front of the wait for the pixels (103 -> 90 us back to back).
// Measured (input not in a cache), old -> this kernel: 128 x 224x224x3, 3x3, 64 channels 151 -> 78 us (with the expansion launch;
// 1.7 TB/s of input and output, the matrix pipe busy 47 %, 9.2 vector instructions per MFMA); stride 2 65 -> 36 us; 64 x 224x224x3, 5x5
// stride 1 139 -> 86 us, 128 channels stride 2 93 -> 53 us; small calls lose the expansion launch (2 to 3 us).
// Left: the MFMAs by themselves take 37 us at the clock held (12 in 187 ns per SIMD); the multiply phase alone, MFMAs and operand reads, about 55,
// packing alone 31, staging alone 34; two waves per SIMD overlap them in part.  Three waves per SIMD (one accumulator set, less read ahead) spill and are slower (101 us back to back against 94).
#include <type_traits>

#include "bnn_internal.h"

namespace bnn {
namespace {

typedef float v16f __attribute__((ext_vector_type(16)));
typedef __bf16 v8bf __attribute__((ext_vector_type(8)));

// Geometry fixed at compile time: window, stride, and the fragment (32 output pixels, FP rows x FQ columns), so that every LDS
// address of the K loop is one of four lane bases plus an immediate.  A tile is 4 * nf * FP rows x FQ columns, nf <= NF.
template <int K_, int STRIDE_, int FQ_>
struct PixGeom {
    static constexpr int K = K_, STRIDE = STRIDE_, FQ = FQ_, FP = 32 / FQ_;
    static constexpr int NF = STRIDE == 1 ? 4 : 2;                           // most fragments of a wave per tile
    static constexpr int PC = (FQ - 1) * STRIDE + K;                         // pixels of a patch row
    static constexpr int UNIT_SLACK = 3;                                     // l2 units in front of a row's: its first pixels write there too
    static constexpr int ROW16 = PC * 16, ROW8 = (PC + UNIT_SLACK) * 8;      // bytes of a patch row of records, of l2 units
    static constexpr int rows(int nf) { return (4 * nf * FP - 1) * STRIDE + K; }
    static constexpr int LDS_D = rows(NF) * ROW16;                           // l2 units behind the records
    static constexpr int LDS_BUF = (LDS_D + rows(NF) * ROW8 + 15) / 16 * 16;
    static constexpr int MAX_PX = rows(NF) * PC;
};

struct PixArgs {
    int H, W, O, pad, P, Q;
    int nf, PR, npx;        // fragments of a wave per tile; rows and pixels of a patch
    int tiles_p, tiles_q, ntiles;
    FastDiv div_tiles, div_tp;
};

__device__ __forceinline__ uint32_t bf16_sign(uint32_t word, int bit) {       // bit set: +1.0, clear: -1.0
    return 0x3F80u | ((~(word >> bit) & 1u) << 15);
}

// CT groups of 64 channels per workgroup (four waves each, sharing the patch).  WANT_Y: also store the fp32 sums (bits may be null then).
template <class G, int CT, bool WANT_Y>
__global__ __launch_bounds__(256 * CT, 2) void bwn_pixel_kernel(
    const float* __restrict__ x, const uint32_t* __restrict__ wbits, const float* __restrict__ thr, float* __restrict__ y,
    uint32_t* __restrict__ bits, PixArgs g) {
    constexpr int K = G::K, TAPS = K * K, STEPS = K * (K + 1) / 2, NTHR = 256 * CT, S = (G::MAX_PX + NTHR - 1) / NTHR;
    constexpr bool THR_LDS = K > 3;                 // thresholds in registers where the weights leave room for them
    constexpr bool OVERLAP = K == 3;                // a fragment is packed between the MFMAs of the next (5x5: no registers for two)
    constexpr int AHEAD = K == 3 ? 6 : 5;           // operand reads run this many K-steps ahead, across fragments
    static_assert((K == 3 || K == 5) && STEPS % AHEAD == 0, "an l2 run is at most two 8-byte units; operand slots are compile-time");
    extern __shared__ uint4 smem[];
    char* lds = reinterpret_cast<char*>(smem);      // two buffers: records [rows][PC] x 16 bytes, l2 units [rows][PC + UNIT_SLACK] x 8 bytes
    const int tid = (int)threadIdx.x;
    const int lane = tid & 63, l32 = lane & 31, half = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wrow = wave & 3, wcol = wave >> 2;
    const int n0 = ((int)blockIdx.y * CT + wcol) * 64;
    const int ow = (g.O + 31) >> 5;

    // ---- tiles of this workgroup: a contiguous range, rows fastest (vertical neighbours share halo rows in this XCD's L2)
    const int t_first = (int)(((long long)blockIdx.x * g.ntiles) / gridDim.x);
    const int t_end = (int)(((long long)(blockIdx.x + 1) * g.ntiles) / gridDim.x);
    struct At { int n, tp, tq; };
    At cur, nxt;
    nxt.n = fast_div(t_first, g.div_tiles);
    nxt.tq = fast_div(t_first - nxt.n * (g.tiles_p * g.tiles_q), g.div_tp);
    nxt.tp = t_first - nxt.n * (g.tiles_p * g.tiles_q) - nxt.tq * g.tiles_p;
    cur = nxt;
    auto advance = [&](At& at) {
        if (++at.tp == g.tiles_p) {
            at.tp = 0;
            if (++at.tq == g.tiles_q) { at.tq = 0; ++at.n; }
        }
    };
    const int TP = 4 * g.nf * G::FP;

    // ---- patch: thread -> S pixels, tid + i * NTHR, the same for every tile.  A tile whose patch lies inside the image (uniform)
    // needs no clamping and no masks.
    auto pixel = [&](int i) { return min(tid + i * NTHR, g.npx - 1); };
    uint32_t poff[S];                               // bytes from the patch's first pixel
#pragma unroll
    for (int i = 0; i < S; ++i) poff[i] = (uint32_t)(((pixel(i) / G::PC) * g.W + pixel(i) % G::PC) * 12);
    float pre[S][3];
    bool inner = false;                             // of the tile in `pre`: the whole patch is image
    int y0 = 0, x0 = 0;
    auto request = [&](const At& at) {
        y0 = at.tp * TP * G::STRIDE - g.pad;
        x0 = at.tq * (G::FQ * G::STRIDE) - g.pad;
        inner = y0 >= 0 && x0 >= 0 && y0 + g.PR <= g.H && x0 + G::PC <= g.W;
        const char* img = reinterpret_cast<const char*>(x + (long long)at.n * g.H * g.W * 3);
        if (inner) {
            const char* first = img + (long long)(y0 * g.W + x0) * 12;
#pragma unroll
            for (int i = 0; i < S; ++i) {
                const float* src = reinterpret_cast<const float*>(first + (size_t)poff[i]);
                pre[i][0] = src[0]; pre[i][1] = src[1]; pre[i][2] = src[2];
            }
        } else {
#pragma unroll
            for (int i = 0; i < S; ++i) {
                const int yy = min(max(y0 + pixel(i) / G::PC, 0), g.H - 1), xx = min(max(x0 + pixel(i) % G::PC, 0), g.W - 1);
                const float* src = reinterpret_cast<const float*>(img + (size_t)(uint32_t)((yy * g.W + xx) * 12));
                pre[i][0] = src[0]; pre[i][1] = src[1]; pre[i][2] = src[2];
            }
        }
    };
    const int l2_lane = G::LDS_D + 8 * G::UNIT_SLACK + tid * 8;
    auto stage = [&](int buf) {
        if (!inner) {                                               // zero padding
#pragma unroll
            for (int i = 0; i < S; ++i) {
                const bool in = (unsigned)(y0 + pixel(i) / G::PC) < (unsigned)g.H && (unsigned)(x0 + pixel(i) % G::PC) < (unsigned)g.W;
#pragma unroll
                for (int c = 0; c < 3; ++c) pre[i][c] = in ? pre[i][c] : 0.f;
            }
        }
#pragma unroll
        for (int i = 0; i < S; ++i) {
            const int e = tid + i * NTHR;
            if (e < g.npx) {
                uint32_t h[3], m[3], l[3];
#pragma unroll
                for (int c = 0; c < 3; ++c) {
                    h[c] = __float_as_uint(pre[i][c]);
                    const float r1 = pre[i][c] - __uint_as_float(h[c] & 0xffff0000u);     // exact: at most 16 significant bits left
                    m[c] = __float_as_uint(r1);
                    l[c] = __float_as_uint(r1 - __uint_as_float(m[c] & 0xffff0000u));     // exact: fits bf16
                }
                constexpr uint32_t HI = 0x07060302u;                                      // upper halves of two registers
                *reinterpret_cast<uint4*>(lds + buf + e * 16) =
                    make_uint4(__builtin_amdgcn_perm(h[1], h[0], HI), __builtin_amdgcn_perm(m[0], h[2], HI),
                               __builtin_amdgcn_perm(m[2], m[1], HI), __builtin_amdgcn_perm(l[1], l[0], HI));
                // slot d of the unit of pixel c - d is l2 of pixel c
                char* unit = lds + buf + l2_lane + i * (NTHR * 8) + (e / G::PC) * (8 * G::UNIT_SLACK);
                const unsigned short l2 = (unsigned short)(l[2] >> 16);
#pragma unroll
                for (int d = 0; d < (K < 4 ? K : 4); ++d) *reinterpret_cast<unsigned short*>(unit - 6 * d) = l2;
            }
        }
    };

    int t = t_first;
    if (t < t_end) request(nxt);

    // ---- weights and thresholds of a group of 64 channels: its four waves fetch them together, in whole lines, and pick them up
    // from LDS (the patch buffers, idle until the first patch is staged).  With every lane loading its own rows and thresholds, 41
    // loads of up to 20 lines each in front of the first product, 8 x 32x32x3 -> 128 took 6.5 us, now 5.2; 16 x 28x28x3 -> 200 with
    // 5x5 filters 10.2, now 7.5; 128 x 224x224x3 -> 64 the same 82.
    constexpr int WPC = 64 * TAPS, WREG = (WPC + 255) / 256;               // words of a channel group
    uint32_t* w_lds = reinterpret_cast<uint32_t*>(lds) + wcol * (WPC + 64);
    {
        const int lt = tid & 255, last = g.O * TAPS - 1;
        uint32_t v[WREG];
#pragma unroll
        for (int i = 0; i < WREG; ++i) v[i] = wbits[min(n0 * TAPS + lt + 256 * i, last)];
        const bool has_thr = !WANT_Y || bits != nullptr;                   // uniform
        float tv = __builtin_inff();
        if (has_thr) tv = thr[min(n0 + (lt & 63), g.O - 1)];
        tv = n0 + (lt & 63) < g.O ? tv : __builtin_inff();
#pragma unroll
        for (int i = 0; i < WREG; ++i)
            if (lt + 256 * i < WPC) w_lds[lt + 256 * i] = v[i];
        if (lt < 64) w_lds[WPC + lt] = __float_as_uint(tv);
    }
    __syncthreads();

    // ---- K-steps: which two runs (one per half-wave).  First the pairs of taps (r, 2i) / (r, 2i + 1), then the pairs of the last
    // column's taps, then the last tap beside the l2 terms of filter row 0, then the l2 terms of rows 2i - 1 and 2i.
    constexpr int SIDE = K * (K / 2), DOWN = K / 2, MIXED = SIDE + DOWN;
    auto tap_of = [](int s, int h) {                // for s <= MIXED (h = 0 in the mixed step)
        return s < SIDE ? (s / (K / 2)) * K + 2 * (s % (K / 2)) + h : s < MIXED ? (2 * (s - SIDE) + h) * K + K - 1 : TAPS - 1;
    };
    auto row_of = [](int s, int h) { return s == MIXED ? 0 : 2 * (s - MIXED) - 1 + h; };

    // ---- weights of this lane's two channels, one word per tap in memory
    uint4 wr[STEPS][2];
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        const int ch = n0 + 32 * ((l32 >> 2) & 1) + 16 * j + 4 * (l32 >> 3) + (l32 & 3);
        const uint32_t* row = w_lds + (ch - n0) * TAPS;
        const uint32_t live = ch < g.O ? 0xFFFFFFFFu : 0u;
#pragma unroll
        for (int s = 0; s < STEPS; ++s) {
            uint4 tap = make_uint4(0u, 0u, 0u, 0u), l2 = tap;
            if (s <= MIXED) {
                const uint32_t w = row[s == MIXED ? TAPS - 1 : half ? tap_of(s, 1) : tap_of(s, 0)];
                const uint32_t c0 = bf16_sign(w, 0), c1 = bf16_sign(w, 1), c2 = bf16_sign(w, 2);
                tap = make_uint4(c0 | (c1 << 16), c2 | (c0 << 16), c1 | (c2 << 16), c0 | (c1 << 16));
            }
            if (s >= MIXED) {
                const int r = s == MIXED ? 0 : half ? row_of(s, 1) : row_of(s, 0);
                uint32_t v[8] = {0u, 0u, 0u, 0u, 0u, 0u, 0u, 0u};
#pragma unroll
                for (int i = 0; i < K; ++i) v[i] = bf16_sign(row[r * K + i], 2);
                l2 = make_uint4(v[0] | (v[1] << 16), v[2] | (v[3] << 16), v[4] | (v[5] << 16), v[6] | (v[7] << 16));
            }
            const bool is_tap = s < MIXED || (s == MIXED && half == 0);
            wr[s][j] = make_uint4((is_tap ? tap.x : l2.x) & live, (is_tap ? tap.y : l2.y) & live, (is_tap ? tap.z : l2.z) & live,
                                  (is_tap ? tap.w : l2.w) & live);
        }
    }
    // ---- thresholds: register r of tile j holds channel n0 + 32 * half + 16 * j + r
    float* thr_lds = reinterpret_cast<float*>(lds + 2 * G::LDS_BUF) + wcol * 64;
    float th[THR_LDS ? 1 : 32];
    if constexpr (THR_LDS) {
        if (wrow == 0) thr_lds[lane] = __uint_as_float(w_lds[WPC + lane]);
    } else {
#pragma unroll
        for (int i = 0; i < 32; ++i) th[i] = __uint_as_float(w_lds[WPC + 32 * half + i]);
    }
    __syncthreads();

    // ---- l2 slots no pixel writes (behind the end of a patch row) must read as finite values: their weights are 0
    for (int e = tid; e < g.PR * (G::PC + G::UNIT_SLACK); e += NTHR)
#pragma unroll
        for (int b = 0; b < 2; ++b) *reinterpret_cast<uint2*>(lds + b * G::LDS_BUF + G::LDS_D + e * 8) = make_uint2(0u, 0u);
    __syncthreads();

    // ---- lane bases of the runs of this wave's fragment 0 in buffer 0
    const int dp = l32 / G::FQ, dq = l32 % G::FQ;
    const int prow = (wrow * g.nf * G::FP + dp) * G::STRIDE, pcol = dq * G::STRIDE;
    const int base16 = prow * G::ROW16 + pcol * 16, base8 = G::LDS_D + prow * G::ROW8 + (pcol + G::UNIT_SLACK) * 8;
    const int b_side = base16 + half * 16, b_down = base16 + half * G::ROW16 + (K - 1) * 16;
    const int b_mix = half ? base8 : base16 + (K - 1) * (G::ROW16 + 16);
    const int b_l2 = base8 + G::ROW8 + half * G::ROW8;
    const int mix_step = half ? G::FP * G::STRIDE * G::ROW8 : G::FP * G::STRIDE * G::ROW16;     // from fragment to fragment
    const uint32_t tap_lane = half ? 0u : 0xFFFFFFFFu;
    const uint32_t out_lane = (uint32_t)(((dp * g.Q + dq) * ow + (n0 >> 5) + half) * 4);

    // ---- one fragment: its K-steps, with the packing of the fragment before it between the MFMAs (a wave alone keeps both
    // pipes busy; left in sequence, the two phases of a wave add up and two waves per SIMD cannot hide them)
    uint4 a[AHEAD];
    auto read = [&](int s, int buf, int f) {
        const int f16 = f * (G::FP * G::STRIDE * G::ROW16), f8 = f * (G::FP * G::STRIDE * G::ROW8);
        uint4& r = a[s % AHEAD];
        if (s < SIDE) {
            r = *reinterpret_cast<const uint4*>(lds + (b_side + buf) + f16 + (s / (K / 2)) * G::ROW16 + (s % (K / 2)) * 32);
        } else if (s < MIXED) {
            r = *reinterpret_cast<const uint4*>(lds + (b_down + buf) + f16 + 2 * (s - SIDE) * G::ROW16);
        } else {
            const char* src = s == MIXED ? lds + (b_mix + buf + f * mix_step) : lds + (b_l2 + buf) + f8 + 2 * (s - MIXED - 1) * G::ROW8;
            const uint2 lo = *reinterpret_cast<const uint2*>(src);
            uint2 hi = make_uint2(0u, 0u);
            // the second half: the rest of the tap's record, or the l2 terms of the filter row's fifth pixel
            if (K == 3) { if (s == MIXED) hi = *reinterpret_cast<const uint2*>(src + 8); }
            else hi = *reinterpret_cast<const uint2*>(src + (s == MIXED && half == 0 ? 8 : 32));
            r = make_uint4(lo.x, lo.y, hi.x, hi.y);
        }
    };
    // Slots past a filter row's end hold other pixels' terms against zero weights: cleared, so that a NaN there stays there.
    auto operand = [&](int s) {
        uint4 r = a[s % AHEAD];
        const uint32_t keep = s == MIXED ? tap_lane : 0u;
        if (s >= MIXED) {
            if (K == 3) { r.y &= keep | 0xFFFFu; r.z &= keep; r.w &= keep; }
            else { r.z &= keep | 0xFFFFu; r.w &= keep; }
        }
        return r;
    };
    uint32_t word[G::NF];
    auto pack_quad = [&](const v16f (&acc)[2], uint32_t& w, int i) {     // channels i .. i + 3 of this lane's 32, i descending
        float tq[4];
        if constexpr (THR_LDS) {
            const float4 v = *reinterpret_cast<const float4*>(thr_lds + 32 * half + i);
            tq[0] = v.x; tq[1] = v.y; tq[2] = v.z; tq[3] = v.w;
        } else {
            tq[0] = th[i]; tq[1] = th[i + 1]; tq[2] = th[i + 2]; tq[3] = th[i + 3];
        }
        const v16f& v = acc[i >> 4];
        const int r = i & 15;
        push4(w, __builtin_amdgcn_ballot_w64(v[r + 3] >= tq[3]), __builtin_amdgcn_ballot_w64(v[r + 2] >= tq[2]),
              __builtin_amdgcn_ballot_w64(v[r + 1] >= tq[1]), __builtin_amdgcn_ballot_w64(v[r] >= tq[0]));
    };
    long long img_pix = 0;
    int p0 = 0, q0 = 0;
    auto store_sums = [&](const v16f (&acc)[2], int f) {
        const int frow = p0 + (wrow * g.nf + f) * G::FP;
        if (frow + dp < g.P && q0 + dq < g.Q) {
            float* dst = y + (img_pix + (long long)(frow + dp) * g.Q + q0 + dq) * g.O + n0 + 32 * half;
#pragma unroll
            for (int i = 0; i < 32; ++i)
                if (n0 + 32 * half + i < g.O) dst[i] = acc[i >> 4][i & 15];
        }
    };
    auto multiply = [&](auto f_tag, v16f (&acc)[2], const v16f (&prev)[2], int buf) {
        constexpr int f = decltype(f_tag)::value;
        const v16f zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int s = 0; s < STEPS; ++s) {
            const uint4 r = operand(s);
            if (s + AHEAD < STEPS) read(s + AHEAD, buf, f);
            else if (f + 1 < G::NF) read(s + AHEAD - STEPS, buf, f + 1);
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                acc[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(v8bf, wr[s][j]), __builtin_bit_cast(v8bf, r),
                                                                 s == 0 ? zero : acc[j], 0, 0, 0);
                __builtin_amdgcn_sched_barrier(0);
                const int m = 2 * s + j;                            // the eight quads spread over the 2 * STEPS MFMAs
                if constexpr (OVERLAP && f > 0) if (m * 8 / (2 * STEPS) != (m + 1) * 8 / (2 * STEPS)) {
                    pack_quad(prev, word[f - 1], 28 - 4 * (m * 8 / (2 * STEPS)));
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
        }
        if (WANT_Y) store_sums(acc, f);
    };
    auto flush = [&](const v16f (&acc)[2], uint32_t& w) {
#pragma unroll
        for (int i = 28; i >= 0; i -= 4) pack_quad(acc, w, i);
    };

    if (t < t_end) stage(0);
    __syncthreads();
    int buf = 0;
    for (; t < t_end; ++t) {
        const bool more = t + 1 < t_end;
        advance(nxt);
        if (more) request(nxt);
        p0 = cur.tp * TP; q0 = cur.tq * G::FQ;
        img_pix = (long long)cur.n * g.P * g.Q;
        // fragments of this wave that hold output rows (uniform)
        const int nf = min(g.nf, max(0, (g.P - p0 - wrow * g.nf * G::FP + G::FP - 1) / G::FP));
        v16f acc[2][2];
#pragma unroll
        for (int f = 0; f < G::NF; ++f) word[f] = 0u;
        if (nf > 0) {
#pragma unroll
            for (int s = 0; s < AHEAD; ++s) read(s, buf, 0);
            static_for<G::NF>([&](auto f_tag) {
                constexpr int f = decltype(f_tag)::value;
                if (f < nf) {
                    multiply(f_tag, acc[OVERLAP ? f & 1 : 0], acc[(f + 1) & 1], buf);
                    if (!OVERLAP) flush(acc[0], word[f]);
                }
            });
            if (OVERLAP) {
                uint32_t w = 0u;
                if (nf & 1) flush(acc[0], w);
                else flush(acc[1], w);
#pragma unroll
                for (int f = 0; f < G::NF; ++f) word[f] = f == nf - 1 ? w : word[f];
            }
        }
        buf = G::LDS_BUF - buf;
        if (more) stage(buf);
        // The words leave only now: memory operations retire in order, so stores issued before the staging would put their
        // own latency in front of the wait for the next tile's pixels.
        if ((!WANT_Y || bits != nullptr) && q0 + dq < g.Q && (n0 >> 5) + half < ow) {
            const int frow = p0 + wrow * g.nf * G::FP;
            char* out = reinterpret_cast<char*>(bits + (img_pix + (long long)(frow * g.Q + q0)) * ow);     // uniform
#pragma unroll
            for (int f = 0; f < G::NF; ++f)
                if (f < nf && frow + f * G::FP + dp < g.P)
                    *reinterpret_cast<uint32_t*>(out + (size_t)(out_lane + (uint32_t)(f * G::FP * g.Q * ow * 4))) = word[f];
        }
        cur = nxt;
        __syncthreads();
    }
}

struct PixCall {
    const float* x; const uint32_t* wbits; const float* thr; float* y; uint32_t* bits;
    int N, cus;
    hipStream_t s;
};

template <class G, int CT, bool WANT_Y>
int launch_pixel_v(const PixCall& c, PixArgs g) {
    constexpr size_t lds = (size_t)2 * G::LDS_BUF + (G::K > 3 ? 256 * CT : 0);
    static_assert(lds <= 160 * 1024, "two patches fit LDS");
    static_assert(CT * (64 * G::K * G::K + 64) * 4 <= 2 * G::LDS_BUF, "the patch buffers hold the weights first");
    static const hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void*>(&bwn_pixel_kernel<G, CT, WANT_Y>),
                                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (attr != hipSuccess) return BNN_ERR_DEVICE;
    const int TP = 4 * g.nf * G::FP;
    g.PR = G::rows(g.nf); g.npx = g.PR * G::PC;
    g.tiles_p = (int)cdiv(g.P, TP); g.tiles_q = (int)cdiv(g.Q, G::FQ);
    g.ntiles = c.N * g.tiles_p * g.tiles_q;
    g.div_tiles = make_fastdiv((uint32_t)(g.tiles_p * g.tiles_q)); g.div_tp = make_fastdiv((uint32_t)g.tiles_p);
    const int ct = (int)cdiv(g.O, 64 * CT);
    // workgroups resident at a time: what registers (launch bounds) and LDS allow
    const long long per_cu = min((long long)(2 / CT), (long long)(160 * 1024 / lds));
    const long long wgs = min((long long)g.ntiles, max(1LL, c.cus * per_cu / ct));
    launch((bwn_pixel_kernel<G, CT, WANT_Y>), dim3((unsigned)wgs, (unsigned)ct), dim3(256 * CT), lds, c.s, c.x, c.wbits, c.thr, c.y, c.bits, g);
    return check_launch();
}

template <class G, int CT>
int launch_pixel(const PixCall& c, const PixArgs& g) {
    return c.y != nullptr ? launch_pixel_v<G, CT, true>(c, g) : launch_pixel_v<G, CT, false>(c, g);
}

template <int K, int STRIDE, int CT>
int launch_pixel_fq(const PixCall& c, const PixArgs& g, int FQ) {
    return FQ == 32 ? launch_pixel<PixGeom<K, STRIDE, 32>, CT>(c, g)
         : FQ == 16 ? launch_pixel<PixGeom<K, STRIDE, 16>, CT>(c, g) : launch_pixel<PixGeom<K, STRIDE, 8>, CT>(c, g);
}

template <int K, int STRIDE>
int launch_pixel_ct(const PixCall& c, const PixArgs& g, int FQ) {
    return g.O > 64 ? launch_pixel_fq<K, STRIDE, 2>(c, g, FQ) : launch_pixel_fq<K, STRIDE, 1>(c, g, FQ);
}

}  // namespace

bool try_bwn_pixel(const float* x, const uint32_t* wbits, const float* thr, float* y, uint32_t* bits, int N, int H, int W, int C, int O,
                   int k, int stride, int pad, int P, int Q, hipStream_t s, int* rc) {
    if (C != 3 || !(k == 3 || k == 5) || !(stride == 1 || stride == 2)) return false;
    // 32-bit byte offsets inside one image, tile indices
    if ((long long)H * W * 12 >= (1LL << 31) || (long long)P * Q * ((O + 31) / 32) * 4 >= (1LL << 31)) return false;
    if ((long long)N * (P + 128LL) * (Q + 32LL) >= (1LL << 31)) return false;
    int dev = 0, cus = 0;
    if (hipGetDevice(&dev) != hipSuccess || hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus < 1) {
        *rc = BNN_ERR_DEVICE;
        return true;
    }
    // Tile: the fragment shape and the number of fragments per wave with the least work for the workgroups that run side by side, a
    // patch pixel costing about as much as a third of an output pixel and a tile itself as much as a hundred; small calls get small
    // tiles (more workgroups) that way.
    PixArgs g = {};
    g.H = H; g.W = W; g.O = O; g.pad = pad; g.P = P; g.Q = Q;
    int FQ = 32;
    double best = 0.;
    for (int fq = 32; fq >= 8; fq /= 2)
        for (int nf = stride == 1 ? 4 : 2; nf >= 1; nf /= 2) {
            const int TP = 4 * nf * (32 / fq);
            const long long tiles = N * cdiv(P, TP) * cdiv(Q, fq) * cdiv(O, 64);
            const double px = ((TP - 1.) * stride + k) * ((fq - 1.) * stride + k);
            const double cost = (double)cdiv(tiles, 2LL * cus) * (TP * fq + px / 3. + 100.);
            if (g.nf == 0 || cost < best) { best = cost; g.nf = nf; FQ = fq; }
        }
    const PixCall c = {x, wbits, thr, y, bits, N, cus, s};
    if (k == 3) *rc = stride == 1 ? launch_pixel_ct<3, 1>(c, g, FQ) : launch_pixel_ct<3, 2>(c, g, FQ);
    else *rc = stride == 1 ? launch_pixel_ct<5, 1>(c, g, FQ) : launch_pixel_ct<5, 2>(c, g, FQ);
    return true;
}

}  // namespace bnn
