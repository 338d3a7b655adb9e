// Matrix-core path for 3x3 convolutions (stride 1, pad 1) of 128, 256 and 512 channels: a workgroup owns a band of consecutive output
// pixels x 64 channels, as many bands as there are compute units, and every input pixel of the band lies in LDS as finished operands.
//
// What bounds the direct kernel there (256 x 14x14x256 -> 256 18.6 us, 256 x 7x7x512 -> 512 18.2): 392 tiles on 256 compute units, two on some
// and one on others, and every wave expanding its own pixels for each of nine taps, 10 vector instructions per MFMA.  Here:
//  * Bands are cut by row tiles of 32 pixels, not by the workgroup's tile: each compute unit gets the same number to within one (24 or 25 for
//    14x14x256).  A wave owns MT row tiles x 64 channels; what is left over is dealt as 32 x 32 tiles, one to a SIMD, so that the busiest SIMD has
//    13 tiles where 12.25 would be even (a wave tile more would be 16).
//  * LDS holds a cell per pixel, 16 bytes per word and one unit more (an odd pitch: neighbouring cells on different banks), in the padded coordinates
//    of the patch kernel: pitch W + 1, padding cells are data.  A tap's fragment is one 16-byte read at a constant offset.
//  * The filters stay packed: each wave reads them two chunks ahead and expands two words per K-step of 4 to 7 MFMAs.  (Timing-only builds that skip the
//    expansion, the filter loads or the pixel reads ran within 0.4 us of this one: the K loop is the matrix pipe's, 8.6 us for
//    59 G operations of random bits, 7.1 of zeros -- the clock falls with what toggles.  MFMAs alone, operands in registers: 7.2 and 6.9.)
//  * Filters are the row operand, channels dealt so that a half-wave owns 32 neighbours (dealt_column); accumulators start at 0.5 - threshold, so an output
//    bit is a sign.  What a chain adds (residual sums, bits, a 1x1 shortcut) is requested during the last chunk of K.
//  * 512 channels: the waves split K in two (the band is half as long at the same LDS), and meet once through LDS.
// Measured (launches queued one after another, direct or patch kernel -> this one): 256 x 14x14x256 -> 256 17.0 -> 13.0 us (4.55 PFLOP/s), 64 x 28x28x256 -> 512
// 31.6 -> 24.6, 256 x 7x7x512 -> 512 17.6 -> 15.7, 128 x 14x14x128 -> 512 11.8 -> 9.5; in a ResNet-18 of batch 256 the
// 14x14x256 layers 27.2 / 19.5 / 24.0 -> 23.3 / 16.2 / 18.4, the second convolutions at 28x28x128 32.7 / 24.4 -> 29.6 / 23.4, the forward 411 -> 383.
// Of the 13 us of a layer 4.5 are outside the K loop: launch 1.7, pixels and filters arriving 1, expansion 1.1, epilogue.
// Three row tiles per wave leave too few registers around the K loop: 13 to 14 spilled vector registers in the 512-channel forms, 54 with a residual sum, 9 to 13 in the
// 256-channel forms that keep sums with a shortcut or add one; none in the others.  Those of 54 are what the layer loses: 256 x 7x7x512 with a residual sum 22.8 us, bits alone 19.1.
#include "bnn_mfma_kernel.h"

namespace bnn {
namespace {

using mfma::v16f;
using mfma::v8i;
using mfma::as_operand;
using mfma::expand_unit;

struct BandArgs {
    int wp1, hp1;                // W + 1, H + 1
    FastDiv div_wp1, div_hp1;
    int images;
    int ntiles;                  // row tiles of 32 output pixels
    int nx, gy;                  // bands; 64-channel groups
    int start_at;                // 16-byte unit of the accumulators' start values
    uint32_t pad_keep;           // -1 padding: all ones (a padding cell is the expansion of 0 bits); excluded padding: 0 (fp4 zeros)
};

// Start values: [tile][half-wave][register], eight copies one unit more than a copy apart (the lanes LDS serves together read different units);
// with WK == 2 eight copies of zeros behind them, for the waves of the second half of K.
constexpr int START_PITCH = 64 + 4;

typedef uint32_t v4u __attribute__((ext_vector_type(4)));

// fast_div without a branch: divisions of several loads in flight stay in one block.
__device__ __forceinline__ int flat_div(int n, const FastDiv& f) {
    return (int)((f.m == 0u ? (uint32_t)n : __umulhi((uint32_t)n, f.m)) >> f.sh);
}

enum BandAdd { ADD_NONE, ADD_SHORTCUT, ADD_SUMS16, ADD_BITS };

// CW: words per pixel; MT: row tiles per wave; WAVES waves, in WK groups that split K.  SUMS: blocked 16-bit sums may leave beside the bits.  RES: what is
// added to the sums (one form each: registers that wait for the one are not kept for the others).
template <int CW, int MT, int WAVES, int WK, bool SUMS, int RES>
__global__ __launch_bounds__(64 * WAVES, 2) void conv_band_kernel(const uint32_t* __restrict__ A, const uint32_t* __restrict__ B, Geom g,
                                                                  Epi e, BandArgs ba) {
    constexpr int RW = WAVES / WK;                   // waves side by side over the rows
    constexpr int V = CW == 4 ? 2 : 4;               // words per lane and chunk: K-steps of a chunk
    constexpr int CH = CW / (2 * V) / WK;            // chunks per tap and wave
    constexpr int PITCH = (CW + 1) * 16;             // bytes of a cell (an odd number of units)
    extern __shared__ uint4 smem[];
    char* const lds = reinterpret_cast<char*>(smem);
    mfma::accumulators_in_agprs();

    const int tid = threadIdx.x, lane = tid & 63, l32 = lane & 31, half = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int rw = wave % RW, kh = wave / RW;
    // consecutive workgroups go round the 8 XCDs: a contiguous range of (band, group) for each, so that the groups of a band share an L2
    const int total = ba.nx * ba.gy, per_xcd = (total + 7) / 8;
    const int id = ((int)blockIdx.x & 7) * per_xcd + ((int)blockIdx.x >> 3);
    if (id >= total) return;                         // uniform for the workgroup
    const int bx = id / ba.gy, n0 = (id - bx * ba.gy) * 64;
    const int t0 = (int)((long long)bx * ba.ntiles / ba.nx), t1 = (int)((long long)(bx + 1) * ba.ntiles / ba.nx);
    const int rows = (int)g.rows;

    uint32_t c2;
    asm volatile("v_mov_b32 %0, 0x22222222" : "=v"(c2));

    // cell of tap (0, 0) of an output pixel
    auto cell_of = [&](int row) {
        const int n = flat_div(row, g.div_pq), rem = row - n * (g.P * g.Q);
        const int p = flat_div(rem, g.div_q), q = rem - p * g.Q;
        return (n * ba.hp1 + p) * ba.wp1 + q;
    };

    // ---- filters: lane (row l32 of a tile, half) reads words half * V .. + V - 1 of a chunk; two chunks ahead
    uint32_t boff[2];
#pragma unroll
    for (int j = 0; j < 2; ++j) boff[j] = (uint32_t)((n0 + mfma::dealt_column(j, l32)) * g.ldb_w + kh * 8 + half * V) * 4u;
    constexpr int RING = 3;
    uint32_t fw[RING][2][V];
    auto load_filters = [&](int c, int slot) {
        const char* base = reinterpret_cast<const char*>(B + (c / CH) * CW + (c % CH) * 8);    // uniform
#pragma unroll
        for (int j = 0; j < 2; ++j) mfma::load_words<V>(reinterpret_cast<const uint32_t*>(base + (size_t)boff[j]), fw[slot][j]);
    };
    load_filters(0, 0);
    load_filters(1, 1);

    // ---- the band's pixels
    const int cell0 = cell_of(32 * t0);
    const int ncells = cell_of(min(32 * t1, rows) - 1) - cell0 + 2 * ba.wp1 + 3;
    {
        constexpr int G4 = CW / 4, CELLS = 64 / G4;  // a wave's load: CELLS cells, 16 bytes per lane, the cells of neighbouring lanes neighbours
        const int grp = lane / CELLS;
        for (int first = wave * CELLS; first < ncells; first += 4 * WAVES * CELLS) {
            uint4 w[4];
            uint32_t keep[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int c = cell0 + min(first + u * WAVES * CELLS + lane % CELLS, ncells - 1);
                const int y = flat_div(c, ba.div_wp1), x = c - y * ba.wp1;
                const int n = flat_div(y, ba.div_hp1), yp = y - n * ba.hp1;
                const bool in = x > 0 && yp > 0 && n < ba.images;
                keep[u] = in ? 0xFFFFFFFFu : 0u;
                const uint32_t off = in ? (uint32_t)((n * g.H + yp - 1) * g.W + x - 1) * (uint32_t)(CW * 4) + grp * 16 : 0u;
                w[u] = *reinterpret_cast<const uint4*>(reinterpret_cast<const char*>(A) + (size_t)off);
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int cell = first + u * WAVES * CELLS + lane % CELLS;
                if (cell >= ncells) continue;
                uint4* dst = reinterpret_cast<uint4*>(lds + cell * PITCH) + grp * 4;
                const uint32_t c2v = c2 & (keep[u] | ba.pad_keep);
                dst[0] = expand_unit(w[u].x & keep[u], c2v);
                dst[1] = expand_unit(w[u].y & keep[u], c2v);
                dst[2] = expand_unit(w[u].z & keep[u], c2v);
                dst[3] = expand_unit(w[u].w & keep[u], c2v);
            }
        }
    }
    // what a second source multiplies beyond its width
    const int steps2 = RES == ADD_SHORTCUT ? (g.cw2 + 1) / 2 : 0, corr = RES == ADD_SHORTCUT ? steps2 * 64 - g.bits2 : 0;
    float* const start_all = reinterpret_cast<float*>(smem + ba.start_at);
    if (tid < 64) {
        const int lim = 1 << 20;                     // beyond every reachable sum (K <= 4608, residual sums are 16-bit)
        const float v = 0.5f - (float)(max(-lim, min(lim, e.thr[n0 + 32 * ((tid >> 4) & 1) + 16 * (tid >> 5) + (tid & 15)])) + corr);
#pragma unroll
        for (int cp = 0; cp < 8; ++cp) {
            start_all[cp * START_PITCH + tid] = v;
            if (WK == 2) start_all[(8 + cp) * START_PITCH + tid] = 0.f;
        }
    }
    __syncthreads();

    // ---- this wave's tiles: MT of its own, and one 32 x 32 tile of the row tiles that are left over
    const int own = t0 + rw * MT;
    const int left = t1 - t0 - RW * MT;              // <= WAVES / 2 (WK == 1: RW / 2)
    // (the extra tiles fall on different SIMDs: those of the two halves of K, and of two workgroups that share a compute unit)
    const int ex_id = WK == 2 ? (rw + 2 * kh) & 3 : WAVES == 4 ? (wave + 2 * (((int)blockIdx.x >> 8) & 1)) & 3 : wave;
    const int ex_tile = t0 + RW * MT + (ex_id >> 1), ex_j = ex_id & 1;
    const bool has_ex = (ex_id >> 1) < left;         // uniform

    uint32_t base[MT + 1];
#pragma unroll
    for (int i = 0; i < MT + 1; ++i) {
        const int tile = i < MT ? own + i : ex_tile;
        base[i] = (uint32_t)((cell_of(min(32 * min(tile, t1 - 1) + l32, rows - 1)) - cell0) * PITCH + (half * V + kh * 8) * 16);
    }
    const float* const start = start_all + ((l32 & 7) + 8 * kh) * START_PITCH + half * 16;
    // with or without an extra tile: two programs to their ends (where two forms of the K loop join, accumulators do not stay in place: 250 spilled registers)
    auto rest = [&](auto with) {
        constexpr bool EX = decltype(with)::value;
        constexpr int NA = MT + (EX ? 1 : 0), NM = 2 * MT + (EX ? 1 : 0);
        auto ex_filter = [&](const uint4 (&f)[2]) {
            return make_uint4(ex_j == 0 ? f[0].x : f[1].x, ex_j == 0 ? f[0].y : f[1].y, ex_j == 0 ? f[0].z : f[1].z, ex_j == 0 ? f[0].w : f[1].w);
        };
        v16f acc[MT][2], ex;
        auto begin = [&](v16f& a, int j, const float* from) {               // 0.5 - threshold of the register's channel
            const float4* sv = reinterpret_cast<const float4*>(from + j * 32);
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const float4 v = sv[q];
                a[4 * q] = v.x; a[4 * q + 1] = v.y; a[4 * q + 2] = v.z; a[4 * q + 3] = v.w;
            }
        };
#pragma unroll
        for (int i = 0; i < MT; ++i)
#pragma unroll
            for (int j = 0; j < 2; ++j) begin(acc[i][j], j, start);
        begin(ex, ex_j, start);
        auto mac = [](v16f& a, const uint4& f, const uint4& p) {
            a = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(as_operand(f), as_operand(p), a, 4, 4, 0, 0, 0, 0);
        };

        // K runs over the window's rows in a loop, over a row's 3 * CH chunks in straight code (all of it straight is three times 10 KB of
        // instructions that every launch fetches anew).  Pixel units and expanded filter words run one K-step ahead, packed filter words two chunks.
        const uint32_t row_pitch = (uint32_t)(ba.wp1 * PITCH);
        constexpr int ROW = 3 * CH * V;              // K-steps of a window row (even)
        uint4 fa[2][NA], fb[2][2];
        auto read_step = [&](auto step) {
            constexpr int s = decltype(step)::value % ROW, c = s / V, slot = s & 1;
#pragma unroll
            for (int i = 0; i < NA; ++i)
                fa[slot][i] = *reinterpret_cast<const uint4*>(lds + base[i] + ((c / CH) * PITCH + (c % CH) * 128 + (s % V) * 16));
#pragma unroll
            for (int j = 0; j < 2; ++j) fb[slot][j] = expand_unit(fw[c % RING][j][s % V], c2);
        };
        read_step(std::integral_constant<int, 0>{});
        // what the epilogue needs from memory, requested during the last chunk of K (behind the last filter words: loads return in order)
        constexpr int WAIT = 2 * MT / WK + (EX ? 1 : 0);
        uint4 rlo[WAIT], rhi[WAIT];                      // 16-bit residuals of the tiles this wave finishes
        uint32_t pw[2][NA], qw[2][2], rb[NA];            // two K-steps of the shortcut; residual bits
        const uint32_t* px[NA];
        const uint32_t* fl[2];
        auto pixel_row = [&](int i) { return min(32 * min(i < MT ? own + i : ex_tile, t1 - 1) + l32, rows - 1); };
        auto shortcut_request = [&](int ks) {
#pragma unroll
            for (int u = 0; u < 2; ++u) {                // past the end: loaded and not multiplied
                const int wo = 2 * (ks + u * WK) + half;
                const bool ok = wo < g.cw2;
#pragma unroll
                for (int i = 0; i < NA; ++i) { const uint32_t w = px[i][ok ? wo : 0]; pw[u][i] = ok ? w : 0u; }
#pragma unroll
                for (int j = 0; j < 2; ++j) { const uint32_t w = fl[j][ok ? wo : 0]; qw[u][j] = ok ? w : 0u; }
            }
        };
        auto block_of = [&](int tile, int j) { return ((long long)tile * (e.ldc >> 5) + ((n0 >> 5) + j)) * 1024 + lane * 16; };
        auto epilogue_request = [&]() {
            if constexpr (RES == ADD_SUMS16) {
#pragma unroll
                for (int u = 0; u < WAIT; ++u) {
                    const int t = u + (WK == 2 && kh == 1 ? MT : 0);                    // of this wave's 2 MT tiles
                    const bool extra = EX && u + 1 == WAIT;
                    const uint4* src = reinterpret_cast<const uint4*>(e.resid16 + block_of(extra ? ex_tile : min(own + (t >> 1), t1 - 1), extra ? ex_j : t & 1));
                    rlo[u] = src[0]; rhi[u] = src[1];
                }
            }
            if constexpr (RES == ADD_SHORTCUT) {
#pragma unroll
                for (int i = 0; i < NA; ++i) {
                    const int row = pixel_row(i);
                    const int n = flat_div(row, g.div_pq), rem = row - n * (g.P * g.Q);
                    const int p = flat_div(rem, g.div_q), q = rem - p * g.Q;
                    px[i] = g.A2 + (((long long)n * g.H2 + p * g.stride2) * g.W2 + q * g.stride2) * g.cw2;
                }
#pragma unroll
                for (int j = 0; j < 2; ++j) fl[j] = g.B2 + (long long)(n0 + mfma::dealt_column(j, l32)) * g.cw2;
                shortcut_request(kh);
            }
            if constexpr (RES == ADD_BITS) {
#pragma unroll
                for (int i = 0; i < NA; ++i)
                    rb[i] = e.resid_bits[(long long)pixel_row(i) * e.ld_resid_bits_w + min((n0 >> 5) + half, e.ld_resid_bits_w - 1)];
            }
        };
        auto window_row = [&](int r, auto last) {
            constexpr bool LAST = decltype(last)::value;
            static_for<ROW>([&](auto step) {
                constexpr int s = decltype(step)::value, c = s / V;
                if constexpr (s % V == 0 && (!LAST || c + 2 < 3 * CH)) load_filters(3 * CH * r + c + 2, (c + 2) % RING);
                if constexpr (WK == 1 && LAST && s == (3 * CH - 1) * V) epilogue_request();
                if constexpr (s + 1 == ROW && !LAST) {
#pragma unroll
                    for (int i = 0; i < NA; ++i) base[i] += row_pitch;
                }
                if constexpr (s + 1 < ROW || !LAST) read_step(std::integral_constant<int, s + 1>{});
#pragma unroll
                for (int i = 0; i < MT; ++i)
#pragma unroll
                    for (int j = 0; j < 2; ++j) mac(acc[i][j], fb[s & 1][j], fa[s & 1][i]);
                if constexpr (EX) mac(ex, ex_filter(fb[s & 1]), fa[s & 1][MT]);
#pragma unroll
                for (int q = 0; q < NM; ++q) {
                    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);   // an even mix: MFMA, vector ALU, LDS read
                    __builtin_amdgcn_sched_group_barrier(0x002, 3, 0);
                    __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
                }
                __builtin_amdgcn_sched_barrier(0);
            });
        };
#pragma unroll 1
        for (int r = 0; r < 2; ++r) window_row(r, std::false_type{});
        window_row(2, std::true_type{});
        if constexpr (WK == 2) epilogue_request();       // (the exchange below hides it; a chunk earlier 40 registers would spill)

        // ---- fused 1x1 shortcut: a few K-steps straight from memory, two at a time
        for (int ks = kh; RES == ADD_SHORTCUT && ks < steps2; ks += 2 * WK) {
            if (ks != kh) shortcut_request(ks);
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                if (ks + u * WK >= steps2) break;        // uniform
                uint4 f2[2];
#pragma unroll
                for (int j = 0; j < 2; ++j) f2[j] = expand_unit(qw[u][j], c2);
#pragma unroll
                for (int i = 0; i < MT; ++i) {
                    const uint4 p2 = expand_unit(pw[u][i], c2);
                    mac(acc[i][0], f2[0], p2);
                    mac(acc[i][1], f2[1], p2);
                }
                if constexpr (EX) mac(ex, ex_filter(f2), expand_unit(pw[u][MT], c2));
            }
        }
        // ---- a first residual taken from packed bits: one more K-step whose filter is the identity (-1.0 at the row's own channel: a 1 bit
        // expands to -1.0, so the product is +1)
        if (RES == ADD_BITS && kh == 0) {
            uint4 ident[2];
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                const int ch = mfma::dealt_column(j, l32);
                const uint4 u = expand_unit((ch >> 5) == half ? 1u << (ch & 31) : 0u, 0u);
                ident[j] = make_uint4(u.x | (u.x >> 2), u.y | (u.y >> 2), u.z | (u.z >> 2), u.w | (u.w >> 2));
            }
#pragma unroll
            for (int i = 0; i < NA; ++i) {
                const uint4 p2 = expand_unit(rb[i], c2);
                if (i < MT) { mac(acc[i][0], ident[0], p2); mac(acc[i][1], ident[1], p2); }
                else if constexpr (EX) mac(ex, ex_filter(ident), p2);
            }
        }

        // ---- epilogue: register r of tile j is channel n0 + 32 half + 16 j + r of pixel l32
        auto finish = [&](v16f& a, int tile, int j, int t) {     // t: its place among the residuals -> the signs of a lane's 16 sums, bit r = register r
            uint32_t m = 0u;
            if constexpr (!SUMS) {
#pragma unroll
                for (int r = 15; r >= 0; --r) m = __builtin_amdgcn_alignbit(m, __float_as_uint(a[r]), 31);
            } else {
                float v[16];
#pragma unroll
                for (int r = 0; r < 16; ++r) v[r] = a[r];
                if constexpr (RES == ADD_SUMS16) {
                    const uint4 lo = rlo[t], hi = rhi[t];
                    const uint32_t w[8] = {lo.x, lo.y, lo.z, lo.w, hi.x, hi.y, hi.z, hi.w};
#pragma unroll
                    for (int r = 0; r < 16; ++r) v[r] += (float)((r & 1) ? ((int)w[r >> 1] >> 16) : (int)(short)(w[r >> 1] & 0xffffu));
                }
#pragma unroll
                for (int r = 15; r >= 0; --r) m = __builtin_amdgcn_alignbit(m, __float_as_uint(v[r]), 31);
                if (e.out16 != nullptr) {
                    v16f st;
                    begin(st, j, start - 8 * kh * START_PITCH);
                    const float corrf = (float)corr;
                    uint32_t pk[8];
#pragma unroll
                    for (int q = 0; q < 8; ++q) {
                        const mfma::v2s two = __builtin_amdgcn_cvt_pk_i16((int)(v[2 * q] - (st[2 * q] + corrf)), (int)(v[2 * q + 1] - (st[2 * q + 1] + corrf)));
                        pk[q] = (uint32_t)(uint16_t)two[0] | ((uint32_t)(uint16_t)two[1] << 16);
                    }
                    uint4* dst = reinterpret_cast<uint4*>(e.out16 + block_of(tile, j));
                    dst[0] = make_uint4(pk[0], pk[1], pk[2], pk[3]);
                    dst[1] = make_uint4(pk[4], pk[5], pk[6], pk[7]);
                }
            }
            return m;
        };
        auto store_half = [&](uint32_t m, int tile, int j) {
            const long long row = 32LL * tile + l32;
            if (row < rows) reinterpret_cast<uint16_t*>(e.bits)[(row * e.ldbits_w + (n0 >> 5) + half) * 2 + j] = (uint16_t)~m;
        };
        if constexpr (WK == 1) {
#pragma unroll
            for (int i = 0; i < MT; ++i) {
                if (own + i >= t1) break;                // uniform
                const uint32_t lo = finish(acc[i][0], own + i, 0, 2 * i), hi = finish(acc[i][1], own + i, 1, 2 * i + 1);
                const long long row = 32LL * (own + i) + l32;
                if (row < rows) e.bits[row * e.ldbits_w + (n0 >> 5) + half] = ~((hi << 16) | lo);
            }
            if constexpr (EX) store_half(finish(ex, ex_tile, ex_j, WAIT - 1), ex_tile, ex_j);
        } else {
            // the two halves of K meet: each wave hands half of its tiles to its partner through LDS (the pixels are no longer needed)
            __syncthreads();
            uint4* const own_slot = smem + (rw * 2 * MT) * 256 + lane, *const ex_slot = smem + (RW * 2 * MT + ex_id) * 256 + lane;
            auto give = [&](const v16f& a, uint4* slot) {
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    slot[q * 64] = make_uint4(__float_as_uint(a[4 * q]), __float_as_uint(a[4 * q + 1]), __float_as_uint(a[4 * q + 2]), __float_as_uint(a[4 * q + 3]));
            };
            auto take = [&](v16f& a, const uint4* slot) {
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const uint4 v = slot[q * 64];
                    a[4 * q] += __uint_as_float(v.x); a[4 * q + 1] += __uint_as_float(v.y);
                    a[4 * q + 2] += __uint_as_float(v.z); a[4 * q + 3] += __uint_as_float(v.w);
                }
            };
            auto halves = [&](auto which) {              // this wave finishes the tiles t of 2 MT with (t < MT) == (which == 0)
                constexpr int K = decltype(which)::value;
#pragma unroll
                for (int t = 0; t < 2 * MT; ++t)
                    if ((t < MT) != (K == 0)) give(acc[t >> 1][t & 1], own_slot + t * 256);
                if constexpr (EX && K == 1) give(ex, ex_slot);
                __syncthreads();
#pragma unroll
                for (int t = 0; t < 2 * MT; ++t)
                    if ((t < MT) == (K == 0) && own + (t >> 1) < t1) {
                        take(acc[t >> 1][t & 1], own_slot + t * 256);
                        store_half(finish(acc[t >> 1][t & 1], own + (t >> 1), t & 1, t % MT), own + (t >> 1), t & 1);
                        __builtin_amdgcn_sched_barrier(0);   // one tile's values at a time
                    }
                if constexpr (EX && K == 0) {
                    take(ex, ex_slot);
                    store_half(finish(ex, ex_tile, ex_j, WAIT - 1), ex_tile, ex_j);
                }
            };
            if (kh == 0) halves(std::integral_constant<int, 0>{});
            else halves(std::integral_constant<int, 1>{});
        }
    };
    if (has_ex) rest(std::true_type{});
    else rest(std::false_type{});
}

constexpr size_t BAND_LDS = 160 * 1024;

struct BandPlan {
    bool ok;
    int kind, add, mt, waves, wk;
    BandArgs ba;
    size_t lds_bytes;
};

// Most cells a band of `pixels` consecutive output pixels spans.
long long band_cells(const Geom& g, long long pixels) {
    return pixels - 1 + ((pixels - 1) / g.Q + 1) + ((pixels - 1) / ((long long)g.P * g.Q) + 1) * (g.W + 1) + 2 * (g.W + 1) + 3;
}

BandPlan plan_band(const Geom& g, const Epi& e) {
    BandPlan pl = {};
    if (!g.conv || g.k != 3 || g.stride != 1 || g.pad != 1 || g.taps != 9 || g.pool2) return pl;
    if ((g.tw != 4 && g.tw != 8 && g.tw != 16) || g.bits_tap != g.tw * 32 || g.lda_w != g.tw) return pl;
    if (g.cols % 64 != 0 || g.P != g.H || g.Q != g.W || g.rows >= (1LL << 31) - 1024) return pl;
    pl.kind = mfma::epilogue_kind(e, true, false);
    if (pl.kind != mfma::EPI_BITS && pl.kind != mfma::EPI_CHAIN) return pl;
    if (e.ldbits_w * 32 != g.cols) return pl;
    // a block adds one thing to its sums
    if ((g.A2 != nullptr) + (e.resid16 != nullptr) + (e.resid_bits != nullptr) > 1) return pl;
    pl.add = g.A2 != nullptr ? ADD_SHORTCUT : e.resid16 != nullptr ? ADD_SUMS16 : e.resid_bits != nullptr ? ADD_BITS : ADD_NONE;
    if (pl.kind == mfma::EPI_CHAIN && pl.add == ADD_NONE) return pl;
    const long long images = g.rows / ((long long)g.P * g.Q);
    if ((images * (g.H + 1) + 2) * (g.W + 1) + 4096 >= (1LL << 31) || images * g.H * g.W * g.tw * 4 >= (1LL << 32)) return pl;
    if ((long long)g.cols * g.ldb_w * 4 >= (1LL << 32)) return pl;
    const int ntiles = (int)cdiv(g.rows, 32), gy = g.cols / 64;
    pl.wk = g.tw == 16 ? 2 : 1;
    pl.waves = g.tw == 4 ? 4 : 8;
    const int rw = pl.waves / pl.wk, slots = 256 * 8 / pl.waves, spare = pl.wk == 1 ? rw / 2 : 2;
    // Bands of equal length in whole rounds of the chip: the number of rounds and the row tiles per wave with the least estimated time.  per_simd: 32 x 32
    // tiles of the busiest SIMD; 9 * tw / 2 / wk K-steps of 34 cycles for each, 6000 cycles for what a round costs beside them.
    const int first = (int)cdiv((long long)ntiles * gy, (long long)slots * (rw * 3 + spare));
    double best = 0.;
    int nx = 0, rounds = 0, most = 0, busiest = 0;
    long long span = 0;                              // cells of a band
    for (int r = first; r <= first + 2; ++r) {
        const int n = (int)min((long long)ntiles, (long long)slots * r / gy);
        if (n == 0) continue;
        const int t = (int)cdiv(ntiles, n);
        if (t > rw * 3 + spare || t < rw) continue;
        const int mt = t <= rw + spare ? 1 : t <= 2 * rw + spare ? 2 : 3, left = max(0, t - rw * mt);
        const int per_simd = 4 * mt + (left == 0 ? 0 : 2 * left * pl.wk <= 4 ? 1 : 2);
        const double cost = r * (6000. + 9. * g.tw / 2 / pl.wk * per_simd * 34.);
        const size_t cells = (size_t)band_cells(g, 32LL * t) * (g.tw + 1);
        const size_t exchange = pl.wk == 2 ? (size_t)(rw * 2 * mt + 4) * 256 : 0, start_at = cells > exchange ? cells : exchange;
        const size_t bytes = start_at * 16 + 8 * pl.wk * START_PITCH * 4;
        if (bytes > BAND_LDS * pl.waves / 8 || (nx != 0 && cost >= best)) continue;
        best = cost; nx = n; rounds = r; most = t; busiest = per_simd; span = band_cells(g, 32LL * t);
        pl.mt = mt; pl.lds_bytes = bytes; pl.ba.start_at = (int)start_at;
    }
    if (nx == 0) return pl;
    // Where this kernel is the faster one (its speed over the patch and direct kernels'; 7x7 to 28x28, bands of every length up to three rounds, and bits of 1124
    // random layers of 5x5 to 200x200).  Beyond a round or two both kernels' times are staircases of different steps, so they are estimated in us: the direct kernel by the
    // tiles of its fullest compute unit, a round here by the tiles of the busiest SIMD and the cells of a band (median errors 1 to 2 %; 4 % at 512 channels).
    const int tile = mfma::pick_tile(g);
    const long long tile_rows = tile == 0 ? 256 : tile == 1 ? 512 : tile == 2 ? 128 : 64, tile_cols = tile == 0 || tile == 2 ? 128 : 64;
    const double fullest = (double)cdiv(cdiv(g.rows, tile_rows) * cdiv(g.cols, tile_cols), 256);
    // (A chain's decision may depend on the geometry alone, the same for every block of it: Epi::sums_tiled.  pick_tile() depends on excl only where
    // conv_stages_through_lds() does, from 320 words of K on; here there are 144 at most.)
    if (g.tw == 4) {
        // 128 channels in.  Up to 128 out, bits alone: 0.88 to 1.09 of the patch kernel, which stays.  With sums (chains of three blocks, whole): one round
        // 1.07 to 1.18, two 0.99 to 1.10, three 0.96 to 0.98.  More channels out, against the direct kernel: 0.92 to 1.01 up to 8 tiles, then 1.05 to 1.37.
        if (pl.kind == mfma::EPI_CHAIN ? rounds > 2 : g.cols <= 128 || (rounds == 1 && most <= 8)) return pl;
    } else if (g.tw == 8) {
        // 256 in: bits 0.96 to 1.02 at 8 tiles, from 9 on 1.04 to 1.4 (64 out: 1.05 to 1.7); chains 1.06 to 1.32.
        if (pl.kind == mfma::EPI_BITS && rounds == 1 && most <= 8) return pl;
        // 256 out with -1 padding, two rounds of 25 tiles: 1.25 to 1.32 here too (26 tiles 1.25, 27 and 28 1.17), but that 128 x 28x28x256 -> 256, which
        // is one of these, is the direct kernel's is tested behaviour of bnn_bconv_kernel_name.
        if (pl.kind == mfma::EPI_BITS && !g.excl && g.cols == 256 && rounds == 2 && most == 25) return pl;
        // The 25 random layers of 495 that this leaves or nearly leaves: 0.95 to 1.03, five rounds and wide images above all (19 x 146x139x256 -> 128 44.7 -> 47.0 us); chains of 61
        // to 64 tiles, three rounds, 0.955 to 0.985 (488 x 16x16x256), 60 tiles 1.07, 66 1.12.
        const double direct = tile == 0 ? 3.1 + 6.8 * fullest : tile == 1 ? 2.5 + 6.9 * fullest : tile == 2 ? 3.9 + 3.1 * fullest : 2.6 + 1.48 * fullest;
        const double corrects = pl.kind == mfma::EPI_BITS && g.excl ? 1.06 : 1.;        // (a chain's blocks choose alike)
        if (1.4 + rounds * (2.4 + 0.643 * busiest + 0.154e-3 * (double)span) > 1.02 * corrects * direct) return pl;
    } else if (g.cols > 64) {
        // 512 in: a round here 1.2 + 0.9 per tile of the busiest SIMD, the direct kernel 14.4 per 256x128 tile of the fullest compute unit, or 4.5 + 6.2 per 128x128 tile.
        // Bits: taken 1.02 to 1.58, left 0.91 to 1.0.  The second convolutions of three blocks of a chain (1x1 shortcut and residual with the
        // sum kept, residual alone) together: taken 1.01 to 1.44, left 0.85 to 1.0; alone each 0.97 to 1.6 where taken.
        const double direct = tile == 0 ? 14.4 * fullest : 4.5 + 6.2 * (double)cdiv(cdiv(g.rows, 128) * cdiv(g.cols, 128), 256);
        if (1. + rounds * (1.2 + 0.9 * busiest) > direct) return pl;
    } else if (tile == 1) {
        // 64 out: 1.0 to 1.74, but 0.92 and 0.97 for two of 86 (28 x 94x94x512 -> 64 30.3 -> 33.1 us).
        if (1.7 + rounds * (1.9 + 0.72 * busiest + 1e-3 * (double)span) > 1.06 * (1.5 + 13.7 * fullest)) return pl;
    }
    pl.ba.wp1 = g.W + 1; pl.ba.hp1 = g.H + 1;
    pl.ba.div_wp1 = make_fastdiv((uint32_t)(g.W + 1)); pl.ba.div_hp1 = make_fastdiv((uint32_t)(g.H + 1));
    pl.ba.images = (int)images;
    pl.ba.ntiles = ntiles; pl.ba.nx = nx; pl.ba.gy = gy;
    pl.ba.pad_keep = g.excl ? 0u : 0xFFFFFFFFu;
    pl.ok = true;
    return pl;
}

template <int CW, int MT, int WAVES, int WK, bool SUMS, int RES>
int launch_band_form(const uint32_t* A, const uint32_t* B, const Geom& g, const Epi& e, const BandPlan& pl, hipStream_t s) {
    static const hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void*>(&conv_band_kernel<CW, MT, WAVES, WK, SUMS, RES>),
                                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)BAND_LDS);
    if (attr != hipSuccess) return BNN_ERR_DEVICE;
    const unsigned nwg = (unsigned)(cdiv((long long)pl.ba.nx * pl.ba.gy, 8) * 8);
    launch((conv_band_kernel<CW, MT, WAVES, WK, SUMS, RES>), dim3(nwg), dim3(64 * WAVES), pl.lds_bytes, s, A, B, g, e, pl.ba);
    return check_launch();
}

template <int CW, int MT, int WAVES, int WK>
int launch_band(const uint32_t* A, const uint32_t* B, const Geom& g, const Epi& e, const BandPlan& pl, hipStream_t s) {
    if (pl.kind == mfma::EPI_BITS)
        return pl.add == ADD_SHORTCUT ? launch_band_form<CW, MT, WAVES, WK, false, ADD_SHORTCUT>(A, B, g, e, pl, s)
                                      : launch_band_form<CW, MT, WAVES, WK, false, ADD_NONE>(A, B, g, e, pl, s);
    switch (pl.add) {
        case ADD_SHORTCUT: return launch_band_form<CW, MT, WAVES, WK, true, ADD_SHORTCUT>(A, B, g, e, pl, s);
        case ADD_SUMS16: return launch_band_form<CW, MT, WAVES, WK, true, ADD_SUMS16>(A, B, g, e, pl, s);
        default: return launch_band_form<CW, MT, WAVES, WK, true, ADD_BITS>(A, B, g, e, pl, s);
    }
}

}  // namespace

bool mfma_conv_band_takes(const Geom& g, const Epi& e) { return plan_band(g, e).ok; }

int launch_mfma_conv_band(const uint32_t* A, const uint32_t* B, const Geom& g, const Epi& e, hipStream_t s) {
    const BandPlan pl = plan_band(g, e);
    if (!pl.ok) return BNN_ERR_UNSUPPORTED;
    auto with = [&](auto mt) {
        constexpr int MT = decltype(mt)::value;
        if (g.tw == 4) return launch_band<4, MT, 4, 1>(A, B, g, e, pl, s);
        if (g.tw == 8) return launch_band<8, MT, 8, 1>(A, B, g, e, pl, s);
        return launch_band<16, MT, 8, 2>(A, B, g, e, pl, s);
    };
    if (pl.mt == 1) return with(std::integral_constant<int, 1>{});
    if (pl.mt == 2) return with(std::integral_constant<int, 2>{});
    return with(std::integral_constant<int, 3>{});
}

}  // namespace bnn
