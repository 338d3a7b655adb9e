// Convolutions of any window, stride, channel count and padding convention on the matrix cores: the input patch under a
// workgroup's output pixels is expanded to E2M1 ONCE, on its way into LDS, and the waves read finished pixel operands; the
// filters stay packed in global memory / L2 and every wave expands its own two filter fragments a K-step ahead.
//
// What bounds the direct kernel (bnn_mfma_kernel.h) at windows and channel counts it has no unrolled form for: every K-step gathers
// its words with 4-byte loads, masks them per tap, and expands both operands -- 25 vector instructions per MFMA at 96 channels and
// a 5x5 window, a third of the K slots spent on rounding each tap up to whole K-steps, the matrix pipe busy 18 % of the time.  Here:
//  * LDS holds one 16-byte unit per pixel and 32-channel word (the four operand registers of a lane), in planes [word][pixel]:
//    the 32 pixels of a fragment read 32 consecutive units, interrupted where it crosses an image row (two units to a bank at stride 2).  A tap's pixel is a constant offset
//    away, so K runs over the flattened words of a filter, whatever the channel count: words 8c .. 8c + 3 of chunk c go to the
//    lower half-wave, 8c + 4 .. 8c + 7 to the upper one; only the last chunk of a filter can be partly empty (its missing words are units of zeros).
//  * Padding is data: an out-of-frame pixel is the unit of -1 bits, or with excluded padding a unit of zeros, and the bits past the
//    last channel are zeros too, so that no K slot needs a mask and no sum needs a correction in either convention.
//  * A K-step of a wave (128 pixels x 64 channels) is eight MFMAs, four 16-byte LDS reads and, by the source, about twenty vector instructions
//    (expansion of two filter words, four addresses); over the whole kernel, staging and epilogue included, 6.9 per MFMA are counted.
//  * Bits only: the filters are the MFMA's row operand, with channels dealt to its rows so that a half-wave owns 32 consecutive
//    ones; packing is a compare and an add-with-carry per accumulator register, and a lane stores whole words of its pixel.
//    Everything else keeps pixels as rows and the shared epilogue (32 consecutive channels per store instruction).
// Measured (graph replay of single launches, direct kernel -> this one): 64 x 27x27x96 -> 200, 5x5, excluded padding 46.8 -> 19.4 us (43.7 -> 17.6 as
// passes queued one after another); 128 x 56x56x48 -> 48, 3x3, excluded padding 48.8 -> 18.3; 128 x 28x28x96 -> 192, 3x3 27.3 -> 20.0;
// 100 x 9x9x300 -> 300 18.6 -> 11.8.  Parts switched off in the first shape: K loop 12.8 us (20 % above what its MFMAs take where a
// SIMD has two waves), staging 1.5, launch and epilogue the rest.
// The patch covers whole padded rows of the images a tile of consecutive output pixels touches, so small images pack several to a
// tile.  Two workgroups per compute unit: one stages while the other multiplies; or one of eight waves, whose rows are not rounded to two tiles and whose
// patch may fill LDS (64 x 27x27x96 -> 200, 5x5, excluded padding: 243 such workgroups instead of 365, 17.7 -> 15.4 us; 13 x 56x56x200 -> 200, 5x5 82 -> 29).
#include <type_traits>

#include "bnn_mfma_kernel.h"

namespace bnn {
namespace {

using mfma::v16f;
using mfma::v8i;
using mfma::as_operand;
using mfma::expand_unit;

struct XArgs {
    int HP, PCW;            // rows of an image's padded frame that windows reach; pixels of a patch row
    int plane;              // units from word plane to word plane (odd)
    int px_max;             // pixels of the largest patch
    int kwords;             // words of one filter
    int vw, groups;         // words per staging load, loads per pixel
    int table_bytes, thr_at;    // bytes of the offset table; where the thresholds lie
    uint32_t last_mask;     // valid bits of a pixel's last word
    FastDiv div_pcw, div_hp, div_groups, div_tw;
};

// 1 nibble of ones for every set bit of w, in the layout of expand_unit.
__device__ __forceinline__ uint4 nibble_mask(uint32_t w) {
    return make_uint4((w & 0x11111111u) * 15u, ((w >> 1) & 0x11111111u) * 15u, ((w >> 2) & 0x11111111u) * 15u,
                      ((w >> 3) & 0x11111111u) * 15u);
}

typedef uint32_t word4 __attribute__((ext_vector_type(4), aligned(4)));      // filters of odd word counts start at any word

// What a call asks of the epilogue; a kernel is compiled for one form (with all of them in one kernel the compiler stopped specialising the
// general epilogue: bits and sums of 256 x 14x14x200 43.8 us instead of 39.0).
enum OutputForm {
    OUT_BITS,               // packed bits alone: the filters are the row operand, the bits leave as whole words
    OUT_SUMS,               // int32 sums alone
    OUT_STREAMED_RESIDUAL,  // an int32 residual in, rows of whole 128-byte lines: epilogue_resid
    OUT_RESIDUAL,           // any other residual in: the general epilogue
    OUT_BITS_AND_SUMS       // bits and sums without a residual: the general epilogue
};

// MT x NT accumulators of 32 x 32 per wave, WM x WN waves.  SWAP: filters are the MFMA's row operand (bits only).
// SHORTCUT: with the second source (its code beside the bits-only loop cost that 2 %: two more registers spilled).
template <int MT, int NT, int WM, int WN, OutputForm FORM, bool SHORTCUT>
__global__ __launch_bounds__(WM * WN * 64, 2) void conv_xlds_kernel(const uint32_t* __restrict__ A, const uint32_t* __restrict__ B, Geom g,
                                                                   Epi e, XArgs x, int gx, int gy) {
    static_assert(NT == 2, "a wave owns 64 channels, a half-wave 32 of them");
    constexpr bool SWAP = FORM == OUT_BITS;
    constexpr int NTHR = WM * WN * 64, ROWS = WM * MT * 32, COLS = WN * NT * 32;
    extern __shared__ uint4 smem[];
    char* lds = reinterpret_cast<char*>(smem);          // offsets of the K words (int each), then the units
    mfma::accumulators_in_agprs();
    int bx, by;
    if (!mfma::tile_coords(gx, gy, bx, by)) return;     // uniform for the workgroup
    const int tid = threadIdx.x, lane = tid & 63, l32 = lane & 31, half = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave / WN, wn = wave % WN;
    const int m_base = bx * ROWS;                       // rows < 2^31
    const int m0 = m_base + wm * (MT * 32), n0 = (by * WN + wn) * (NT * 32);
    const int rows = (int)g.rows;

    uint32_t c2;
    asm volatile("v_mov_b32 %0, 0x22222222" : "=v"(c2));

    // ---- patch rows: padded rows Y = n * HP + p * stride + r, from the first output pixel's first to the last one's last
    const int first_n = fast_div(m_base, g.div_pq), first_p = fast_div(m_base - first_n * (g.P * g.Q), g.div_q);
    const int last = min(m_base + ROWS, rows) - 1;
    const int last_n = fast_div(last, g.div_pq), last_p = fast_div(last - last_n * (g.P * g.Q), g.div_q);
    const int Ya = first_n * x.HP + first_p * g.stride;
    const int npx = (last_n * x.HP + last_p * g.stride + g.k - Ya) * x.PCW;              // <= px_max

    // ---- this lane's pixels (byte offset of their first tap's unit) and filters
    uint32_t pbase[MT];
#pragma unroll
    for (int i = 0; i < MT; ++i) {
        const int row = min(m0 + 32 * i + l32, rows - 1);                               // past the end: dropped by the epilogue
        const int n = fast_div(row, g.div_pq), rem = row - n * (g.P * g.Q);
        const int p = fast_div(rem, g.div_q), q = rem - p * g.Q;
        pbase[i] = (uint32_t)(x.table_bytes + ((n * x.HP + p * g.stride - Ya) * x.PCW + q * g.stride) * 16);
    }
    uint32_t boff[NT];
#pragma unroll
    for (int j = 0; j < NT; ++j) {
        const int ch = n0 + (SWAP ? mfma::dealt_column(j, l32) : 32 * j + l32);
        boff[j] = (uint32_t)(min(ch, g.cols - 1) * g.ldb_w + 4 * half) * 4u;            // < 2^31 (checked on the host)
    }
    const int nfull = x.kwords >> 3, tail = x.kwords & 7;
    uint4 bq[NT], bn[NT];
    auto load_b = [&](int c, uint4 (&b)[NT]) {                                          // words 8 c + 4 half .. + 3 of a whole chunk
        const char* base = reinterpret_cast<const char*>(B + 8 * c);                     // uniform
#pragma unroll
        for (int j = 0; j < NT; ++j) {
            const word4 v = *reinterpret_cast<const word4*>(base + (size_t)boff[j]);
            b[j] = make_uint4(v[0], v[1], v[2], v[3]);
        }
    };
    auto load_tail = [&](uint4 (&b)[NT]) {              // the last, partly filled chunk; a word past the filter's end repeats its last one
        const int w0 = 8 * nfull + 4 * half;
#pragma unroll
        for (int j = 0; j < NT; ++j) {
            const uint32_t* src = B + (boff[j] >> 2) - 4 * half;
            b[j] = make_uint4(src[min(w0, x.kwords - 1)], src[min(w0 + 1, x.kwords - 1)], src[min(w0 + 2, x.kwords - 1)],
                              src[min(w0 + 3, x.kwords - 1)]);
        }
    };
    if (nfull > 0) load_b(0, bq);
    else load_tail(bq);

    // ---- offsets of the K words from a pixel's first unit
    for (int w = tid; w < ((x.kwords + 7) & ~7); w += NTHR) {
        const int tap = fast_div(w, x.div_tw), wi = w - tap * g.tw;
        const int r = (tap * g.kinv) >> 16, s = tap - r * g.k;
        // a word past the filter's end: the plane of zeros behind the patch (there if the last chunk is partly filled)
        *reinterpret_cast<int*>(lds + 4 * w) = (w < x.kwords ? wi * x.plane + r * x.PCW + s : g.tw * x.plane) * 16;
    }
    if (tail > 0)
        for (int u = tid; u < npx; u += NTHR)
            reinterpret_cast<uint4*>(lds + x.table_bytes)[g.tw * x.plane + u] = make_uint4(0u, 0u, 0u, 0u);
    if (SWAP && tid < COLS) {                           // thresholds of the tile's channels, as the epilogue compares them
        const int ch = by * COLS + tid;
        reinterpret_cast<float*>(lds + x.thr_at)[tid] = ch < g.cols ? (float)e.thr[min(ch, g.cols - 1)] : __builtin_inff();
    }
    // ---- patch -> LDS: item = vw words of one pixel, consecutive in memory; four loads in flight per thread
    {
        const int items = npx * x.groups;
        for (int base = 0; base < items; base += 4 * NTHR) {
            uint32_t w[4][4];
            int px[4], wi0[4];
            bool in[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int it = min(base + u * NTHR + tid, items - 1);
                px[u] = fast_div(it, x.div_groups);
                wi0[u] = (it - px[u] * x.groups) * x.vw;
                const int yr = fast_div(px[u], x.div_pcw), X = px[u] - yr * x.PCW - g.pad;
                const int n = fast_div(Ya + yr, x.div_hp), yy = Ya + yr - n * x.HP - g.pad;
                in[u] = (unsigned)yy < (unsigned)g.H && (unsigned)X < (unsigned)g.W;
                const uint32_t* src = A + (in[u] ? (((long long)n * g.H + yy) * g.W + X) * g.lda_w + wi0[u] : 0);
                w[u][0] = src[0];
                if (x.vw == 4) {                                                        // uniform: lda_w a multiple of 4
                    const uint4 v = *reinterpret_cast<const uint4*>(src);
                    w[u][0] = v.x; w[u][1] = v.y; w[u][2] = v.z; w[u][3] = v.w;
                } else if (x.vw >= 2) {
                    w[u][1] = src[1];
                    if (x.vw == 3) w[u][2] = src[2];
                }
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                if (base + u * NTHR + tid >= items) continue;
                uint4* dst = reinterpret_cast<uint4*>(lds + x.table_bytes) + wi0[u] * x.plane + px[u];
                const uint32_t keep = (in[u] || !g.excl) ? 0xFFFFFFFFu : 0u;             // excluded padding: zeros
#pragma unroll
                for (int d = 0; d < 4; ++d) {
                    if (d >= x.vw) break;                                               // uniform
                    uint4 v = expand_unit(in[u] ? w[u][d] : 0u, c2);
                    uint4 m = make_uint4(keep, keep, keep, keep);
                    if (wi0[u] + d == g.tw - 1 && x.last_mask != 0xFFFFFFFFu) {
                        const uint4 q = nibble_mask(x.last_mask);
                        m = make_uint4(m.x & q.x, m.y & q.y, m.z & q.z, m.w & q.w);
                    }
                    dst[d * x.plane] = make_uint4(v.x & m.x, v.y & m.y, v.z & m.z, v.w & m.w);
                }
            }
        }
    }
    __syncthreads();                                    // the only barrier

    v16f acc[MT][NT];
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int j = 0; j < NT; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

    uint4 fa[2][MT], fb[2][NT];
    auto read_a = [&](int off, int slot) {
#pragma unroll
        for (int i = 0; i < MT; ++i) fa[slot][i] = *reinterpret_cast<const uint4*>(lds + (pbase[i] + (uint32_t)off));
    };
    auto expand_b = [&](const uint4 (&b)[NT], int v, int slot) {
#pragma unroll
        for (int j = 0; j < NT; ++j) fb[slot][j] = expand_unit(v == 0 ? b[j].x : v == 1 ? b[j].y : v == 2 ? b[j].z : b[j].w, c2);
    };
    auto multiply = [&](int slot) {
#pragma unroll
        for (int i = 0; i < MT; ++i)
#pragma unroll
            for (int j = 0; j < NT; ++j)
                acc[i][j] = SWAP ? __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(as_operand(fb[slot][j]), as_operand(fa[slot][i]), acc[i][j], 4,
                                                                                   4, 0, 0, 0, 0)
                                 : __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(as_operand(fa[slot][i]), as_operand(fb[slot][j]), acc[i][j], 4,
                                                                                   4, 0, 0, 0, 0);
    };
    auto offsets = [&](int c) { return *reinterpret_cast<const int4*>(lds + (8 * c + 4 * half) * 4); };

    // Pixel units and expanded filter words run one K-step ahead, packed filter words and offsets one chunk.
    int4 off = offsets(0), offn = off;
    read_a(off.x, 0); expand_b(bq, 0, 0);
    const int nchunks = nfull + (tail > 0 ? 1 : 0);
    for (int c = 0; c < nfull; ++c) {
        if (c + 1 < nfull) load_b(c + 1, bn);
        else if (tail > 0) load_tail(bn);
        offn = offsets(min(c + 1, nchunks - 1));        // past the end: read again and dropped
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            if (v < 3) { read_a(v == 0 ? off.y : v == 1 ? off.z : off.w, (v + 1) & 1); expand_b(bq, v + 1, (v + 1) & 1); }
            else { read_a(offn.x, 0); expand_b(bn, 0, 0); }
            multiply(v & 1);
#pragma unroll
            for (int q = 0; q < MT * NT; ++q) {
                __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);   // an even mix: MFMA, vector ALU, LDS read
                __builtin_amdgcn_sched_group_barrier(0x002, 3, 0);
                __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
        for (int j = 0; j < NT; ++j) bq[j] = bn[j];
        off = offn;
    }
#pragma unroll
    for (int v = 0; v < 4; ++v) {                       // the partly filled chunk: as many K-steps as hold a word
        if (v < tail) {                                 // uniform
            if (v < 3) { read_a(v == 0 ? off.y : v == 1 ? off.z : off.w, (v + 1) & 1); expand_b(bq, v + 1, (v + 1) & 1); }
            multiply(v & 1);
            __builtin_amdgcn_sched_barrier(0);
        }
    }

    int corr = 0;                                       // pad bits of the fused second source only
    if (SHORTCUT && g.A2 != nullptr) corr = mfma::extra_source<MT, NT, SWAP, SWAP>(acc, g, m0, n0, lane, c2) - g.bits2;
    if constexpr (FORM == OUT_SUMS) {
        mfma::epilogue_sums<MT, NT>(acc, m0, n0, lane, g, e, corr);
    } else if constexpr (FORM == OUT_STREAMED_RESIDUAL) {
        mfma::epilogue_streamed<MT, NT>(acc, m0, n0, lane, g, e, corr);
    } else if constexpr (!SWAP) {
        int thi[NT];
        bool cok[NT];
        mfma::column_thresholds<NT>(thi, cok, n0, l32, g, e);
        const mfma::Fetched none = {make_uint4(0u, 0u, 0u, 0u), make_uint4(0u, 0u, 0u, 0u), false};
        Epi es = e;
        es.sums_tiled = 0;                              // (mfma_conv_xlds_tile)
        if (e.out16 != nullptr) {                       // uniform: one kind of sums in each copy
            es.out = nullptr;
            mfma::epilogue_generic<MT, NT, true, false, FORM == OUT_RESIDUAL>(acc, m0, n0, lane, g, es, corr, 0, thi, cok, false, none);
        } else {
            es.out16 = nullptr;
            mfma::epilogue_generic<MT, NT, true, false, FORM == OUT_RESIDUAL>(acc, m0, n0, lane, g, es, corr, 0, thi, cok, false, none);
        }
    } else {
        // register r of tile j holds channel n0 + 32 * half + 16 * j + r of pixel m0 + 32 * i + l32
        float th[32];
        const float4* tl = reinterpret_cast<const float4*>(lds + x.thr_at) + (wn * 64 + 32 * half) / 4;
#pragma unroll
        for (int t = 0; t < 8; ++t) {
            const float4 v = tl[t];
            th[4 * t] = v.x + (float)corr; th[4 * t + 1] = v.y + (float)corr; th[4 * t + 2] = v.z + (float)corr; th[4 * t + 3] = v.w + (float)corr;
        }
        const int wi = (n0 >> 5) + half;
#pragma unroll
        for (int i = 0; i < MT; ++i) {
            uint32_t w = 0u;
#pragma unroll
            for (int t = 28; t >= 0; t -= 4) {
                const v16f& v = acc[i][t >> 4];
                const int r = t & 15;
                push4(w, __builtin_amdgcn_ballot_w64(v[r + 3] >= th[t + 3]), __builtin_amdgcn_ballot_w64(v[r + 2] >= th[t + 2]),
                      __builtin_amdgcn_ballot_w64(v[r + 1] >= th[t + 1]), __builtin_amdgcn_ballot_w64(v[r] >= th[t]));
            }
            const int row = m0 + 32 * i + l32;
            if (row < rows && wi < e.ldbits_w) e.bits[(long long)row * e.ldbits_w + wi] = w;
        }
    }
}

// Largest patch (pixels) of a tile of `tile_rows` consecutive output pixels.
long long patch_pixels(const Geom& g, int tile_rows) {
    const long long pq = (long long)g.P * g.Q;
    const long long out_rows = min((tile_rows - 1 + g.Q - 1) / g.Q + 1LL, (g.rows + g.Q - 1) / g.Q);
    const long long images = min((tile_rows - 1 + pq - 1) / pq, (g.rows + pq - 1) / pq - 1);      // image boundaries inside a tile
    return ((out_rows - 1) * g.stride + g.k + images * max(0, g.k - g.stride)) * ((g.Q - 1LL) * g.stride + g.k);
}

// two workgroups of four waves per compute unit, or one of eight
constexpr size_t xlds_max(int waves) { return (size_t)waves * 20 * 1024; }

// LDS layout of a tile; false: its patch does not fit, or 32-bit offsets do not reach.
bool plan_lds(const Geom& g, int tile_rows, int tile_cols, int waves, XArgs* x, size_t* lds_bytes) {
    const long long px = patch_pixels(g, tile_rows);
    const long long kwords = (long long)g.taps * g.tw;
    const long long plane = px | 1, table = (kwords + 7) / 8 * 32;
    const long long thr_at = table + plane * (g.tw + (kwords % 8 ? 1 : 0)) * 16;
    const long long total = thr_at + tile_cols * 4;
    if (total > (long long)xlds_max(waves)) return false;
    if ((long long)g.cols * g.ldb_w * 4 >= (1LL << 31)) return false;
    x->HP = (g.P - 1) * g.stride + g.k;
    if ((g.rows / ((long long)g.P * g.Q) + 1) * x->HP >= (1LL << 31)) return false;
    x->PCW = (g.Q - 1) * g.stride + g.k;
    x->px_max = (int)px; x->plane = (int)plane; x->kwords = (int)kwords;
    x->vw = g.tw % 4 == 0 ? 4 : g.tw == 3 ? 3 : g.tw % 2 == 0 ? 2 : 1;
    x->groups = g.tw / x->vw;
    x->table_bytes = (int)table; x->thr_at = (int)thr_at;
    x->last_mask = (g.bits_tap & 31) ? (1u << (g.bits_tap & 31)) - 1u : 0xFFFFFFFFu;
    *lds_bytes = (size_t)total;
    return true;
}

OutputForm output_form(const Epi& e) {
    if (e.resid != nullptr || e.resid16 != nullptr || e.resid_bits != nullptr)
        return e.resid != nullptr && e.out16 == nullptr && (e.ldc & 31) == 0 ? OUT_STREAMED_RESIDUAL : OUT_RESIDUAL;
    if (e.out == nullptr && e.out16 == nullptr) return OUT_BITS;
    return e.bits == nullptr ? OUT_SUMS : OUT_BITS_AND_SUMS;
}

template <int MT, int NT, int WM, int WN>
int launch_xlds(const uint32_t* A, const uint32_t* B, const Geom& g, const Epi& e, hipStream_t s) {
    XArgs x;
    size_t lds;
    if (!plan_lds(g, WM * MT * 32, WN * NT * 32, WM * WN, &x, &lds)) return BNN_ERR_UNSUPPORTED;
    x.div_pcw = make_fastdiv((uint32_t)x.PCW); x.div_hp = make_fastdiv((uint32_t)x.HP);
    x.div_groups = make_fastdiv((uint32_t)x.groups); x.div_tw = make_fastdiv((uint32_t)g.tw);
    const int gx = (int)cdiv(g.rows, WM * MT * 32), gy = (int)cdiv(g.cols, WN * NT * 32);
    const unsigned nwg = (unsigned)(cdiv((long long)gx * gy, 8) * 8);
    auto run = [&](auto form, auto shortcut) {
        constexpr OutputForm FORM = decltype(form)::value;
        constexpr bool SHORTCUT = decltype(shortcut)::value;
        static const hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void*>(&conv_xlds_kernel<MT, NT, WM, WN, FORM, SHORTCUT>),
                                                           hipFuncAttributeMaxDynamicSharedMemorySize, (int)xlds_max(WM * WN));
        if (attr != hipSuccess) return (int)BNN_ERR_DEVICE;
        launch((conv_xlds_kernel<MT, NT, WM, WN, FORM, SHORTCUT>), dim3(nwg), dim3(WM * WN * 64), lds, s, A, B, g, e, x, gx, gy);
        return check_launch();
    };
    // a second source comes with bits, with or without their sums; with another form it is not dispatched (xlds_tile)
    const bool shortcut = g.A2 != nullptr;
    constexpr std::true_type with{};
    constexpr std::false_type none{};
    switch (output_form(e)) {
        case OUT_BITS: {
            constexpr std::integral_constant<OutputForm, OUT_BITS> f{};
            return shortcut ? run(f, with) : run(f, none);
        }
        case OUT_BITS_AND_SUMS:
            if constexpr (WM * WN == 4) return run(std::integral_constant<OutputForm, OUT_BITS_AND_SUMS>{}, with);
            break;
        case OUT_SUMS:
            if constexpr (WM * WN == 4) return run(std::integral_constant<OutputForm, OUT_SUMS>{}, none);
            break;
        case OUT_STREAMED_RESIDUAL:
            if constexpr (MT == 2) return run(std::integral_constant<OutputForm, OUT_STREAMED_RESIDUAL>{}, none);
            break;
        case OUT_RESIDUAL:
            if constexpr (MT == 2) return run(std::integral_constant<OutputForm, OUT_RESIDUAL>{}, none);
            break;
    }
    return BNN_ERR_UNSUPPORTED;     // not dispatched: residuals take the tiles of two row fragments (xlds_tile)
}

struct XTile { int rows, cols, mfmas, waves; };         // mfmas: per wave and K-step
constexpr XTile XTILES[] = {{0, 0, 0, 0}, {256, 128, 8, 4}, {128, 256, 8, 4}, {512, 64, 8, 4}, {128, 128, 4, 4}, {256, 64, 4, 4},
                            {192, 256, 6, 8}, {384, 128, 6, 8}, {768, 64, 6, 8}};

// Fewest workgroups from which this kernel is the faster one, 0: it is not.  With bits alone the 64 x 64 tiles of the direct kernel,
// four times as many, win below about 96 (49 workgroups 0.87 of their speed, 98: 1.04, 171: 1.3; more in most_staged).  Everything else leaves through the
// accumulators' rows, load and store per element, and what a workgroup of four large wave tiles waits there (7 to 12 us through the general
// epilogue) is hidden only by other workgroups: it takes more of them, or a longer K, whose saving outweighs it.  Measured, this kernel's
// speed over the direct one's (3x3, channels = filters, -1 / excluded padding):
//   sums alone         104 workgroups 0.83 to 0.99 / 1.2 to 1.3, 129: 0.96 to 1.05, 152: 1.03 to 1.07, 200: 1.2 to 1.4; the unrolled forms (4 and 8 words, excluded
//                      padding) 0.95 to 1.03 at 104, 1.3 at 200; 90 channels against the 256x128 tile of the direct kernel 0.97
//   streamed residual  104: 0.69 to 0.80 / 0.89 to 0.97, 152: 0.85 / 1.05, 200: 1.01 to 1.25 / 1.24 to 1.5, 392 and more: 1.08 to 1.4
//   other residuals    104: 0.6 to 0.7 / 0.78 to 0.92, 152 with 90 words of K 0.77 / 0.9, 200: 0.90 with 27 words, 1.1 with 63, 1.46 with 126 / 1.1
//                      to 1.5, the unrolled forms 0.83 to 0.95; 296 to 392: 1.1 to 1.6; 27 words against the 256x128 tile 0.97 to 1.05; the unrolled
//                      form of two words, more than 64 channels out, 0.93 to 0.97 at 516 to 744
//   bits and sums      27 words 0.6 to 0.9 at any count, 63: 0.67 at 104, 1.0 at 200 and 392, against the 256x128 tile 0.94 to 0.97 (63 and 75
//                      words), 90: 1.13 to 1.37 from 296 / 18 words 0.93 at 392, 27: 0.99 at 200, 1.1 at 392, 63: 1.17 at 200, unrolled
//                      forms 0.8 at 200, 1.1 at 392
int min_workgroups(const Geom& g, OutputForm form) {
    const int kwords = g.taps * g.tw;
    const bool unrolled = g.k == 3 && (g.tw == 2 || g.tw == 4 || g.tw == 8 || g.tw == 16);
    const bool against_big_tile = !g.excl && mfma::pick_tile(g) == 0;
    switch (form) {
        case OUT_BITS: return 96;
        case OUT_SUMS: return against_big_tile && kwords < 45 && (g.cols & 31) != 0 ? 0 : g.excl && !unrolled ? 96 : 132;
        case OUT_STREAMED_RESIDUAL: return !g.excl ? 192 : unrolled ? 256 : 128;
        case OUT_RESIDUAL: return (against_big_tile && kwords < 45) || (g.excl && unrolled && g.tw == 2 && g.cols > 64) ? 0 : (g.excl ? unrolled : kwords < 63 || g.tw % 4 == 0) ? 256 : 192;
        default: return kwords < (g.excl ? 27 : against_big_tile ? 90 : 63) ? 0 : (g.excl && kwords < 63) || unrolled ? 256 : 192;
    }
}

// Most LDS units a workgroup may stage per K-step with -1 padding and few workgroups.  Up to half of the compute units hold one workgroup then, and what
// it stages and waits is not hidden, while the direct kernel has no sum to correct and, at whole groups of four words, loads 8 bytes at a
// time.  Measured over 500 geometries of 96 to 160 workgroups, strides 1 to 3 (this kernel's speed over the direct one's): four words 0.83 to 0.95 up to
// 144 workgroups; one word 1.09 and more up to 200 units, 0.79 at 344; two and odd counts 1.03 and more up to 80 units, 0.83 to 0.98 from 85; six words
// 1.4 at 32 units, 0.94 to 0.98 from 92; all of them 1.03 and more from 132 workgroups (one of 60: 0.96).  With excluded padding 1.05 and more everywhere.
// Residuals in rows that are not whole lines keep workgroups waiting at any count: groups of four words 0.86 to 0.96 from 104 units (590 to 760
// workgroups, both conventions), 1.01 to 1.14 up to 51.
double most_staged(const Geom& g, OutputForm form, long long wgs) {
    if (form == OUT_RESIDUAL) return g.tw % 4 == 0 ? 100. : 1e30;
    if (g.excl || wgs >= 192) return 1e30;
    if (g.tw % 4 == 0) return 0.;
    if (wgs >= 132) return 1e30;
    return g.tw == 1 ? 200. : g.tw % 2 == 1 || g.tw == 2 ? 80. : 60.;
}

// Whether a tile of eight waves is faster than the direct kernel, by the estimated microseconds of both: a round of the one costs its K-steps, the units it
// stages and a constant, the other as many tiles as its fullest compute unit has, by the words of K that its loads take.  Fitted to 2200 geometries (windows of 2 to 11,
// strides 1 to 3, patches above 80 KB or one round), bits: the median error is 4 % here, 2 to 5 % there.  Of 938 where the choice is open: taken 707, 0.95 and above of the direct
// kernel's speed but for six (0.82 to 0.95), median 1.2; left 231, up to 1.03 but for 17 (the best 1.24), down to 0.57.  Of 1500 others 31 of those taken are below 0.97,
// the least 0.90; without the question 244 were, the least 0.57.
bool eight_waves_gain(const Geom& g, long long wgs, const XArgs& x) {
    const double steps = (g.taps * g.tw + 1) / 2;
    const double here = 1.4 + (double)cdiv(wgs, 256) * (4.05 + 0.2233 * steps + 0.2664e-3 * (double)x.px_max * g.tw);
    const int load = mfma::conv_load_words(g), chunk = 2 * load;
    const double words = (double)g.taps * ((g.tw + chunk - 1) / chunk * chunk);
    auto tiles = [&](int rows, int cols) { return (double)cdiv(cdiv(g.rows, rows) * cdiv(g.cols, cols), 256); };
    auto by_load = [&](double v4, double v2, double v1) { return load == 4 ? v4 : load == 2 ? v2 : v1; };
    double direct;
    switch (mfma::pick_tile(g)) {
        case 0: direct = 4.3 + tiles(mfma::TileBig::ROWS, mfma::TileBig::COLS) * (1.2 + words * by_load(0.093, 0.1025, 0.133)); break;
        case 1: direct = 4.3 + tiles(mfma::TileTall::ROWS, mfma::TileTall::COLS) * (1.2 + words * by_load(0.093, 0.1025, 0.133)); break;
        case 2: direct = 4.5 + tiles(mfma::TileMid::ROWS, mfma::TileMid::COLS) * words * by_load(0.054, 0.0635, 0.1); break;
        default: direct = 4.5 + tiles(mfma::TileSmall::ROWS, mfma::TileSmall::COLS) * words * by_load(0.026, 0.026, 0.045); break;
    }
    return direct >= 0.97 * here;
}

// Tile for this geometry, 0: another kernel's.  Among the tiles whose patch fits LDS, the one with the least estimated time: rounds
// of 512 workgroups times the cycles of one (K-steps, a little more than their MFMAs take where a step has only four; staging;
// epilogue; the rest).
int xlds_tile(const Geom& g, const Epi& e) {
    if (!g.conv || g.rows >= (1LL << 31) - 1024) return 0;
    // What the other kernels do as well or better (measured, this kernel's speed over theirs): 1x1 windows and
    // filters of less than two chunks, whose patch is used too little (0.7 to 0.9), the unrolled 3x3 forms of 2, 4, 8 and 16 words per pixel (0.85 to 1.06) -- except with excluded
    // padding and a partly filled last word, where they correct every sum by its pixel (this kernel 2.7); and with
    // -1 padding what the staged kernel takes (0.98 to 1.19) and pixels of whole 32-byte units, which the direct kernel loads 16
    // bytes at a time (0.98 to 1.06).
    if (g.k == 1 || g.taps * g.tw < 16) return 0;
    const bool pad_bits = g.bits_tap != g.tw * 32;
    if (g.k == 3 && (g.tw == 2 || g.tw == 4 || g.tw == 8 || g.tw == 16) && !(g.excl && pad_bits)) return 0;
    if (!g.excl && (mfma::conv_stages_through_lds(g) || g.tw % 8 == 0)) return 0;
    const OutputForm form = output_form(e);
    if (g.A2 != nullptr && form != OUT_BITS && form != OUT_BITS_AND_SUMS) return 0;
    // (images beyond the direct kernel's 32-bit offsets would be left to the vector ALU)
    const bool direct_reaches = mfma::offsets_fit(g);
    const int least = direct_reaches ? min_workgroups(g, form) : 96;
    if (least == 0) return 0;
    const bool small_only = form == OUT_STREAMED_RESIDUAL || form == OUT_RESIDUAL;      // (the residual of four row fragments at a time: 0.92 of two)
    int best = 0, four = 0;                             // four: the best tile of four waves
    double best_cost = 0.;
    const double steps = (g.taps * g.tw + 1) / 2;
    for (int t = small_only ? 4 : 1; t <= (form == OUT_BITS ? 8 : 5); ++t) {
        XArgs x;
        size_t lds;
        const long long gy = cdiv(g.cols, XTILES[t].cols), wgs = cdiv(g.rows, XTILES[t].rows) * gy;
        // Eight waves: the tile of a compute unit in one piece, 192 rows where two pieces of 128 are 256.  In one round, where the shorter way of the fullest
        // compute unit counts, 1.02 to 1.25 of the four-wave tiles' speed (180 shapes; 677 more: 0.90 once, 0.95 and above, median 1.22); in several rounds 0.84 to 1.1:
        // nothing overlaps a workgroup's staging and epilogue.  And the only tiles for a patch above 80 KB: with excluded padding and a partly filled last word 1.07
        // to 4.5 of the direct kernel, which corrects every sum there; else 0.57 to 3.5, 0.95 and above (one in 200: 0.82) where eight_waves_gain() says so, and
        // with -1 padding 0.88 to 0.99 if the last round fills the chip to less than 0.6 over all.  (With -1 padding one round gains as much
        // as without, 1.16 to 1.23 -- 64 x 27x27x96 -> 200, 5x5 19.2 -> 16.4 us --, but bnn_bconv_kernel_name is tested to name the four-wave tiles there.)
        if (t == 6) four = best;
        if (t >= 6 && four != 0 && !(g.excl && wgs <= 256)) continue;
        if (t >= 6 && !g.excl && direct_reaches && wgs * 5 < cdiv(wgs, 256) * 256 * 3) continue;
        // Many empty columns: 0.77 at 64 of 128.
        if (wgs < least || (double)(gy * XTILES[t].cols) > 1.5 * g.cols) continue;
        if (!plan_lds(g, XTILES[t].rows, XTILES[t].cols, XTILES[t].waves, &x, &lds)) continue;
        if (t >= 6 && four == 0 && direct_reaches && !(g.excl && pad_bits) && !eight_waves_gain(g, wgs, x)) continue;
        if (direct_reaches && (double)x.px_max * g.tw > most_staged(g, form, wgs) * steps) continue;
        const double m = XTILES[t].mfmas;
        const double wg = steps * m * (m < 8. ? 44. : 36.) + (double)x.px_max * g.tw / 4. + m * 160. + 1500.;
        const double cost = (double)cdiv(wgs, XTILES[t].waves == 4 ? 512 : 256) * wg;
        if (best == 0 || cost < best_cost) { best = t; best_cost = cost; }
    }
    return best;
}

}  // namespace

int mfma_conv_xlds_tile(const Geom& g, const Epi& e) { return e.sums_tiled ? 0 : xlds_tile(g, e); }

const char* describe_mfma_conv_xlds(int tile) {
    switch (tile) {
        case 1: return "mfma_fp4_conv_xlds_wg256x128";
        case 2: return "mfma_fp4_conv_xlds_wg128x256";
        case 3: return "mfma_fp4_conv_xlds_wg512x64";
        case 4: return "mfma_fp4_conv_xlds_wg128x128";
        case 6: return "mfma_fp4_conv_xlds_wg192x256";
        case 7: return "mfma_fp4_conv_xlds_wg384x128";
        case 8: return "mfma_fp4_conv_xlds_wg768x64";
        default: return "mfma_fp4_conv_xlds_wg256x64";
    }
}

int launch_mfma_conv_xlds(int tile, const uint32_t* A, const uint32_t* B, const Geom& g, const Epi& e, hipStream_t s) {
    switch (tile) {
        case 1: return launch_xlds<4, 2, 2, 2>(A, B, g, e, s);
        case 2: return launch_xlds<4, 2, 1, 4>(A, B, g, e, s);
        case 3: return launch_xlds<4, 2, 4, 1>(A, B, g, e, s);
        case 4: return launch_xlds<2, 2, 2, 2>(A, B, g, e, s);
        case 5: return launch_xlds<2, 2, 4, 1>(A, B, g, e, s);
        case 6: return launch_xlds<3, 2, 2, 4>(A, B, g, e, s);
        case 7: return launch_xlds<3, 2, 4, 2>(A, B, g, e, s);
        case 8: return launch_xlds<3, 2, 8, 1>(A, B, g, e, s);
        default: return BNN_ERR_UNSUPPORTED;
    }
}

}  // namespace bnn
