// Matrix products on bits that mean 0 or 1: both operands travel through LDS packed, every wave makes its own MFMA operands with one vector
// instruction per register.
//
// Why 0 and 1.  As +1 / -1 a packed word costs seven instructions (three shifts, four and-or) for the four registers of its operand, and on random bits
// what toggles costs clock: register-resident MFMAs run at 8.3 to 8.5 PFLOP/s on random signs, at 9.4 to 9.8 on random {0, 1}, and the kernel that
// expanded signs (the row operand once per workgroup, into LDS) needed 1424 us for 16384^3 on random bits, 1088 on zeros.  So the products counted
// here are those of set bits: four packed words w0 .. w3 of a row serve four K-steps, and K-step v takes bit v of every nibble of all four, left where it stands --
// four ANDs -- as an E2M1 value (0.5, 1 or 2; bit 3 is moved to bit 2's place).  Both operands hold the same bits of the same words, a
// product of two set bits is 0.25, 1, 4 or 4, and the instruction's block scale, a constant of the K-step, makes it 4.  With s = 2 b - 1
//     sum of s_a s_b  =  4 #(both set)  -  2 #(set in a)  -  2 #(set in b)  +  K:
// the loader threads count the set bits of their part of a row as they store it, and the epilogue adds two numbers to each sum.  Bits past K are zero in both
// operands and count nothing.  All exact: multiples of 2 below 2^23 (K <= 2^20).
//
// Both operands packed in LDS: a quarter of the bytes written to and read from LDS (the expanded form was at 53 % of its bandwidth), which leaves
// room for slabs of 512 bits -- four lanes of a load cover 64 neighbouring bytes of a row, half as many lines per instruction as with 256 -- and one
// barrier for eight K-steps.
//
// Measured, us, the kernel that expanded into LDS -> this one: bits of 16384^3 1414 -> 1195 (7.4 P binary op/s), of 8192^3 182 -> 160, of 4096^3 24.8 -> 23.0, of
// 4096x4096x2048 14.1 -> 14.0 (x1024 9.5 -> 10.0: left to that kernel, bnn_mfma_signs.hip); sums of 8192^3 197 -> 182.  On the way, 16384^3: signs as {0, 1} with the row operand still expanded in LDS 1336, both packed 1275, operands
// made one row tile ahead of their MFMAs with an even mix of instructions 1228, no masks where K is whole slabs (FULL) 1219.  Tried: four waves of 128 x 128 (one per
// SIMD, 256 accumulators) 1234, and slower below (4096^3 25.5).
#ifndef BNN_MFMA_BITS_H
#define BNN_MFMA_BITS_H

#include <type_traits>

#include "bnn_mfma_kernel.h"

namespace bnn {
namespace mfma {

// Tile of WM x WN waves, each MT x NT accumulators of 32 x 32; MINW waves per SIMD that the registers are meant for.
template <int MT_, int NT_, int WM_, int WN_, int MINW_>
struct BitsTile {
    static constexpr int MT = MT_, NT = NT_, WM = WM_, WN = WN_, MINW = MINW_;
    static constexpr int ROWS = WM_ * MT_ * 32, COLS = WN_ * NT_ * 32, THREADS = WM_ * WN_ * 64;
    // units between granules: the rows that whole passes of the loader cover, and 2 (its writes, four granules of 16 rows, hit distinct banks)
    static constexpr int RA = (ROWS * 4 + THREADS - 1) / THREADS * (THREADS / 4) + 2, RB = (COLS * 4 + THREADS - 1) / THREADS * (THREADS / 4) + 2;
    static constexpr size_t LDS_BYTES = (size_t)2 * 4 * (RA + RB) * 16 + (RA + RB) * 4;
};

// FULL: K is whole slabs, no word is masked; else the last slab may end early and its second half be left out.
// PANELS: both operands (and the packed output, if there is one) are in the K-panel layout of bnn.h: panel p holds words 8 p .. 8 p + 7 of
// every row back to back, so that a load covers contiguous memory.
template <class TL, bool FULL, bool PANELS>
__global__ __launch_bounds__(TL::THREADS, TL::MINW) void mfma_bits_kernel(const uint32_t* __restrict__ A, const uint32_t* __restrict__ B,
                                                                        Geom g, Epi e, int gx, int gy) {
    constexpr int MT = TL::MT, NT = TL::NT, ROWS = TL::ROWS, COLS = TL::COLS, NTHR = TL::THREADS;
    constexpr int LA = (ROWS * 4 + NTHR - 1) / NTHR, LB = (COLS * 4 + NTHR - 1) / NTHR;     // granules each thread moves per slab
    constexpr int RA = TL::RA, RB = TL::RB;              // padded row counts, in 16-byte units
    constexpr int STAGE = 4 * (RA + RB);                 // units per slab of 512 bits: [granule 0..3][row]
    extern __shared__ uint4 lds[];                       // 2 * STAGE units, ROWS + COLS floats
    if constexpr (TL::MINW <= 2) accumulators_in_agprs();
    int bx, by;
    if (!tile_coords(gx, gy, bx, by)) return;
    const int tid = threadIdx.x;
    const int lane = tid & 63, l32 = lane & 31, half = lane >> 5, wave = tid >> 6;
    const int wm = wave / TL::WN, wn = wave % TL::WN;
    const long long m_base = (long long)bx * ROWS;
    const int n_base = by * COLS;

    // ---- loader: thread -> granule g4 of rows r4 + (NTHR / 4) * q: four lanes cover 64 neighbouring bytes of a row
    const int g4 = tid & 3, r4 = tid >> 2;
    const int kwords = g.tw, nchunks = (kwords + 7) / 8, nslabs = (nchunks + 1) / 2;
    const int b_first = min(n_base, g.cols - 1);         // (a tile of output words past the last column)
    const int a_pitch = PANELS ? 8 : g.lda_w, b_pitch = PANELS ? 8 : g.ldb_w;
    const char* a_base = reinterpret_cast<const char*>(A + m_base * a_pitch);                  // uniform
    const char* b_base = reinterpret_cast<const char*>(B + (long long)b_first * b_pitch);
    uint32_t arow[LA], brow[LB];                         // byte offset of a thread's rows from there (bits_fit); rows past the matrix repeat its last one
#pragma unroll
    for (int q = 0; q < LA; ++q) arow[q] = 4u * (uint32_t)((int)min((long long)min(r4 + (NTHR / 4) * q, ROWS - 1), g.rows - 1 - m_base) * a_pitch);
#pragma unroll
    for (int q = 0; q < LB; ++q) brow[q] = 4u * (uint32_t)(min(min(r4 + (NTHR / 4) * q, COLS - 1), g.cols - 1 - b_first) * b_pitch);
    uint4 sa[LA], sb[LB];
    int set_a[LA], set_b[LB];
#pragma unroll
    for (int q = 0; q < LA; ++q) set_a[q] = 0;
#pragma unroll
    for (int q = 0; q < LB; ++q) set_b[q] = 0;
    // a granule past the end of K reads the last one instead: a valid address, cleared by the store
    auto word_bytes = [&](int s, long long rows) {
        const int w = min(s * 16 + g4 * 4, kwords - 4);
        if constexpr (PANELS) return (size_t)(w >> 3) * (size_t)rows * 32 + (w & 4) * 4;
        else return (uint32_t)(4 * w);
    };
    auto load_a = [&](int s, int q) { sa[q] = *reinterpret_cast<const uint4*>(a_base + (size_t)(arow[q] + word_bytes(s, g.rows))); };
    auto load_b = [&](int s, int q) { sb[q] = *reinterpret_cast<const uint4*>(b_base + (size_t)(brow[q] + word_bytes(s, g.cols))); };
    auto store = [&](uint4* to, const uint4& v, int s, int& set) {
        const uint32_t keep = FULL || s * 16 + g4 * 4 < kwords ? 0xFFFFFFFFu : 0u;
        const uint4 w = make_uint4(v.x & keep, v.y & keep, v.z & keep, v.w & keep);
        *to = w;
        set += __popc(w.x) + __popc(w.y) + __popc(w.z) + __popc(w.w);
    };
    auto store_a = [&](int buf, int s, int q) { store(lds + buf * STAGE + g4 * RA + r4 + (NTHR / 4) * q, sa[q], s, set_a[q]); };
    auto store_b = [&](int buf, int s, int q) { store(lds + buf * STAGE + 4 * RA + g4 * RB + r4 + (NTHR / 4) * q, sb[q], s, set_b[q]); };

    v16f acc[MT][NT];
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int j = 0; j < NT; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

    // ---- fragments: four packed words of a row (pa, pb) serve four K-steps; K-step v multiplies their bits 4 n + v.  Operands
    // are made one row tile (A) and one K-step (B) ahead of the MFMAs that take them.
    uint4 pa[MT], pb[NT], ea[2], eb[2][NT];
    const int a_unit = half * RA + wm * (MT * 32) + l32, b_unit = 4 * RA + half * RB + wn * (NT * 32) + l32;
    auto read_a = [&](int buf, int c, int i) { pa[i] = lds[buf * STAGE + a_unit + 2 * c * RA + 32 * i]; };
    auto read_b = [&](int buf, int c, int j) { pb[j] = lds[buf * STAGE + b_unit + 2 * c * RB + 32 * j]; };
    auto expand_b = [&](auto v_tag, int j) { constexpr int v = decltype(v_tag)::value; eb[v & 1][j] = bit_unit<v>(pb[j]); };
    auto expand_a = [&](auto v_tag, int i, int slot) { constexpr int v = decltype(v_tag)::value; ea[slot] = bit_unit<v>(pa[i]); };
    // Chunk c (256 bits) of slab s, and on the way: the next slab (in sa / sb) is stored and the registers are requested anew (c = 0), the words of the next
    // chunk are read as soon as this one's are used up.  The ONE barrier of a slab stands in chunk 1, ahead of the first read of the next slab: by then every
    // wave has stored its share of it, in chunk 0, and has read the last words of the buffer that chunk 0 of the next slab will store to.
    // The same program for every slab, the last one too (it stores and reads what nobody uses; its loads repeat valid addresses): with a form of its own for the end the
    // compiler moved accumulators through 600 spilled registers.
    auto chunk = [&](int s, auto c_tag) {
        constexpr int c = decltype(c_tag)::value;
        const int buf = s & 1, next = c == 0 ? buf : buf ^ 1;
        static_for<4 * MT>([&](auto t_tag) {
            constexpr int t = decltype(t_tag)::value, v = t / MT, i = t % MT, half_steps = MT / 2;
            constexpr int vn = (v + 1) & 3, jn = (NT + half_steps - 1) / half_steps;         // B operands of the next K-step: made in the first half of this one
            if constexpr (v == 3) read_a(next, c ^ 1, i);
            expand_a(std::integral_constant<int, ((t + 1) / MT) & 3>{}, (t + 1) % MT, (t + 1) & 1);
            if constexpr (v < 3 && i < half_steps)
#pragma unroll
                for (int j = i * jn; j < (i + 1) * jn && j < NT; ++j) expand_b(std::integral_constant<int, vn>{}, j);
            if constexpr (v == 3 && i >= half_steps)
#pragma unroll
                for (int j = (i - half_steps) * jn; j < (i - half_steps + 1) * jn && j < NT; ++j) expand_b(std::integral_constant<int, vn>{}, j);
            if constexpr (v == 2 && i == half_steps) {
                if constexpr (c == 1) __syncthreads();
#pragma unroll
                for (int j = 0; j < NT; ++j) read_b(next, c ^ 1, j);
            }
            if constexpr (c == 0 && t < LA) { store_a(buf ^ 1, s + 1, t); load_a(min(s + 2, nslabs - 1), t); }
            if constexpr (c == 0 && t >= 4 && t < 4 + LB) { store_b(buf ^ 1, s + 1, t - 4); load_b(min(s + 2, nslabs - 1), t - 4); }
#pragma unroll
            for (int j = 0; j < NT; ++j)
                acc[i][j] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(as_operand(ea[t & 1]), as_operand(eb[v & 1][j]), acc[i][j], 4, 4, 0,
                                                                            scale_of_bit(v), 0, 127);
#pragma unroll
            for (int q = 0; q < NT; ++q) {               // an even mix: MFMA, vector ALU, LDS
                __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                __builtin_amdgcn_sched_group_barrier(0x002, 4, 0);
                __builtin_amdgcn_sched_group_barrier(0x080, 1, 0);
            }
            __builtin_amdgcn_sched_barrier(0);
        });
    };
    std::integral_constant<int, 0> c0;
    std::integral_constant<int, 1> c1;

#pragma unroll
    for (int q = 0; q < LA; ++q) load_a(0, q);
#pragma unroll
    for (int q = 0; q < LB; ++q) load_b(0, q);
#pragma unroll
    for (int q = 0; q < LA; ++q) { store_a(0, 0, q); load_a(min(1, nslabs - 1), q); }
#pragma unroll
    for (int q = 0; q < LB; ++q) { store_b(0, 0, q); load_b(min(1, nslabs - 1), q); }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < NT; ++j) { read_b(0, 0, j); expand_b(c0, j); }
#pragma unroll
    for (int i = 0; i < MT; ++i) read_a(0, 0, i);
    expand_a(c0, 0, 0);
    int s = 0;
    do {
        chunk(s, c0);
        if (FULL || 2 * s + 1 != nchunks) chunk(s, c1);  // (a break here: 98 spilled registers)
    } while (++s < nslabs);

    // whole accumulators up to here: the compiler took them apart, for the epilogue, at the end of every pass of the loop (88 spilled registers)
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int j = 0; j < NT; ++j) {
            if constexpr (TL::MINW <= 2) asm volatile("" : "+a"(acc[i][j]));
            else asm volatile("" : "+v"(acc[i][j]));
        }
    // ---- 4 x (positions where both bits are set) - 2 x set bits of the row - 2 x set bits of the column = sum - K
    float* set_lds = reinterpret_cast<float*>(lds + 2 * STAGE);         // [RA], [RB]
    auto quad_sum = [](int v) {
        v += __builtin_amdgcn_update_dpp(0, v, 0xB1, 0xF, 0xF, true);   // quad_perm 1 0 3 2
        return v + __builtin_amdgcn_update_dpp(0, v, 0x4E, 0xF, 0xF, true);   // quad_perm 2 3 0 1
    };
#pragma unroll
    for (int q = 0; q < LA; ++q) {
        if (FULL) set_a[q] -= __popc(sa[q].x) + __popc(sa[q].y) + __popc(sa[q].z) + __popc(sa[q].w);     // the last slab was stored twice
        const int n = quad_sum(set_a[q]);
        if (g4 == 0) set_lds[r4 + (NTHR / 4) * q] = -2.f * (float)n;
    }
#pragma unroll
    for (int q = 0; q < LB; ++q) {
        if (FULL) set_b[q] -= __popc(sb[q].x) + __popc(sb[q].y) + __popc(sb[q].z) + __popc(sb[q].w);
        const int n = quad_sum(set_b[q]);
        if (g4 == 0) set_lds[RA + r4 + (NTHR / 4) * q] = -2.f * (float)n;
    }
    __syncthreads();
    float col_set[NT];
#pragma unroll
    for (int j = 0; j < NT; ++j) col_set[j] = set_lds[RA + wn * (NT * 32) + 32 * j + l32];
    const float* row_lds = set_lds + wm * (MT * 32) + 4 * half;
    auto subtract_set = [&](int i, auto columns) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const float4 row_set = *reinterpret_cast<const float4*>(row_lds + 32 * i + 8 * q);
            const float rs[4] = {row_set.x, row_set.y, row_set.z, row_set.w};
#pragma unroll
            for (int j = 0; j < NT; ++j)
#pragma unroll
                for (int r = 0; r < 4; ++r) acc[i][j][4 * q + r] += decltype(columns)::value ? rs[r] + col_set[j] : rs[r];
        }
    };
    const long long m0 = m_base + (long long)wm * (MT * 32);
    const int n0 = n_base + wn * (NT * 32);
    if (e.bits != nullptr) {                             // uniform
        int thi[NT];
        bool cok[NT];
        column_thresholds<NT>(thi, cok, n0, l32, g, e);
        // the column's count goes to the threshold instead: one addition to a sum (4096 x 4096 bits out, K = 1024 10.3 -> 10.0 us, 4096 23.3 -> 23.0)
        epilogue_bits<MT, NT, PANELS>(acc, m0, n0, lane, g, e, -g.bits_tap, thi, cok, [&](int i) { subtract_set(i, std::false_type{}); }, col_set);
    } else {
        epilogue_sums<MT, NT>(acc, m0, n0, lane, g, e, -g.bits_tap, [&](int i) { subtract_set(i, std::true_type{}); });
    }
}

// The same for products of few tiles and long K, which are a chain of waits: the workgroup's waves are WK groups, each taking its own 256 bits of every slab of
// 256 * WK, and their partial sums meet in LDS.  What bounded such products in the direct kernel (64 x 64 tiles, operands straight from memory) was the address
// side of its loads, a cycle for nearly every lane when each reads another row: 8 loads a chunk and workgroup, about 500 cycles beside 128 of MFMAs.  Here eight or
// sixteen lanes of a load cover 128 or 256 neighbouring bytes, each row is loaded once, and two slabs are in flight.  Measured (graph replays, bits / int32):
// 160x504x8310 9.8 -> 5.3 us (32 x 32 tiles), 152x211x14254 15.4 -> 6.0, 1386x246x11885 13.2 -> 8.3, 4673x40x6064 7.8 -> 6.5 (64 x 64 tiles).
template <int MT_, int NT_, int WM_, int WN_, int WK_, int MINW_>
struct KsplitTile {
    static constexpr int MT = MT_, NT = NT_, WM = WM_, WN = WN_, WK = WK_, MINW = MINW_;
    static constexpr int ROWS = WM_ * MT_ * 32, COLS = WN_ * NT_ * 32, THREADS = WM_ * WN_ * WK_ * 64;
    static constexpr int RA = ROWS + 4, RB = COLS + 4;
    static constexpr size_t SLABS = (size_t)2 * 2 * WK_ * (RA + RB) * 16, PARTS = (size_t)WK_ * ROWS * COLS * 4;
    static constexpr size_t SET_AT = (SLABS > PARTS ? SLABS : PARTS) / 16, LDS_BYTES = SET_AT * 16 + (RA + RB) * 4;
};

template <class TL>
__global__ __launch_bounds__(TL::THREADS, TL::MINW) void mfma_ksplit_kernel(const uint32_t* __restrict__ A, const uint32_t* __restrict__ B,
                                                                          Geom g, Epi e, int gx, int gy) {
    constexpr int MT = TL::MT, NT = TL::NT, WN = TL::WN, WK = TL::WK, ROWS = TL::ROWS, COLS = TL::COLS, NTHR = TL::THREADS;
    constexpr int GR = 2 * WK;                           // granules of 16 bytes of a row and slab (256 * WK bits)
    constexpr int RA = TL::RA, RB = TL::RB, STAGE = GR * (RA + RB);
    constexpr int LA = ROWS * GR / NTHR, LB = COLS * GR / NTHR, RSTEP = NTHR / GR;
    static_assert(LA >= 1 && LB >= 1 && LA * NTHR == ROWS * GR && LB * NTHR == COLS * GR && (GR == 4 || GR == 8 || GR == 16), "whole granules per thread");
    extern __shared__ uint4 lds[];
    int bx, by;
    if (!tile_coords(gx, gy, bx, by)) return;
    const int tid = threadIdx.x;
    const int lane = tid & 63, l32 = lane & 31, half = lane >> 5, wave = tid >> 6;
    const int kg = wave / (TL::WM * WN), wt = wave % (TL::WM * WN), wm = wt / WN, wn = wt % WN;
    const long long m_base = (long long)bx * ROWS;
    const int n_base = by * COLS;
    const int gr = tid % GR, r0 = tid / GR;
    const int kwords = g.tw, nslabs = (kwords + 8 * WK - 1) / (8 * WK);
    const char* a_base = reinterpret_cast<const char*>(A + m_base * g.lda_w);
    const int b_first = min(n_base, g.cols - 1);
    const char* b_base = reinterpret_cast<const char*>(B + (long long)b_first * g.ldb_w);
    uint32_t arow[LA], brow[LB];
#pragma unroll
    for (int q = 0; q < LA; ++q) arow[q] = 4u * (uint32_t)((int)min((long long)(r0 + RSTEP * q), g.rows - 1 - m_base) * g.lda_w);
#pragma unroll
    for (int q = 0; q < LB; ++q) brow[q] = 4u * (uint32_t)(min(r0 + RSTEP * q, g.cols - 1 - b_first) * g.ldb_w);
    uint4 sa[2][LA], sb[2][LB];
    int set_a[LA], set_b[LB];
#pragma unroll
    for (int q = 0; q < LA; ++q) set_a[q] = 0;
#pragma unroll
    for (int q = 0; q < LB; ++q) set_b[q] = 0;
    auto load = [&](int set, int s) {
        const uint32_t w = 4u * (uint32_t)min(s * (8 * WK) + gr * 4, kwords - 4);
#pragma unroll
        for (int q = 0; q < LA; ++q) sa[set][q] = *reinterpret_cast<const uint4*>(a_base + (size_t)(arow[q] + w));
#pragma unroll
        for (int q = 0; q < LB; ++q) sb[set][q] = *reinterpret_cast<const uint4*>(b_base + (size_t)(brow[q] + w));
    };
    auto store1 = [&](uint4* to, const uint4& v, int s, int& set) {
        const uint32_t keep = s * (8 * WK) + gr * 4 < kwords ? 0xFFFFFFFFu : 0u;
        const uint4 w = make_uint4(v.x & keep, v.y & keep, v.z & keep, v.w & keep);
        *to = w;
        set += __popc(w.x) + __popc(w.y) + __popc(w.z) + __popc(w.w);
    };
    auto store = [&](int buf, int set, int s) {
#pragma unroll
        for (int q = 0; q < LA; ++q) store1(lds + buf * STAGE + gr * RA + r0 + RSTEP * q, sa[set][q], s, set_a[q]);
#pragma unroll
        for (int q = 0; q < LB; ++q) store1(lds + buf * STAGE + GR * RA + gr * RB + r0 + RSTEP * q, sb[set][q], s, set_b[q]);
    };
    v16f acc[MT][NT];
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int j = 0; j < NT; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;
    uint4 pa[MT], pb[NT], ea[2], eb[2][NT];
    const int a_unit = (2 * kg + half) * RA + wm * (MT * 32) + l32, b_unit = GR * RA + (2 * kg + half) * RB + wn * (NT * 32) + l32;
    auto read_a = [&](int buf, int i) { pa[i] = lds[buf * STAGE + a_unit + 32 * i]; };
    auto read_b = [&](int buf, int j) { pb[j] = lds[buf * STAGE + b_unit + 32 * j]; };
    auto expand_b = [&](auto v_tag, int j) { constexpr int v = decltype(v_tag)::value; eb[v & 1][j] = bit_unit<v>(pb[j]); };
    auto expand_a = [&](auto v_tag, int i, int slot) { constexpr int v = decltype(v_tag)::value; ea[slot] = bit_unit<v>(pa[i]); };
    auto slab = [&](int s, auto p_tag) {
        constexpr int p = decltype(p_tag)::value;
        store(p ^ 1, p ^ 1, s + 1);
        load(p ^ 1, min(s + 3, nslabs - 1));
        static_for<4 * MT>([&](auto t_tag) {
            constexpr int t = decltype(t_tag)::value, v = t / MT, i = t % MT;
            if constexpr (v == 3) read_a(p ^ 1, i);
            expand_a(std::integral_constant<int, ((t + 1) / MT) & 3>{}, (t + 1) % MT, (t + 1) & 1);
            if constexpr (i == MT - 1)
#pragma unroll
                for (int j = 0; j < NT; ++j) expand_b(std::integral_constant<int, (v + 1) & 3>{}, j);
            if constexpr (v == 2 && i == MT - 1) {
                __syncthreads();
#pragma unroll
                for (int j = 0; j < NT; ++j) read_b(p ^ 1, j);
            }
#pragma unroll
            for (int j = 0; j < NT; ++j)
                acc[i][j] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(as_operand(ea[t & 1]), as_operand(eb[v & 1][j]), acc[i][j], 4, 4, 0,
                                                                            scale_of_bit(v), 0, 127);
        });
    };
    std::integral_constant<int, 0> p0;
    std::integral_constant<int, 1> p1;
    load(0, 0);
    load(1, min(1, nslabs - 1));
    store(0, 0, 0);
    load(0, min(2, nslabs - 1));
    __syncthreads();
#pragma unroll
    for (int j = 0; j < NT; ++j) { read_b(0, j); expand_b(p0, j); }
#pragma unroll
    for (int i = 0; i < MT; ++i) read_a(0, i);
    expand_a(p0, 0, 0);
    int s = 0;
    do {
        slab(s, p0);
        if (s + 1 < nslabs) slab(s + 1, p1);
    } while ((s += 2) < nslabs);

    // ---- partial sums meet: a block of 32 x 32 for each of the first waves
    float* set_lds = reinterpret_cast<float*>(lds + TL::SET_AT);        // [RA], [RB]
    auto row_sum = [](int v) {
        v += __builtin_amdgcn_update_dpp(0, v, 0xB1, 0xF, 0xF, true);                       // quad_perm 1 0 3 2
        v += __builtin_amdgcn_update_dpp(0, v, 0x4E, 0xF, 0xF, true);                       // quad_perm 2 3 0 1
        if (GR >= 8) v += __builtin_amdgcn_update_dpp(0, v, 0x141, 0xF, 0xF, true);         // row_half_mirror
        if (GR >= 16) v += __builtin_amdgcn_update_dpp(0, v, 0x140, 0xF, 0xF, true);        // row_mirror
        return v;
    };
#pragma unroll
    for (int q = 0; q < LA; ++q) {
        const int n = row_sum(set_a[q]);
        if (gr == 0) set_lds[r0 + RSTEP * q] = -2.f * (float)n;
    }
#pragma unroll
    for (int q = 0; q < LB; ++q) {
        const int n = row_sum(set_b[q]);
        if (gr == 0) set_lds[RA + r0 + RSTEP * q] = -2.f * (float)n;
    }
    constexpr int BLOCKS = TL::WM * WN * MT * NT;
    __syncthreads();                                     // the slabs are done with: their memory takes the partial sums
    float4* part = reinterpret_cast<float4*>(lds);       // [kg][block][quad][lane]
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int j = 0; j < NT; ++j) {
            const int block = (wm * MT + i) * (WN * NT) + wn * NT + j;
#pragma unroll
            for (int q = 0; q < 4; ++q)
                part[((kg * BLOCKS + block) * 4 + q) * 64 + lane] = make_float4(acc[i][j][4 * q], acc[i][j][4 * q + 1], acc[i][j][4 * q + 2], acc[i][j][4 * q + 3]);
        }
    __syncthreads();
    for (int block = wave; block < BLOCKS; block += NTHR / 64) {
        const int bm = block / (WN * NT), bn = block % (WN * NT);
        const float col_set = set_lds[RA + 32 * bn + l32];
        v16f sum[1][1];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            float4 v = part[(block * 4 + q) * 64 + lane];
#pragma unroll
            for (int k = 1; k < WK; ++k) {
                const float4 o = part[((k * BLOCKS + block) * 4 + q) * 64 + lane];
                v.x += o.x; v.y += o.y; v.z += o.z; v.w += o.w;
            }
            const float4 rs = *reinterpret_cast<const float4*>(set_lds + 32 * bm + 8 * q + 4 * half);
            sum[0][0][4 * q] = v.x + rs.x + col_set; sum[0][0][4 * q + 1] = v.y + rs.y + col_set;
            sum[0][0][4 * q + 2] = v.z + rs.z + col_set; sum[0][0][4 * q + 3] = v.w + rs.w + col_set;
        }
        const long long m0 = m_base + 32 * bm;
        const int n0 = n_base + 32 * bn;
        if (e.bits != nullptr) {
            int thi[1];
            bool cok[1];
            column_thresholds<1>(thi, cok, n0, l32, g, e);
            epilogue_bits<1, 1>(sum, m0, n0, lane, g, e, -g.bits_tap, thi, cok);
        } else {
            epilogue_sums<1, 1>(sum, m0, n0, lane, g, e, -g.bits_tap);
        }
    }
}

}  // namespace mfma
}  // namespace bnn
#endif
