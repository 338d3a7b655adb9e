// A run of small fully-connected layers as ONE launch: a workgroup takes 16 * RT rows through all of them.
//
// A layer of the MLP (1024 x 1024 bits of weights) is 1 us of work for the chip and a launch of 3.5 to 4.5 us, and each layer
// waits for the one before: the pass is bound by launches.  But fully-connected layers never mix rows, so a workgroup can carry
// its rows through the whole run with no more than a workgroup barrier between two layers.  What it pays is that every
// workgroup reads and expands all weights itself -- its time is vector instructions, nearly all for the weights --, so the run is
// taken only while its layers are small (fc_chain_takes()).
//  * A wave owns groups of 64 output columns.  v_mfma_f32_16x16x128_f8f6f4 with the WEIGHTS as row operand: lane l supplies weight
//    row l % 16 and 32 K slots of group l / 16, which is one packed word.  The lanes of a load take 8 rows x 128 neighbouring bytes and the
//    words change lanes through 8 KB of LDS that belong to the wave: loaded as operands, every lane in another row than its neighbours, the
//    address side takes a cycle for each lane (measured: 128 such loads of 1 KB, a layer's weights, 8400 cycles, whatever was multiplied; 6700 now, 6050 of them vector instructions).
//    64 weight rows x 1024 bits are in flight, across layers: weights do not wait for activations.
//  * Weight words cost four instructions instead of seven.  Bits 0, 1 and 2 of a nibble are left where they are and mean 0.5, 1 and
//    2 or zero (b in {0, 1}), bit 3 is the sign of 1.  The activations, which are expanded once per workgroup, carry the factors 4, 2 and
//    1 that make each product 2 a b = a + a s (s = 2 b - 1), and a s for bit 3.  What is too much, the sum of a over three of four K
//    slots, is one number per row: the accumulators start at minus it.  All exact: whole and half numbers below 2^23.
//  * A layer's activations lie in LDS as finished operands (one 16-byte unit per row and word), written by the epilogue of the layer
//    before or by the input stage.
//  * Weight rows are dealt to the MFMA's rows so that a lane ends up with 16 consecutive channels of one row (tile j, row m:
//    channel 16 * (m / 4) + 4 * j + m % 4); accumulators start half an integer beside minus the threshold, the bits are collected from their
//    signs, and two lanes meet in a word by one v_permlane16_swap.  The packed bits are also stored, as bnn_net_layer_bits hands them out.
#include <algorithm>

#include "bnn_fc_chain.h"
#include "bnn_mfma_kernel.h"

namespace bnn {
namespace {

using mfma::as_operand;

typedef float v4f __attribute__((ext_vector_type(4)));
typedef uint32_t v4u __attribute__((ext_vector_type(4)));
typedef int32_t raw16 __attribute__((ext_vector_type(4), aligned(1)));     // 16 bytes at any address
typedef uint8_t bytes16 __attribute__((ext_vector_type(16)));

constexpr int CT = 4;          // column tiles of 16 in a group
constexpr uint32_t B0 = 0x11111111u, B1 = 0x22222222u, B2 = 0x44444444u, B3 = 0x88888888u;   // bit 0 .. 3 of every nibble

// A packed word of activations as operand: +-4, +-2, +-1 at bits 0, 1, 2 (set: plus) and, the other way round, -+1 at bit 3.
__device__ __forceinline__ uint4 activation_unit(uint32_t w) {
    const uint32_t n = ~w;
    return make_uint4(((n << 3) & B3) | (B1 | B2), ((n << 2) & B3) | B2, ((n << 1) & B3) | B1, (w & B3) | B1);
}

__device__ __forceinline__ int scalar(int v) { return __builtin_amdgcn_readfirstlane(v); }

// RT row tiles of 16; WAVES waves; U8: the input is 8-bit values (rows of 16 or more), else packed rows.
template <int RT, int WAVES, bool U8>
__global__ __launch_bounds__(64 * WAVES, 1) void fc_chain_kernel(FcChain a) {
    constexpr int R = 16 * RT, NTHR = 64 * WAVES;
    // two activation buffers of a.buf_words words x R rows; thresholds; packed bits; set bits (0, 1, 2 of a nibble) by layer and row
    extern __shared__ uint4 smem[];
    float* th_lds = reinterpret_cast<float*>(smem + 2 * a.buf_words * R);
    uint32_t* bits_lds = reinterpret_cast<uint32_t*>(th_lds + a.thr_count);
    int* set_lds = reinterpret_cast<int*>(bits_lds + R * a.bit_words);
    v4u* turn = reinterpret_cast<v4u*>(smem) + a.turn_at + (threadIdx.x >> 6) * 512;             // this wave's 8 KB for weights that change lanes
    const int tid = (int)threadIdx.x, lane = tid & 63, l16 = lane & 15, grp = lane >> 4;
    const int wave = scalar(tid >> 6);
    const long long row0 = (long long)blockIdx.x * R;
    const int rows = (int)min((long long)R, a.rows - row0);

    // ---- input: packed rows or 8-bit values, one word per thread and strip; the first strip is requested ahead of everything else
    const int nw = U8 ? a.in_ldw : a.layer[0].tw;
    uint32_t in_word;
    raw16 in_lo, in_hi;
    auto request_input = [&](int i) {
        const int word = min(i, nw * R - 1) / R, row = min(i % R, rows - 1);               // R is a power of two
        if constexpr (U8) {     // a half-word whose values pass the end of the row loads the row's last 16 and shifts its bits
            const uint8_t* src = a.in_u8 + (row0 + row) * a.in_cols;
            in_lo = *reinterpret_cast<const raw16*>(src + min(32 * word, a.in_cols - 16));
            in_hi = *reinterpret_cast<const raw16*>(src + min(32 * word + 16, a.in_cols - 16));
        } else {
            in_word = a.in_bits[(row0 + row) * a.in_ldw + word];
        }
    };
    auto store_input = [&](int i) {                 // (the loaded values are used outside the branches: a load that may be pending at a join holds up every wait behind it)
        const int word = i / R, row = i % R;
        uint32_t w;
        if constexpr (U8) {
            auto pack = [&](raw16 raw, int over) {
                const bytes16 v = __builtin_bit_cast(bytes16, raw);
                uint32_t m = 0u;
#pragma unroll
                for (int q = 0; q < 16; ++q) m |= (int)v[q] >= a.in_thr ? 1u << q : 0u;
                return over < 16 ? m >> max(over, 0) : 0u;
            };
            w = pack(in_lo, 32 * word - (a.in_cols - 16)) | (pack(in_hi, 32 * word + 16 - (a.in_cols - 16)) << 16);
        } else {
            w = in_word;
        }
        w = row < rows ? w : 0u;
        asm volatile("" :: "v"(w));
        if (i < nw * R) {
            if (U8 && row < rows) a.in_bits_out[(row0 + row) * a.in_ldw + word] = w;
            smem[i] = activation_unit(w);
            atomicAdd(&set_lds[row], __popc(w & ~B3));
        }
    };
    request_input(tid);
    int tv[FC_CHAIN_MAX];                           // thresholds, likewise: waiting for them does not wait for weights
#pragma unroll
    for (int l = 0; l < FC_CHAIN_MAX; ++l) tv[l] = a.layer[l].thr[min(tid, a.layer[l].N - 1)];

    // ---- weight stream of this wave: groups of 64 columns, 1024 bits of K at a time, layer after layer.  The two buffers (tiles 0 and 1,
    // 2 and 3) hold or wait for part np of group ng of layer nl; past the end the last part is requested again (no branch: the
    // count of loads in flight is a constant of the program).
    int nl = 0, ng = wave, np = 0, ncols = 1, ntw = 0;
    const char* nw_base = reinterpret_cast<const char*>(a.layer[0].W);
    auto enter_layer = [&](int l) {                                        // the first layer from l on in which this wave has columns
        for (; l < a.nlayers; l = scalar(l + 1))
            if (wave * 64 < a.layer[l].N) {
                nl = scalar(l); ng = wave; np = 0;
                nw_base = reinterpret_cast<const char*>(a.layer[l].W); ncols = a.layer[l].N; ntw = a.layer[l].tw;
                return;
            }
    };
    auto advance = [&]() {
        if (32 * (np + 1) < ntw) np = scalar(np + 1);
        else if ((ng + WAVES) * 64 < ncols) { ng = scalar(ng + WAVES); np = 0; }
        else enter_layer(scalar(nl + 1));
    };
    v4u raw[CT][2];                                 // of each tile: weight rows lane / 8 and 8 + lane / 8, words 4 * (lane % 8) .. + 3
    const int lrow = lane >> 3, lunit = lane & 7;
    const int lch = 16 * (lrow >> 2) + (lrow & 3);                         // channel of row lrow of tile 0
    auto request = [&](auto first) {                                       // two tiles
        constexpr int j0 = decltype(first)::value;
        const int word = 32 * np + 4 * lunit;
        const uint32_t off = (uint32_t)(word < ntw ? word : 0);            // past the row (a multiple of four words): masked when expanded
#pragma unroll
        for (int j = j0; j < j0 + 2; ++j)
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const int ch = min(ng * 64 + 32 * h + 4 * j + lch, ncols - 1);
                raw[j][h] = *reinterpret_cast<const v4u*>(nw_base + (size_t)(4u * (__umul24(ch, ntw) + off)));     // below 2^24 words (fc_chain_takes)
            }
    };
    enter_layer(0);
    request(std::integral_constant<int, 0>{}); request(std::integral_constant<int, 2>{});

    // ---- thresholds of all layers, as what a sum is compared with: half an integer below threshold + pad bits
    for (int i = tid; i < a.nlayers * R; i += NTHR) set_lds[i] = 0;
    __syncthreads();
    store_input(tid);
    for (int i = NTHR + tid; i < (nw * R + NTHR - 1) / NTHR * NTHR; i += NTHR) {
        request_input(i);
        store_input(i);
    }
    {
        int at = 0;
        auto value = [&](const FcChainLayer& L, int c, int t) {            // + pad bits inside the row: +1 each
            return (float)((c < L.N ? min(max(t, -(1 << 20)), 1 << 20) : 1 << 20) + (32 * L.tw - L.K)) - 0.5f;
        };
#pragma unroll
        for (int l = 0; l < FC_CHAIN_MAX; ++l) {
            const float first = value(a.layer[l], tid, tv[l]);
            asm volatile("" :: "v"(first));         // before the branch, see store_input
            if (tid < a.layer[l].thr_cols) th_lds[at + tid] = first;
            at += a.layer[l].thr_cols;
        }
        if (a.thr_most > NTHR) {                    // layers of more columns than threads
            at = 0;
            for (int l = 0; l < a.nlayers; ++l) {
                const FcChainLayer& L = a.layer[l];
                for (int c = NTHR + tid; c < L.thr_cols; c += NTHR) th_lds[at + c] = value(L, c, L.thr[min(c, L.N - 1)]);
                at += L.thr_cols;
            }
        }
    }
    __syncthreads();

    v4f acc[RT][CT];
    int th_at = 0, bits_at = 0;                     // of the current layer
    auto pass = [&](int l, auto kind) {             // one layer; two forms, so that no store to memory stands in the loop over the layers with bits
        constexpr bool SUMS = decltype(kind)::value;
        const FcChainLayer& L = a.layer[l];
        const uint4* in = smem + (l & 1) * a.buf_words * R;
        uint4* out = smem + (~l & 1) * a.buf_words * R;
        auto multiply = [&](auto first, const v4u (&w)[2][2], int part, const uint4 (&af)[8][RT]) {      // two tiles
            constexpr int j0 = decltype(first)::value;
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                // words past the end of a weight row: zeros, so that whatever the activation buffer holds there counts nothing
                const uint32_t keep = part + 8 * grp + 4 * h < L.tw ? ~0u : 0u;
                const uint32_t m0 = B0 & keep, m1 = B1 & keep, m2 = B2 & keep, m3 = B3 & keep;
#pragma unroll
                for (int k = 0; k < 4; ++k)
#pragma unroll
                    for (int j = 0; j < 2; ++j) {
                        const uint32_t v = w[j][h][k];
                        const uint4 bu = make_uint4(v & m0, v & m1, v & m2, (v & m3) | m1);
#pragma unroll
                        for (int i = 0; i < RT; ++i)
                            acc[i][j0 + j] = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(as_operand(bu), as_operand(af[4 * h + k][i]), acc[i][j0 + j], 4, 4, 0, 0, 0, 0);
                    }
            }
        };
        float too_much[RT];                         // sum of +-1 over the K slots whose weights are 0 or 1
#pragma unroll
        for (int i = 0; i < RT; ++i) too_much[i] = (float)(2 * set_lds[l * R + 16 * i + l16] - 24 * L.tw);
        for (int group = wave; group < L.groups; group += WAVES) {
            const int n0 = group * 64;
#pragma unroll
            for (int j = 0; j < CT; ++j) {
                v4f th;
                if constexpr (SUMS) { const float c = (float)(32 * L.tw - L.K); th = v4f{c, c, c, c}; }
                else th = *reinterpret_cast<const v4f*>(th_lds + th_at + n0 + 16 * grp + 4 * j);
#pragma unroll
                for (int i = 0; i < RT; ++i)
#pragma unroll
                    for (int r = 0; r < 4; ++r) acc[i][j][r] = -too_much[i] - th[r];
            }
            if (n0 < L.N)
                for (int part = 0; part < L.tw; part += 32) {
                    uint4 af[8][RT];
                    const uint4* ap = in + (part + 8 * grp) * R + l16;
#pragma unroll
                    for (int k = 0; k < 8; ++k)
#pragma unroll
                        for (int i = 0; i < RT; ++i) af[k][i] = ap[k * R + 16 * i];
                    advance();
                    v4u w[2][2][2];
                    auto change_lanes = [&](auto first) {                  // two tiles; the wave's own LDS, in order: no barrier
                        constexpr int j0 = decltype(first)::value;
#pragma unroll
                        for (int j = 0; j < 2; ++j)
#pragma unroll
                            for (int h = 0; h < 2; ++h) turn[(j0 + j) * 128 + (lrow + 8 * h) * 8 + (lunit ^ lrow)] = raw[j0 + j][h];
#pragma unroll
                        for (int j = 0; j < 2; ++j)
#pragma unroll
                            for (int h = 0; h < 2; ++h) w[j0 / 2][j][h] = turn[(j0 + j) * 128 + l16 * 8 + ((2 * grp + h) ^ (l16 & 7))];
                    };
                    std::integral_constant<int, 0> lo;
                    std::integral_constant<int, 2> hi;
                    change_lanes(lo);
                    request(lo);
                    change_lanes(hi);
                    request(hi);
                    __builtin_amdgcn_sched_barrier(0);
                    multiply(lo, w[0], part, af);
                    multiply(hi, w[1], part, af);
                }
            if constexpr (!SUMS) {
                const int word = (n0 >> 5) + (grp >> 1);
#pragma unroll
                for (int i = 0; i < RT; ++i) {
                    uint32_t below = 0u;                                   // bit c: the sum of channel 16 * grp + c is below its threshold
#pragma unroll
                    for (int c = 4 * CT - 1; c >= 0; --c) below = __builtin_amdgcn_alignbit(below, __float_as_uint(acc[i][c >> 2][c & 3]), 31);
                    const uint32_t half = ~below & 0xFFFFu;
                    const auto two = __builtin_amdgcn_permlane16_swap(half, half, false, false);
                    const uint32_t w32 = (uint32_t)two[0] | ((uint32_t)two[1] << 16);
                    const int row = 16 * i + l16;
                    if ((grp & 1) == 0 && word < L.ldo) {
                        out[word * R + row] = activation_unit(w32);
                        bits_lds[bits_at + row * L.ldo + word] = w32;
                        if (l + 1 < a.nlayers) atomicAdd(&set_lds[(l + 1) * R + row], __popc(w32 & ~B3));
                    }
                }
            } else {
#pragma unroll
                for (int j = 0; j < CT; ++j)
#pragma unroll
                    for (int i = 0; i < RT; ++i) {
                        const int ch = n0 + 16 * grp + 4 * j, row = 16 * i + l16;
                        if (row < rows) {
                            int32_t* dst = a.out + (row0 + row) * (long long)L.N + ch;
#pragma unroll
                            for (int r = 0; r < 4; ++r)
                                if (ch + r < L.N) dst[r] = (int)acc[i][j][r];
                        }
                    }
            }
        }
        th_at += 64 * L.groups; bits_at += R * L.ldo;
    };
    const int nbits = a.layer[a.nlayers - 1].bits != nullptr ? a.nlayers : a.nlayers - 1;  // only the last layer may have sums
    for (int l = 0; l < nbits; ++l) {
        pass(l, std::false_type{});
        __syncthreads();
    }
    if (nbits < a.nlayers) pass(nbits, std::true_type{});
    // ---- the packed bits leave here: stores inside the loop would stand in front of the weights (memory operations retire in order)
    int at = 0;
    for (int l = 0; l < a.nlayers && a.layer[l].bits != nullptr; ++l) {
        const FcChainLayer& L = a.layer[l];
        uint32_t* dst = L.bits + row0 * L.ldo;
        for (int i = tid; i < rows * L.ldo; i += NTHR) dst[i] = bits_lds[at + i];
        at += R * L.ldo;
    }
}

// Row tiles and waves: 16 rows (12 waves: 168 registers) while that is a workgroup per compute unit, else 32 (8 waves: 256 registers, which hold two
// rows' operands).  MLP 784-1024-1024-1024-10, 8192 rows: 29 us as 512 workgroups of 16 rows, 23 as 256 of 32.
constexpr int ROWS1 = 16, ROWS2 = 32, CUS = 256;

void fill(FcChain& a) {
    a.buf_words = a.thr_count = a.thr_most = a.bit_words = 0;
    int most = a.in_u8 != nullptr ? a.in_ldw : a.layer[0].tw;
    for (int l = 0; l < a.nlayers; ++l) {
        FcChainLayer& L = a.layer[l];
        L.groups = L.bits != nullptr ? (L.ldo + 1) / 2 : (L.N + 63) / 64;
        L.thr_cols = L.bits != nullptr ? 64 * L.groups : 0;
        most = std::max(most, std::max((L.tw + 31) / 32 * 32, L.bits != nullptr ? L.ldo : 0));
        a.thr_count += L.thr_cols; a.thr_most = std::max(a.thr_most, L.thr_cols);
        if (L.bits != nullptr) a.bit_words += L.ldo;
        else L.thr = reinterpret_cast<const int32_t*>(L.W);                // something to read: the kernel's first loads have no branches
    }
    a.buf_words = most;
    for (int l = a.nlayers; l < FC_CHAIN_MAX; ++l) {
        a.layer[l] = FcChainLayer{};
        a.layer[l].thr = a.layer[0].thr; a.layer[l].N = 1;
    }
}

// LDS in front of the waves' own parts, in 16-byte units
long long turn_at(const FcChain& a, int rows) {
    return cdiv(2LL * a.buf_words * rows * 16 + a.thr_count * 4LL + (a.bit_words + a.nlayers) * (long long)rows * 4, 16);
}
long long lds_bytes(const FcChain& a, int rows, int waves) { return (turn_at(a, rows) + waves * 512LL) * 16; }

template <int RT, int WAVES, bool U8>
int launch_chain(FcChain a, hipStream_t s) {
    a.turn_at = (int)turn_at(a, 16 * RT);
    static const hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void*>(&fc_chain_kernel<RT, WAVES, U8>),
                                                       hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
    if (attr != hipSuccess) return BNN_ERR_DEVICE;
    launch((fc_chain_kernel<RT, WAVES, U8>), dim3((unsigned)cdiv(a.rows, 16 * RT)), dim3(64 * WAVES),
                       (size_t)lds_bytes(a, 16 * RT, WAVES), s, a);
    return check_launch();
}

}  // namespace

// One launch is worth what it saves and costs about 2.7 us for each 2^20 weight bits that every workgroup expands.
// Queued from the host it saves 2.2 us (host) to 4 us (kernels of 129 rows and more) for each layer.  Measured, a pass of a network through
// Net.forward, one launch per layer -> one launch, us:
//   784-1024-1024-1024-10 on 8-bit values: 8 rows 17.6 -> 14.8, 128 19.6 -> 15.2, 1024 19.6 -> 15.4, 4096 24.5 -> 16.0, 8192 28.2 -> 23.0; 16384 38.8 -> 43.5
//   the same on packed rows: 256 16.7 -> 14.8; 8 rows 13.3 -> 14.0 (2.8 * 2^20 bits, four launches); 784-1024-1024-10, 8 rows 12.6 -> 11.2
//   784-512-512-10 on 8-bit values: 8 rows 15.1 -> 9.6, 1024 15.2 -> 10.2; 1024-1024-10 on packed rows: 8 rows 10.1 -> 8.3, 1024 10.1 -> 8.7
// Sums of more than 64 columns leave element by element (784-256, 4096 rows: 8.8 -> 10.4; 1024-1024-1024-1000 19.9 -> 33.2), and behind other layers, where the
// queue is full and a launch costs less, two layers are no gain (1024-1024-10 at the end of a VGG for 32x32 images: 41.5 -> 43.4).
// Replayed from a graph a layer costs its kernel alone, and the kernels for few rows (bnn_mfma_skinny.hip) end after 2.3 us: the run's gain over them, graph replays,
// at 1 to 16 / 17 to 64 / 65 to 128 / 129 to 1024 / 1025 to 4096 rows (launches, 2^20 bits):
//   784-1024-1024-1024-10 on 8-bit values (5, 2.9)  0.82 to 0.85 / 0.99 to 1.10 / 1.27 / 1.18 / 1.34 to 1.49;  packed (4, 2.9)  - / - / - / 1.05 / 1.22 to 1.42
//   784-640-640-640-10 on 8-bit values (5, 1.3)     0.91 to 0.96 / 1.11 to 1.22 / 1.40 / 1.22 / 1.24 to 1.44;  512 wide (5, 0.7)  1.04 / 1.23 / 1.5 / 1.3 / 1.3
//   784-1024-1024-10 on 8-bit values (4, 1.9)       0.79 to 0.85 / 1.01 to 1.11 / 1.27 / 1.16 / 1.29 to 1.46;  packed (3, 1.9)  0.70 / 0.87 to 0.98 / 1.15 / 1.04 / 1.16
//   784-512-512-10 on 8-bit values (4, 0.7)         0.97 to 1.02 / 1.20 to 1.31 / 1.5 / 1.28 / 1.29 to 1.41;   packed (3, 0.7)  0.87 / 1.06 to 1.19 / 1.37 / 1.13 / 1.14
//   256-256-256-256-10 (5 and 4, 0.2)               1.07 to 1.19 / 1.3 to 1.5 / 1.65 to 1.75 / 1.2 to 1.4 / 1.2 to 1.4
//   784-128-10, 784-256-10 on 8-bit values (3; 0.1, 0.2)  0.96 to 1.06 / 1.19 to 1.32 / 1.47 / 1.25 / 1.27
//   1500-1024-512-10 (3, 2.0)  - / - / - / 0.92 to 0.94 / 0.98 to 1.13;  1024-1024-10 packed (2, 1.01)  0.65 / 0.82 to 0.92 / 1.08 / 0.99 to 1.01 / 1.10 to 1.24
//   2048-512-64 packed (2, 1.03)  0.65 / 0.76 to 0.84 / 1.02 / 0.95 to 0.97 / 0.94 to 1.12;  784-512-10 packed (2, 0.4)  0.75 / 0.94 to 1.05 / 1.22 / 1.03 / 1.06
//   784-64 on 8-bit values (2, 0.05)  0.83 to 0.89 / 0.97 to 1.08 / 1.13 / 1.03 / 0.96 to 1.02, beyond 4096 rows 0.85 to 0.88; everything else there 0.97 to 1.4
// (2048-512-64 at 8192 rows, where a launch of its own takes the 128x128 tiles for the first layer, is the one loss found there: 0.85, queued 0.91 to 0.96).
bool fc_chain_takes(const FcChain& in, bool replayed) {
    const int launches = in.nlayers + (in.in_u8 != nullptr ? 1 : 0);
    if (in.nlayers < 1 || launches < 2 || in.rows > (long long)ROWS2 * CUS || (in.in_u8 != nullptr && in.in_cols < 16)) return false;
    long long bits = 0;
    for (int l = 0; l < in.nlayers; ++l) bits += (long long)in.layer[l].N * in.layer[l].tw * 32;
    if (bits > (in.rows > 128 ? launches << 20 : launches * 680000LL)) return false;
    if (replayed) {
        constexpr long long M = 1 << 20;
        if (in.nlayers == 1 && in.rows > (long long)ROWS1 * CUS) return false;
        if (in.rows <= 16 && bits > (launches - 3) * M / 2 + M / 5) return false;
        if (in.rows > 16 && in.rows <= 64 && bits > (15 * launches - 28) * M / 16) return false;
        if (in.rows > 128 && in.rows <= 1024 && bits > (launches - 1) * M) return false;
    }
    FcChain a = in;
    fill(a);
    return a.rows <= (long long)ROWS1 * CUS ? lds_bytes(a, ROWS1, 12) <= 160 * 1024 : lds_bytes(a, ROWS2, 8) <= 160 * 1024;
}

int launch_fc_chain(FcChain a, hipStream_t s) {
    fill(a);
    if (a.rows <= (long long)ROWS1 * CUS) return a.in_u8 != nullptr ? launch_chain<1, 12, true>(a, s) : launch_chain<1, 12, false>(a, s);
    return a.in_u8 != nullptr ? launch_chain<2, 8, true>(a, s) : launch_chain<2, 8, false>(a, s);
}

}  // namespace bnn
