// A run of fully-connected layers in one launch (bnn_fc_chain.hip).
#ifndef BNN_FC_CHAIN_H
#define BNN_FC_CHAIN_H
#include "bnn_internal.h"

namespace bnn {

constexpr int FC_CHAIN_MAX = 4;

struct FcChainLayer {
    const uint32_t* W;     // [N][tw] packed weights
    const int32_t* thr;    // with bits
    uint32_t* bits;        // [rows][ldo]: thresholded output; nullptr: int32 sums to FcChain::out (last layer only, at most 64 columns)
    int K, N, tw, ldo;
    int groups, thr_cols;  // filled by launch_fc_chain: groups of 64 columns, those of the pad words in `bits` included; 64 * groups or, for sums, 0
};
struct FcChain {
    int nlayers;
    long long rows;
    const uint8_t* in_u8;  // input: 8-bit values [rows][in_cols] (16 or more), bit = (x >= in_thr), packed into in_bits_out [rows][in_ldw] on the way ...
    int in_cols, in_thr, in_ldw;
    uint32_t* in_bits_out;
    const uint32_t* in_bits;    // ... or packed rows [rows][in_ldw]
    int32_t* out;
    int buf_words, thr_count, thr_most, bit_words, turn_at;     // filled by launch_fc_chain: words of an activation buffer, thresholds, packed words of a row, an LDS offset
    FcChainLayer layer[FC_CHAIN_MAX];
};

// Whether one launch is the better one for these layers (the fields that launch_fc_chain fills are not read).  replayed: for launches that are recorded into a
// graph, whose replay costs the host nothing.
bool fc_chain_takes(const FcChain& a, bool replayed);
int launch_fc_chain(FcChain a, hipStream_t s);

}  // namespace bnn
#endif
