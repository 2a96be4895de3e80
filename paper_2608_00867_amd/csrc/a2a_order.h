// a2a_order.h -- Algorithm 1 for the all-to-all dispatch (host).
//
// The copies of one token share its source row and nothing else, so the
// logical groups are the tokens; each group goes to the next of the 8 XCDs in
// decreasing size order, tokens of equal size in token order, which evens out
// the copies per XCD.  Every copy is charged the same, so the request budgets
// never bind and only the XCD matters.
//
// These are the domains that nap_plan gives for the workload of one
// threadblock per copy, touching its source row and its destination row.  The
// general planner finds the groups through hash maps over the chunks and homes
// every chunk, none of which this workload needs: a layout of 8 ranks and 128
// tokens per rank, top-8, took 794 us to create with it and takes 31 us now.
// Sizes are at most 64, so a counting sort gives the order.
#ifndef NUNA_A2A_ORDER_H
#define NUNA_A2A_ORDER_H

#include <cstdint>

#include "placement.h"

namespace nuna {

// mask[i]: the destination ranks of token i (at least one).  Writes every
// token's XCD and the copies per XCD.
inline void a2a_token_xcds(const uint64_t* mask, int64_t ntok, uint8_t* xcd, int64_t (&copies)[kNumXcd]) {
    int64_t first[65] = {};  // place in the order of the next token of a size
    for (int64_t i = 0; i < ntok; ++i) ++first[__builtin_popcountll(mask[i])];
    int64_t at = 0;
    for (int size = 64; size >= 0; --size) {
        const int64_t n = first[size];
        first[size] = at;
        at += n;
    }
    for (int64_t& c : copies) c = 0;
    for (int64_t i = 0; i < ntok; ++i) {
        const int size = __builtin_popcountll(mask[i]);
        xcd[i] = static_cast<uint8_t>(first[size]++ & (kNumXcd - 1));
        copies[xcd[i]] += size;
    }
}

}  // namespace nuna

#endif
