// Internal interface of the draw-ahead kernel (class masks in global memory).
#pragma once

#include "sd_kernels.hpp"

namespace sd {

// Lattices the kernel takes: up to two words per thread of a workgroup.  (Four
// words a thread spill: 512^2 3.5 us a half-step against 2.6 for five chains in
// the whole-step kernel.)
constexpr uint32_t kAheadMaxWords = 2048;
inline bool ahead_size(int32_t L) { return L >= 8 && ((uint64_t)L * (uint64_t)L + 63u) / 64u <= kAheadMaxWords; }

// A call's run of several chains of one size in rounds: launch r draws the
// class masks of round r, walks the chains through round r - 1 and takes the
// records of round r - 2.  Every slot-sized area exists twice (r mod 2).
struct AheadArgs {
    void* sigma[kManyMax];
    void* tau[kManyMax];
    uint32_t T[kManyMax][6];
    uint32_t stream[kManyMax];
    uint32_t n_chains;
    uint32_t key0, key1, rng_xor;
    uint32_t L, N, n;        // side, sites, 64-site words (the last one may be partial)
    FastDiv div_n, div_L;
    uint32_t int8_io;        // lattices are int8 (any address), else 64-bit words
    uint32_t H;              // half-steps per round, even
    uint64_t* masks;         // [2][chain][H][3][n][2] (classes 2 k, 2 k + 1)
    uint64_t* hist;          // [2][chain][H][n] new words of a round (null: no records)
    uint64_t* state;         // [chain][2][n] sigma, tau between rounds
    int64_t* obs;            // record r of chain a: obs + a * obs_chain + 3 r
    uint64_t obs_chain;
    uint32_t obs_every;
    // this launch
    uint32_t draw_t, draw_count, draw_slot, draw_blocks;
    uint32_t walk_count, walk_slot, walk_first, walk_last;
    uint32_t rec_step, rec_count, rec_slot, rec_blocks;   // rec_step: steps done before the round
};

// Scratch that holds rounds of four half-steps of the most and largest chains
// (two slots of six masks and the new word per half-step, and the two lattices).
constexpr size_t kAheadMinBytes = sizeof(uint64_t) * kManyMax * kAheadMaxWords * (2u * 4u * 7u + 2u);
// Runs every round of k_steps steps from step step0; the caller fills the
// chains, keys, geometry (L, int8_io), and records, and gives `bytes` >=
// kAheadMinBytes of scratch (16-byte aligned device memory).
hipError_t run_ahead(AheadArgs a, uint64_t step0, uint32_t k_steps, void* scratch, size_t bytes, hipStream_t st);

}  // namespace sd
