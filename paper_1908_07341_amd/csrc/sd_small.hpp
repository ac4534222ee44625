// Internal interface of the small-lattice kernel (class masks drawn ahead).
#pragma once

#include "sd_kernels.hpp"

namespace sd {

struct SmallArgs {
    uint32_t T[6];        // threshold table of the chain(s)
    uint32_t key0, key1;
    uint32_t stream;      // of the chain, or of pair 0 (pair p: stream + p)
    uint32_t t0;          // first half-step index (even)
    uint32_t n_half;      // half-steps to run (even, 2 x steps)
    uint32_t rng_xor;
    uint32_t L, n;        // side and 64-site words (L * L / 64 <= 64)
    FastDiv div_n, div_L;
    uint32_t H;           // half-steps per epoch (set by launch_small)
    // one chain
    void* sigma;
    void* tau;
    uint32_t int8_io;     // sigma and tau are int8 (any address), else 64-bit words
    int64_t* obs;         // records, or null
    uint32_t obs_every;
    // coupled pairs: workgroup b runs pair pairs[b]
    const uint32_t* pairs;
    uint8_t* samples;     // pair p's top lattice at time 0 at samples + p * lattice bytes
    uint32_t* equal;      // equal[b] = the two chains of pairs[b] agree
};

// True for the sides the kernel takes (L % 8 == 0, at most 64 words).
bool small_supported(int32_t L);
// One workgroup per chain (blocks = 1, pair false) or per coupled pair; n_half > 0.
hipError_t launch_small(SmallArgs a, uint32_t blocks, bool pair, uint32_t n_cu, size_t max_lds, hipStream_t st);

}  // namespace sd
