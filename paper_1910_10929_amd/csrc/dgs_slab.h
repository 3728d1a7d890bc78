// Positions of the slabs of an emission: what a slab publishes for the slabs of its tensor that
// lie behind it, and how a slab adds up what lies before it (the single-pass prefix sum with
// decoupled look-back of Merrill and Garland).
#pragma once
#include "dgs_select.h"

namespace dgs {

// A slab's entries above the k-th key and equal to it (SLAB_OWN), or the same for all slabs of the
// tensor up to and including it (SLAB_SUM); SLAB_FAIL: it gave up waiting and emits nothing, and so
// does every slab behind it; 0: nothing published yet.
constexpr uint32_t SLAB_OWN = 1u, SLAB_SUM = 2u, SLAB_FAIL = 3u;

// WIDE: two words, (g, kind) and (q, kind), for counts of any size: a dense request counts every
// element of its tensor, up to 2^32 - 1 of them.  Otherwise one word with 31 bits for either count:
// candidates, of which a tensor has fewer than n / 4.
template <bool WIDE>
struct SlabWord {
    uint64_t w = 0;
    __device__ __forceinline__ uint32_t kind() const { return (uint32_t)(w >> 62); }
    __device__ __forceinline__ bool published() const { return w != 0; }
    __device__ __forceinline__ uint32_t g() const { return (uint32_t)w & 0x7FFFFFFFu; }
    __device__ __forceinline__ uint32_t q() const { return (uint32_t)(w >> 31) & 0x7FFFFFFFu; }
    __device__ __forceinline__ void read(const uint2 *word)
    {
        const uint2 x = ld_dev(word);
        w = ((uint64_t)x.y << 32) | x.x;
    }
};

template <>
struct SlabWord<true> {
    uint32_t k = 0, above = 0, equal = 0;
    __device__ __forceinline__ uint32_t kind() const { return k; }
    __device__ __forceinline__ bool published() const { return k != 0; }
    __device__ __forceinline__ uint32_t g() const { return above; }
    __device__ __forceinline__ uint32_t q() const { return equal; }
    // (two words of different kinds: the slab is between its two publications, read again)
    __device__ __forceinline__ void read(const uint2 *word)
    {
        const uint2 a = ld_dev(word), b = ld_dev(word + 1);
        k = (a.y == b.y) ? a.y : 0u;
        above = a.x;
        equal = b.x;
    }
};

template <bool WIDE>
__device__ __forceinline__ void slab_publish(uint2 *word, uint32_t kind, uint32_t g, uint32_t q)
{
    if (WIDE) {
        st_dev(word, make_uint2(g, kind));
        st_dev(word + 1, make_uint2(q, kind));
    } else {
        st_dev(word, make_uint2(g | (q << 31), (q >> 1) | (kind << 30)));
    }
}

// Entries above / equal to the k-th key in the tensor's slabs [first, slab), by one wavefront
// looking back over up to 64 slabs at a time until one has published its running sum
// (word_of(i): where slab i publishes).  Those are blocks with lower indices; bounded by
// A.spin_limit polls.  Returns false, in every lane, if it gave up (counted as an internal error) or
// if a slab before it has: the positions are not known then.
template <bool WIDE, class WordOf>
__device__ __forceinline__ bool slab_look_back(const SelectArgs &A, uint32_t slab, uint32_t first, WordOf word_of,
                                               uint32_t &g, uint32_t &q)
{
    const uint32_t lane = lane_id();
    g = q = 0;
    for (uint32_t hi = slab; hi > first;) {          // slabs [first, hi) are still to be added
        const bool in = hi - first > lane;
        SlabWord<WIDE> w;
        uint64_t have = 0, sums = 0;
        for (uint32_t spin = 0; spin < A.spin_limit; ++spin) {
            if (in && !w.published()) w.read(word_of(hi - 1u - lane));
            have = ballot64(!in || w.published());
            sums = ballot64(in && w.kind() >= SLAB_SUM);
            // everything up to the nearest running sum (or all 64) has been published
            const uint64_t upto = sums ? (((sums & (0ull - sums)) << 1) - 1ull) : ~0ull;
            if ((have & upto) == upto) break;
            __builtin_amdgcn_s_sleep(1);
        }
        const uint64_t upto = sums ? (((sums & (0ull - sums)) << 1) - 1ull) : ~0ull;
        if ((have & upto) != upto) {                 // gave up waiting
            if (lane == 0) atomicAdd(&A.stats->internal_errors, 1ull);
            return false;
        }
        const uint32_t counts = 0u - (uint32_t)((upto >> lane) & 1u);      // (lanes beyond `first` hold 0)
        g += wave_sum(w.g() & counts);
        q += wave_sum(w.q() & counts);
        if (sums) return (ballot64(w.kind() == SLAB_FAIL) & upto) == 0;
        hi = (hi - first > 64u) ? hi - 64u : first;
    }
    return true;
}

}  // namespace dgs
