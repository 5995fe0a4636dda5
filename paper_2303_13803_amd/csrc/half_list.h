// The two best of a wavefront's values, an entry of a list a lane (Core::bid in core.hip).
//
// A maximum of doubles over a wavefront is a dozen dependent instructions of eight cycles and more, one of integers half
// a dozen of four.  So the two best are looked for by their distances above what nothing else is worth more than, as
// floats, whose bits are in their order.  Values are whole numbers: up to 2^24 floats tell them all apart, and above that
// rounding keeps their order, so the best is among those with the largest float.  Where several share that, the doubles
// decide; both values are exact.  (The second one from its float, rounded up, made bids that rise by a
// little less than they may; seven measured calls took 0.98 to 1.02 of the time.)
//
// No dependence on the device: tests/half_list.cpp runs it with arrays in the lanes' place.
#pragma once

#if defined(__HIPCC__)
#define MF_HALF_FN __host__ __device__ __forceinline__
#else
#define MF_HALF_FN inline
#endif

constexpr int HALF_EXACT = 0x4b800000;      // bits of 2^24 as a float

// The lane of the best value; among ties the first at or after lane `turn`.  largest: 0 if none exceeds `outside`.
template <class Wave>
MF_HALF_FN int best_lane(const Wave &wave, const typename Wave::Values &v, const typename Wave::Keys &key, unsigned turn, int *largest)
{
    *largest = wave.largest(key);
    unsigned long long hit = wave.equal(key, *largest);
    if (hit & (hit - 1ull)) {
        hit = wave.equal_among(v, wave.largest_among(v, hit), hit);
        const unsigned long long turned = hit & (~0ull << turn);
        hit = turned ? turned : hit;
    }
    return __builtin_ctzll(hit);
}

// The largest value of the other lanes, if that is more than `outside`; *next: 0 if it is not.
template <class Wave>
MF_HALF_FN double next_value(const Wave &wave, const typename Wave::Values &v, const typename Wave::Keys &key, int best, double outside, int *next)
{
    const typename Wave::Keys others = wave.without(key, best);
    *next = wave.largest(others);
    if (*next < HALF_EXACT) return outside + wave.distance(*next);         // (`outside` itself, if none is)
    const unsigned long long hit = wave.equal(others, *next);
    return hit & (hit - 1ull) ? wave.largest_among(v, hit) : wave.at(v, __builtin_ctzll(hit));
}
