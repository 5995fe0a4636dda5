// Which entries of a line core_list_kernel looks at exactly (core.hip).
//
// An entry belongs on the list, or ties with the cut, if K w - dual >= cut in whole numbers below 2^44.  Doubles show that exactly, in
// seven instructions an entry, floats nearly, in three.  An entry worth the cut has K w of at most `most` and so a dual of at most
// most - cut; float(w), K float(w) and float(dual) are off by 2^-24 of these or less, and rounding the difference by
// 2^-24 of it once more, together less than 2^-21 (most + |cut|).  So what floats show to be less than the cut
// by 2^-20 of that is less than the cut; the others are looked at exactly.
//
// No dependence on the device: tests/list_cut.cpp tries it on both sides of the cut.
#pragma once

#include <math.h>

#if defined(__HIPCC__)
#define MF_CUT_FN __host__ __device__ __forceinline__
#else
#define MF_CUT_FN inline
#endif

constexpr double LIST_ALL = -1.0e300, LIST_NONE = 1.0e300;      // cuts

MF_CUT_FN float cut_in_floats(double cut, double most)
{
    if (cut >= LIST_NONE) return INFINITY;
    if (cut <= LIST_ALL) return -INFINITY;
    return (float)(cut - 0x1p-20 * (most + fabs(cut)));
}
MF_CUT_FN bool may_reach(float K, int w, float dual, float cut) { return fmaf(K, (float)w, -dual) >= cut; }
