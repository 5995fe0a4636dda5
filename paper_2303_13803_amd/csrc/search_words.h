// What a search on lists keeps of a scanned row, and how scans publish it (see Core::search in core.hip).
//
// Two wavefronts may scan one row in the same step, from different labels of the column it holds: the
// column is on the frontier once for every time its label was lowered.  What a scan found is several
// words, and nothing keeps one scan's words together.  Each of them therefore only goes down between
// two served paths, by an atomic minimum: prices stand still meanwhile, so every value of the scan
// from the shorter label is at most that of the other, and in whatever order the two land the shorter
// label's stay.  (Plain stores could leave a longer label's `base` beside the shorter one's `expanded`:
// path ends and labels too long, which nobody would look at again.)
//
// No dependence on the device: tests/search_words.cpp puts these functions through every order of
// their memory accesses on the CPU.
#pragma once

#if defined(__HIPCC__)
#define MF_SEARCH_FN __host__ __device__ __forceinline__
#else
#define MF_SEARCH_FN inline
#endif

struct ScanWords {
    double *base;                       // of the row: length of the path to it + its profit + eps
    double *dropped;                    // of its column: the shortest candidate left out because it lay beyond every path end
    unsigned long long *expanded;       // of its column: the label the row was scanned from
};

// mem.lower(word, value): atomic minimum; values are not negative.
template <class Mem>
MF_SEARCH_FN void publish_scan(const Mem &mem, const ScanWords &at, unsigned long long length, double base, double left_out)
{
    mem.lower(at.base, base);
    mem.lower(at.dropped, left_out);
    mem.lower(at.expanded, length);
}

// The pass over all columns: the row counts as scanned from the column's label as it is now.
MF_SEARCH_FN bool scanned_from(unsigned long long length, unsigned long long expanded) { return length >= expanded; }
