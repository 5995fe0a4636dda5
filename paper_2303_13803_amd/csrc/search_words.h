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

// ---- lines read whole ----
// What is not on a row's list is at least as far off as the list's bound says.  The pass over all
// columns, during which no label changes, has the whole line read once that is near enough, and notes
// the label the column has (`read_from`) and that nothing has been left out (`left`).  The slices of the
// line read the label for themselves, that one or a shorter one, offer what they find and lower `left`
// to the nearest entry that lay beyond every path end.  So the reading counts for as long as the label
// is not below `read_from`; from a shorter label the list's bound holds again.  Scans of the row do not
// touch either word: a scan in the step that reads the line, as the pass asks for when it also has
// candidates to offer again, neither undoes the reading (the line was read twice) nor gets in its way.
struct WholeLine {
    unsigned long long *read_from;      // of the column: the label its holder's line has been read whole from
    double *left;                       // the nearest entry that reading left out
};

// (by the pass over all columns, which looks at a column once)
template <class Mem>
MF_SEARCH_FN void begin_whole_line(const Mem &mem, const WholeLine &at, unsigned long long length, double nothing)
{
    mem.set(at.read_from, length);
    mem.set(at.left, nothing);
}

template <class Mem>
MF_SEARCH_FN void publish_slice(const Mem &mem, const WholeLine &at, double left_out) { mem.lower(at.left, left_out); }

// How far off the nearest entry is at least that has neither been offered nor is in `dropped`, for a row
// scanned from `length`; `by_bound`: base - the list's bound.
MF_SEARCH_FN double unlisted_from(unsigned long long length, unsigned long long read_from, double left, double by_bound)
{
    return length >= read_from ? left : by_bound;
}

// ---- searches that end before all their bidders are placed ----
// Serving a path of length d raises its own tree's columns by d less their labels.  The columns of other trees with labels below d are
// left as they are until their own tree is served, by a path at least as long: until then a row of the served tree may like one of
// them better than what it holds, by up to d less that column's label, which is more than the epsilon that bids and searches rest on.
// So a search that ends early raises them by that: as far as if their trees had been served at the length of the last
// path.  (Labels below that length are final; those of the served tree's columns are not below it.  Left out, later searches met cycles of
// negative length, found no root and gave up: one in twelve solves of rank-one weights, 848 x 924.)
MF_SEARCH_FN unsigned long long pending_rise(unsigned long long label, unsigned long long none, int id_bits, unsigned long long served)
{
    const unsigned long long length = label >> id_bits;
    return label != none && length < served ? served - length : 0ull;
}
