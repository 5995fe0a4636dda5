// The matching on short lists (paper: Algorithm "Scheduling algorithm", GetMatching).
//
// Once the duals are known to within a few epsilons, a bidder chooses among a handful of lines: on
// cluster-scale rounds a row has 2-200 columns within a hundred epsilons of its best one, out of
// 20,000.  From that phase on every bidding line is kept as a list of its CORE_LIST best entries
// and one number, the largest value K w - dual of any entry that is not on the list.  Duals only
// rise while a side bids, so as long as the best listed value is at least that number the list
// decides the bid exactly as the whole line would; a line whose list has sunk below it is read whole.
//
// With lists the work of a phase is small (8 x CORE_LIST bytes a bid instead of 80,000) and what
// bounds it is the latency of dependent steps: bid -> evicted holder -> its bid, or one super-step
// of a shortest-path search after another.  So all the remaining phases run in ONE launch, on the
// workgroups of ONE die (XCD): what they share sits in that die's L2, where a load or an atomic
// takes about 0.1 us and a barrier over its 32 compute units 1 us (measured; across the eight dies
// 0.7 us and 4.4 us).  A chain step takes 1 us here instead of 4 us, a search super-step 2 us
// instead of 10 us, and nothing goes back to the host between them.
//
// While thousands of lines bid at once throughput counts instead: the proof and the first bids of a
// phase of a large problem run in launches over all dies, which hand over to one die once at most
// core_narrow lines bid and get it back for the next phase (two launches a phase more, about 50 us).
// The auction with all phases on one die / with such launches, mean over seeds: 2048 x 4096 3.6 / 3.9 ms,
// 4096 x 8192 5.7 / 6.1, 6001 x 9007 13.5 / 13.3, 8192 x 8192 8.8 / 8.1, 8192 x 12288 11.7 / 11.7,
// 12,000 x 16,000 29.8 / 26.6, 20,000 x 20,000 29.6 / 24.5; 20,000 x 40,000 with prefixes of a tenth
// 21.6 / 20.8.  The line is drawn at 8192 rows.
#include "scan.h"
#include "report.h"
#include "half_list.h"
#include "line_parts.h"
#include "list_cut.h"
#include "search_words.h"
#include "team_join.h"
#include "team_steps.h"

namespace {

constexpr int CORE_THREADS = 512;
constexpr int CORE_WAVES = CORE_THREADS / 64;
constexpr int CORE_LIST = MF_CORE_LIST;
static_assert(CORE_LIST == 128, "two entries per lane");
constexpr int CORE_PUSH_BUFFER = 4096;
constexpr int CORE_MAX_SOURCES = 64;
constexpr int CORE_MAX_WORKGROUPS = 1024;
constexpr int CORE_SLICE = 1024;                    // entries of a whole line one wavefront takes at a time
// Rounds a workgroup goes on by itself within a step of a search or a refinement, and rows it does so
// with at most (four for each of its wavefronts).  4 to 16 rounds measure the same within 3 %.
constexpr int CORE_OWN_ROUNDS = 10, CORE_OWN_MOST = 32;
constexpr int CORE_RESCANS = 4;                     // rows looked at once more for served trees, in lines of the side, before the lists are kept by column
constexpr unsigned long long CORE_INF = ~0ull;
constexpr unsigned CORE_IN_TREE = 0xffffffffu, CORE_READ = 1u;     // of a column, in a search: in the tree being served; its holder's line has been read whole
constexpr int CORE_NO_LABEL = INT32_MIN;
constexpr int CORE_JUMP_HOPS = 4, CORE_JUMP_PASSES = 48;
constexpr unsigned CORE_WAITING = 32;               // bidders waiting for better lists above which these are made
constexpr unsigned CORE_GAVE_UP = 0x80000000u;
// Looks at the word that says how many have joined before a workgroup takes those that have (see
// team_join.h): long enough for another context's longest kernel to make room.
constexpr unsigned CORE_JOIN_LOOKS = 1u << 16;
constexpr double CORE_FAR = 1.0e300;                  // no candidate
constexpr double CORE_WHOLE = 2.0e300;                // in CoreShared's remainder: the bidder's line has been read whole
constexpr double CORE_UNBOUNDED = -1.0e300;         // bound of a line whose list holds all of its entries

// ---------------------------------------------------------------- the lists

// The CORE_LIST entries with the largest K w - dual of every line, and what no other entry exceeds.
//
// What bounds it is reading the lines, once, four at a time so that a load of duals serves
// them all (as in round_kernel; one at a time where there are too few lines to fill the device so).  Which entries are kept on the way is decided by a cut taken from a sample of
// the line (LIST_SAMPLE_GROUPS groups, an eighth of a long line, in pieces of 128 bytes all along it): about LIST_AIM entries
// lie above it, they go to LDS, and the best CORE_LIST of those make the list.  Everything is in doubles,
// so the bound is exact; the cut only has to be near: with a few entries less than CORE_LIST above it the list is that
// much shorter, with more than LDS holds the line is read again with a cut from those that were kept.
// Entries tied with the cut fill the list up, whichever come first from a place that differs from group to group
// of lines (tied bidders would otherwise all hold the same few of many tied entries).
// A wavefront per line finds cut and list by bisection: counts come from ballots, no barrier in between.
//
// In the pass nearly every wavefront has a few entries to keep in every step, and looking at sixteen entries a lane exactly, and
// keeping each behind a branch and an atomic of its own, took 1.5 us a step where the loads take half of that.  So floats decide which
// entries are looked at exactly, a lane goes through its own few one after the other, and the next step's loads are on
// their way meanwhile.  One step a time: by twos four lines need more registers than four wavefronts a SIMD leave each (334 / 366 us for 20,000
// lines of 20,000).  Four are as many as LDS lets in with four lines; held to five, one line and two spill eight and twelve
// registers and take 1 to 3 % longer (1000 lines of 20,000 30.0 / 29.4 us, 2003 of 3001 23.6 / 22.9).
// (Lists of 20,000 lines of 20,000 entries: 926 us when a workgroup of 1024 threads kept a whole line in
// registers and found the cut by histograms, a dozen barriers a line; 400 us with every entry looked at exactly; 346 us now, 4.6 TB/s.  6500,
// 2500 and 1200 of them 155 -> 132, 78 -> 61 and 68 -> 42 us; 4096 lines of 8192 52 -> 45, 2003 of 3001 26 -> 24.
// One line a workgroup up to four a compute unit, two up to eight: 256 lines of 20,000 take 60 us by fours, 24 us so;
// 1200 46 by fours, 41 by twos; 4096 of 8192 entries 45 by fours, 54 by twos.  Aiming at 300 entries above the first cut, not 240: fewer
// lists fall short of CORE_LIST, more are looked at, 1 to 3 % longer: 1000 lines of 20,000 30.8 / 30.0, 1900
// 45.8 / 44.7, 4096 of 8192 45.4 / 44.6, 20,000 of 20,000 335 / 333.)
constexpr int LIST_THREADS = 256, LIST_CAP = 512, LIST_AIM = 240, LIST_SAMPLE_GROUPS = 512;

// Of the integers in v (PER a lane; `low`: unused), a cut with at most `most` of them above it, and at
// least `least` unless ties forbid it.  All lanes return the same.
template <int PER>
__device__ __forceinline__ double cut_above(const double (&v)[PER], int least, int most, double low)
{
    double top = low, bottom = 1.0e300;
#pragma unroll
    for (int q = 0; q < PER; ++q) { top = fmax(top, v[q]); if (v[q] > low) bottom = fmin(bottom, v[q]); }
    double hi = wave_max(top), lo = -wave_max(-bottom) - 1.0;
    while (hi - lo > 1.0) {
        const double mid = floor(0.5 * (lo + hi));
        int above = 0;
#pragma unroll
        for (int q = 0; q < PER; ++q) above += __popcll(__ballot(v[q] > mid));
        if (above > most) lo = mid;
        else { hi = mid; if (above >= least) break; }
    }
    return hi;
}

template <int LINES>                                    // lines a workgroup makes lists of, at most one a wavefront
__global__ __launch_bounds__(LIST_THREADS, 4) void core_list_kernel(
    const int32_t *__restrict__ A, long long pitch, int len, const int *__restrict__ line_len, int lines, int stride,
    const int *__restrict__ which, const double *__restrict__ dual, double Kd, int2 *__restrict__ entries,
    double *__restrict__ bound, double *__restrict__ half_bound, double *depth, const double *__restrict__ own_dual,
    const int *__restrict__ partner, double *__restrict__ built, int some, double most)
{
    // The duals the side's lists were made for; where some lines' lists are newer than others', the larger ones (a
    // bound holds as long as no dual is lower than when the list was made).  (A launch of its own took 5 us and its gap.)
    if (built)
        for (int k = blockIdx.x * LIST_THREADS + threadIdx.x; k < len; k += gridDim.x * LIST_THREADS) {
            const double d = dual[k];
            built[k] = some ? fmax(built[k], d) : d;
        }
    // line number q of this launch's `lines`: every stride-th, or the q-th listed in `which`
    auto line_number = [&](int q) { return which ? (long long)which[q] : (long long)q * stride; };
    constexpr int PER = LIST_CAP / 64;
    static_assert(LINES <= LIST_THREADS / 64, "a wavefront per line chooses");
    __shared__ double s_value[LINES][LIST_CAP];
    __shared__ int2 s_entry[LINES][LIST_CAP], s_tie[LINES][CORE_LIST];
    __shared__ int s_count[LINES], s_ties[LINES], s_again[LINES], s_to[LINES];
    __shared__ double s_cut[LINES];
    static_assert(LIST_CAP >= LIST_THREADS, "a sample's largest values, one a thread");
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int32_t *line[LINES];
    int to[LINES], longest = 0;
#pragma unroll
    for (int r = 0; r < LINES; ++r) {
        const int q = blockIdx.x * LINES + r;
        const bool have = q < lines;
        const long long b = have ? line_number(q) : 0;
        // a column nobody holds and that has no price will not bid soon: an empty list that says so (should
        // it bid before the lists are made again, it reads its whole line)
        const bool idle = have && partner && partner[b] < 0 && !(own_dual[b] > 0.0);
        line[r] = A + (size_t)b * pitch;
        to[r] = !have ? -1 : idle ? 0 : line_len ? min(line_len[b], len) : len;
        longest = max(longest, to[r]);
    }
    const int groups = (longest + 3) / 4;
    const int turn = groups > 0 ? (int)((blockIdx.x * 2654435761u >> 8) % (unsigned)groups) : 0;
    auto value_of = [&](int r, int j, int32_t w, double p) { return j < to[r] && w != MF_INFEASIBLE ? fma(Kd, (double)w, -p) : LIST_ALL; };
    // ---- the sample: each thread's best of up to two groups ----
    const int pieces = min(groups / 8, LIST_SAMPLE_GROUPS / 8);         // of eight groups
    const bool sampled = longest > LIST_CAP;
    int looked = 0;                                                     // groups looked at, one or two a thread
    if (sampled) {
        double best[LINES];
#pragma unroll
        for (int r = 0; r < LINES; ++r) best[r] = LIST_ALL;
#pragma unroll
        for (int q = 0; q < LIST_SAMPLE_GROUPS / LIST_THREADS; ++q) {
            const int piece = (q * LIST_THREADS + tid) >> 3;
            if (piece < pieces) {
                const int g = (int)((long long)piece * groups / pieces) + (tid & 7);
                const double2 p01 = *(const double2 *)(dual + g * 4);
                const double2 p23 = *(const double2 *)(dual + g * 4 + 2);
#pragma unroll
                for (int r = 0; r < LINES; ++r) {
                    const int4 w = *(const int4 *)(line[r] + g * 4);
                    best[r] = fmax(best[r], fmax(fmax(value_of(r, g * 4, w.x, p01.x), value_of(r, g * 4 + 1, w.y, p01.y)),
                                                 fmax(value_of(r, g * 4 + 2, w.z, p23.x), value_of(r, g * 4 + 3, w.w, p23.y))));
                }
            }
        }
        looked = pieces * 8;
#pragma unroll
        for (int r = 0; r < LINES; ++r) s_value[r][tid] = best[r];
        __syncthreads();
    }
    const bool choosing = wave < LINES;                                 // this wavefront has a line to choose for
    {
        double cut = LIST_NONE;
        int mine = -1;
#pragma unroll
        for (int r = 0; r < LINES; ++r) if (r == wave) mine = to[r];
        if (mine > 0 && (!sampled || mine <= LIST_CAP)) cut = LIST_ALL;
        else if (mine > 0) {
            double v[LIST_THREADS / 64];
            int feasible = 0;
#pragma unroll
            for (int q = 0; q < LIST_THREADS / 64; ++q) { v[q] = s_value[wave][q * 64 + lane]; feasible += __popcll(__ballot(v[q] > LIST_ALL)); }
            // LIST_AIM of the line's entries are above the cut that so many of the sample's parts have an entry above
            const int parts = min(min(looked, LIST_THREADS), max(1, (int)((long long)looked * mine / longest)));
            const float each = 4.0f * (float)looked / (float)min(looked, LIST_THREADS), share = fminf(1.0f, (float)LIST_AIM / (float)mine);
            const int want = max(1, (int)(parts * (1.0f - powf(1.0f - share, each))));
            cut = feasible <= want ? LIST_ALL : cut_above(v, want - want / 16, want, LIST_ALL);
        }
        __syncthreads();
        if (choosing && lane == 0) { s_cut[wave] = cut; s_count[wave] = 0; s_ties[wave] = 0; s_to[wave] = mine; }
        __syncthreads();
    }
    // ---- every line, once ----
    // (floats tell what has to be looked at exactly: list_cut.h)
    float cut_f[LINES];
#pragma unroll
    for (int r = 0; r < LINES; ++r) cut_f[r] = cut_in_floats(s_cut[r], most);
    const float kf = (float)Kd;                                         // (exact: K is at most 2^20)
    for (int attempt = 0;; ++attempt) {
        // (the next groups are on their way while these are looked at: the compiler moves no load past a branch that may keep an entry)
        int4 w[LINES], w_next[LINES];
        double2 p01, p23, p01_next, p23_next;
        auto fetch = [&](int g0, int4 (&w)[LINES], double2 &p01, double2 &p23) {
            const int g = g0 + turn >= groups ? g0 + turn - groups : g0 + turn, j = g * 4;
#pragma unroll
            for (int r = 0; r < LINES; ++r) w[r] = *(const int4 *)(line[r] + j);      // (lines are padded to a multiple of four)
            p01 = *(const double2 *)(dual + j);
            p23 = *(const double2 *)(dual + j + 2);
        };
        if (tid < groups) fetch(tid, w_next, p01_next, p23_next);
#pragma unroll 1
        for (int g0 = tid; g0 < groups; g0 += LIST_THREADS) {
            const int g = g0 + turn >= groups ? g0 + turn - groups : g0 + turn, j = g * 4;
#pragma unroll
            for (int r = 0; r < LINES; ++r) w[r] = w_next[r];
            p01 = p01_next; p23 = p23_next;
            if (g0 + LIST_THREADS < groups) fetch(g0 + LIST_THREADS, w_next, p01_next, p23_next);
            // Floats tell what may be above the cut, or at it; only that is looked at exactly.
            const float p[4] = {(float)p01.x, (float)p01.y, (float)p23.x, (float)p23.y};
            unsigned hits = 0u;
#pragma unroll
            for (int r = 0; r < LINES; ++r) {
                const int32_t we[4] = {w[r].x, w[r].y, w[r].z, w[r].w};
#pragma unroll
                for (int e = 0; e < 4; ++e) hits |= may_reach(kf, we[e], p[e], cut_f[r]) ? 1u << (4 * r + e) : 0u;
            }
            while (hits) {
                const int bit = __ffs((int)hits) - 1, r = bit >> 2, e = bit & 3;
                hits &= hits - 1u;
                int4 of = w[0];
#pragma unroll
                for (int q = 1; q < LINES; ++q)
                    if (r == q) of = w[q];
                const int32_t we = e == 0 ? of.x : e == 1 ? of.y : e == 2 ? of.z : of.w;
                const double v = fma(Kd, (double)we, -(e == 0 ? p01.x : e == 1 ? p01.y : e == 2 ? p23.x : p23.y)), line_cut = s_cut[r];
                if (we == MF_INFEASIBLE || j + e >= s_to[r] || v < line_cut) continue;
                if (v > line_cut) {
                    const int at = atomicAdd(&s_count[r], 1);
                    if (at < LIST_CAP) { s_value[r][at] = v; s_entry[r][at] = make_int2(j + e, we); }
                } else if (s_ties[r] < CORE_LIST) {
                    const int at = atomicAdd(&s_ties[r], 1);
                    if (at < CORE_LIST) s_tie[r][at] = make_int2(j + e, we);
                }
            }
        }
        __syncthreads();
        // more than LDS holds: once more, for these lines only
        const int found = choosing ? s_count[wave] : 0;
        const bool again = found > LIST_CAP && attempt < 4;
        double higher = LIST_NONE;
        if (again) {
            double v[PER];
#pragma unroll
            for (int q = 0; q < PER; ++q) v[q] = s_value[wave][q * 64 + lane];
            const int want = max(1, (int)((long long)LIST_AIM * LIST_CAP / found));
            higher = cut_above(v, want - want / 16, want, LIST_ALL);
        }
        if (choosing && lane == 0) s_again[wave] = again;
        __syncthreads();
        if (again && lane == 0) { s_cut[wave] = higher; s_count[wave] = 0; s_ties[wave] = 0; }
        bool any = false;
#pragma unroll
        for (int r = 0; r < LINES; ++r) any |= s_again[r] != 0;
        __syncthreads();
        if (!any) break;
#pragma unroll
        for (int r = 0; r < LINES; ++r) cut_f[r] = cut_in_floats(s_again[r] ? s_cut[r] : LIST_NONE, most);
    }
    // ---- a wavefront per line ----
    const int number = blockIdx.x * LINES + wave;
    if (!choosing || number >= lines) return;
    const long long b = line_number(number);
    int2 *out = entries + (size_t)b * CORE_LIST;
    int mine = 0;
#pragma unroll
    for (int r = 0; r < LINES; ++r) if (r == wave) mine = to[r];
    const bool idle = partner && partner[b] < 0 && !(own_dual[b] > 0.0);
    const int found = s_count[wave], have = min(found, LIST_CAP);
    const double line_cut = s_cut[wave];
    double v[PER], best = LIST_ALL;
#pragma unroll
    for (int q = 0; q < PER; ++q) { v[q] = q * 64 + lane < have ? s_value[wave][q * 64 + lane] : LIST_ALL; best = fmax(best, v[q]); }
    const double chosen_above = have > CORE_LIST ? cut_above(v, CORE_LIST - 4, CORE_LIST, LIST_ALL) : LIST_ALL;
    // the best half of them comes first (a bid looks at the rest only if that does not decide it)
    constexpr int HALF = CORE_LIST / 2;
    const double half_above = have > HALF ? cut_above(v, HALF - 4, HALF, LIST_ALL) : LIST_ALL;
    int used = 0;
    double past = LIST_ALL, past_half = LIST_ALL;                       // the best that is not on the list, not in its first half
    const unsigned long long below = (1ull << lane) - 1ull;
    auto put = [&](bool mine, double worth, int2 entry) {               // what there is no room for is `past`
        const unsigned long long in = __ballot(mine);
        const int at = used + __popcll(in & below);
        if (mine && at < CORE_LIST) out[at] = entry;
        if (mine && at >= CORE_LIST) past = fmax(past, worth);
        if (mine && at >= HALF) past_half = fmax(past_half, worth);
        used = min(CORE_LIST, used + __popcll(in));
    };
#pragma unroll
    for (int q = 0; q < PER; ++q) put(v[q] > half_above, v[q], s_entry[wave][q * 64 + lane]);
#pragma unroll
    for (int q = 0; q < PER; ++q) put(v[q] > chosen_above && v[q] <= half_above, v[q], s_entry[wave][q * 64 + lane]);
    // ... and of those at the cut as many as there is room for
#pragma unroll
    for (int q = 0; q < PER; ++q) {
        put(v[q] > LIST_ALL && v[q] == chosen_above, v[q], s_entry[wave][q * 64 + lane]);
        if (v[q] < chosen_above) past = fmax(past, v[q]);
    }
    if (found <= CORE_LIST) {
        const int ties = min(s_ties[wave], CORE_LIST);
        for (int t = 0; t < ties; t += 64) put(t + lane < ties, line_cut, s_tie[wave][min(t + lane, CORE_LIST - 1)]);
        if (ties > 0) best = fmax(best, line_cut);
    }
    for (int t = used + lane; t < CORE_LIST; t += 64) out[t] = make_int2(0, MF_INFEASIBLE);
    best = wave_max(best);
    past = wave_max(past);
    past_half = wave_max(past_half);
    // (what did not reach the cut may be worth as much; what LDS had no room for after five readings, as much as the best)
    if (mine > 0 && line_cut > LIST_ALL) past = fmax(past, line_cut);
    if (found > LIST_CAP) past = CORE_FAR;
    past_half = fmax(past_half, past);
    if (lane == 0) {
        const bool all = past == LIST_ALL;
        bound[b] = idle ? CORE_FAR : all ? CORE_UNBOUNDED : past;
        half_bound[b] = idle ? CORE_FAR : past_half == LIST_ALL ? CORE_UNBOUNDED : past_half;
        depth[which ? b : (long long)number] = idle ? 0.0 : all ? 1.0e13 : fmax(best - past, 0.0);
    }
}

// ---------------------------------------------------------------- the engine

struct CoreReport {
    int reason, phase, stage, count, parity, columns_wait;
    unsigned columns_ready;
    unsigned long long bids, depth, steps, scans, whole_groups, rested;      // (whole_groups: of four entries, of lines read whole)
};
static_assert(sizeof(CoreReport) % 8 == 0, "told in words");

struct alignas(256) CoreCtl {
    // who takes part: the workgroups of the die the first one to arrive runs on
    int die;
    unsigned joined, arrived, members;                   // (see team_join.h)
    // barriers each workgroup has reached (top bit: it gave up); one lane polls each
    alignas(256) unsigned reached[CORE_MAX_WORKGROUPS];
    // rings by step (team_steps.h), clear when the launch begins
    alignas(128) int cnt[STEP_RING];                     // bidders handed on
    int whole_count[STEP_RING];                          // rows whose whole lines a refinement looks at next
    unsigned dense[STEP_RING];                           // whole lines read in a step
    alignas(128) unsigned long long slack[3];            // see slack_of: bits of a non-negative double, two means
    int rev_count, tree_count, read_count;
    unsigned long long rescans;                          // rows looked at once more for a served tree's columns, this search
    // searches
    // (read together, a lane each: [0..2] lowest label left per slot, [3..5] path ends found, [6..8] frontier lengths, [9] sink, [10..12] lines to be read whole)
    alignas(128) unsigned long long low[3];
    unsigned long long sink_found[3], frontier[3], sink, whole_front[3];
    alignas(128) unsigned long long src_profit[CORE_MAX_SOURCES], src_outside[CORE_MAX_SOURCES], src_dropped[CORE_MAX_SOURCES], src_left[CORE_MAX_SOURCES];
    alignas(128) unsigned jump_pending[CORE_JUMP_PASSES + 1];
    // refinement
    alignas(128) unsigned failed[3];
    unsigned told;                                       // the launch has told the host itself how it ended
    // what the launch reports (phase -1: it did not get to one)
    alignas(128) CoreReport out;
};

struct CoreSide {
    const int32_t *A;                   // the bidding side's lines
    long long pitch;
    int lines, len;                     // how many, how long
    long long read_limit;               // lines one search may read whole
    const int *line_len;                // optional
    unsigned long long *otherword;      // opposite (dual, holder) words
    double *other_dual;                 // the same duals, brought up to date at the end of a side
    const int2 *entries;
    int *t_start, *t_at;                // the lists by opposite line: where each one's entries start (and, while they are made, end)
    int2 *t_entries;                    // (line, weight)
    const double *bound, *half_bound, *built, *reach;    // built: the opposite duals when the lists were made; reach: from a line's best entry to its bound
};

struct CoreArgs {
    CoreSide side[2];                   // 0: rows bid, 1: columns bid
    double Kd;
    int n_phases, first_phase, first_stage, first_count, first_parity;
    double eps[MF_CORE_PHASES];
    int stop[MF_CORE_PHASES], stop_grown[MF_CORE_PHASES];   // bidders that may be left over (second: while few have given up)
    int growth_rest;
    unsigned long long rested_before;
    int have_columns;                   // the lists of side 1 exist
    int may_refine;
    unsigned columns_ready;
    int columns_wait;                    // where the launch begins with columns that bid: they may be left to the next phase (side_end.h)
    double stale_rise;
    double stale;                       // epsilons a dual may have come down since the lists were made before they are made again
    int refine_rounds, refine_patience; // rounds in all; rounds without a new least number of rows left
    int refined;                     // refined: a launch before this one has begun the refinement it starts with
    double refine_lower;
    double refine_below;                // epsilon at or below which a complete phase is followed by a refinement
    int path_max;
    long long path_after, tail_steps;
    int tail_always;                    // of a side on which columns have to come down, too (side_end.h)
    int steps_many, steps_few;
    double path_width;
    int frontier_high;
    unsigned spin_limit;
    int workgroups;
    int wide, use_wide;                 // this launch spans all dies; such launches do the wide parts
    int narrow_at;
    int dense_limit;
    int frontier_room;
    double bid_limit;
    void *tell_to; unsigned *told, number;               // where the host looks for the report, and the report's number
    int *row2col, *col2row, *tree;
    unsigned long long *rowword;        // == side[1].otherword
    int *list0, *list1;
    // searches and refinement
    unsigned long long *label, *expanded, *frontier0, *frontier1;
    unsigned *stamp;
    int *held, *jump;
    unsigned long long *parent;
    double *base;                       // [lines] of a line that has been scanned: length of its path + its profit + eps; else CORE_FAR
    double *dropped;                    // [columns] the shortest candidate the holder's scan left out because it lay beyond every path end
    unsigned long long *read_from;      // [columns] label from which the holder's line has been read whole, else CORE_INF
    double *left;                       // [columns] ... and the nearest entry that left out
    int *whole0, *whole1;               // lines to be read whole (by step parity)
    int32_t *held_weight;               // [max(rows, columns)] weight of each opposite line's pair with its holder
};

struct CoreShared {
    unsigned long long list[CORE_PUSH_BUFFER];
    double profit[CORE_MAX_SOURCES], remainder[CORE_MAX_SOURCES], outside[CORE_MAX_SOURCES];
    int row[CORE_MAX_SOURCES], alive[CORE_MAX_SOURCES];
    Top2 part[CORE_WAVES];
    unsigned pushes, base;
    unsigned long long sink, low, served;      // served: length of the search's last path
    int n_alive, ok, dense, columns_wait;
    unsigned failed;
};

__device__ __forceinline__ unsigned die_number()
{
    return (unsigned)__builtin_amdgcn_s_getreg((31 << 11) | 20) & 0xfu;     // XCC_ID
}

__device__ __forceinline__ int load_fresh_i32(const int *p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ __forceinline__ void store_i32(int *p, int v) { __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ __forceinline__ void store_u32(unsigned *p, unsigned v) { __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ __forceinline__ void store_f64(double *p, double v) { store_through((unsigned long long *)p, (unsigned long long)__double_as_longlong(v)); }

struct TeamMemory {
    __device__ __forceinline__ unsigned load(const unsigned *p) const { return load_fresh_u32(p); }
    __device__ __forceinline__ void store(unsigned *p, unsigned v) const { store_u32(p, v); }
    __device__ __forceinline__ unsigned add(unsigned *p, unsigned v) const { return atomicAdd(p, v); }
    __device__ __forceinline__ unsigned set_bits(unsigned *p, unsigned v) const { return atomicOr(p, v); }
    __device__ __forceinline__ int swap_if(int *p, int from, int to) const { return atomicCAS(p, from, to); }
    __device__ __forceinline__ void settle() const { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }
};

struct WaveLanes {                      // for half_list.h: a value a lane
    typedef double Values;
    typedef int Keys;
    __device__ __forceinline__ int keys(double v, double outside) const { return __float_as_int((float)fmax(v - outside, 0.0)); }
    __device__ __forceinline__ double distance(int key) const { return (double)__int_as_float(key); }
    __device__ __forceinline__ int largest(int key) const { return wave_max(key); }
    __device__ __forceinline__ unsigned long long equal(int key, int to) const { return __ballot(key == to); }
    __device__ __forceinline__ bool in(unsigned long long lanes) const { return (lanes >> (threadIdx.x & 63u)) & 1ull; }
    __device__ __forceinline__ double largest_among(double v, unsigned long long lanes) const { return wave_max(in(lanes) ? v : NEG_HUGE); }
    __device__ __forceinline__ unsigned long long equal_among(double v, double to, unsigned long long lanes) const { return __ballot(v == to) & lanes; }
    __device__ __forceinline__ int without(int key, int lane) const { return (int)(threadIdx.x & 63u) == lane ? 0 : key; }
    __device__ __forceinline__ double at(double v, int lane) const
    {
        return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), lane), __builtin_amdgcn_readlane(__double2loint(v), lane));
    }
};

struct SharedWords {                    // (the bits of doubles that are not negative are in the doubles' order)
    __device__ __forceinline__ void set(unsigned long long *p, unsigned long long v) const { store_through(p, v); }
    __device__ __forceinline__ void set(double *p, double v) const { store_f64(p, v); }
    __device__ __forceinline__ void lower(unsigned long long *p, unsigned long long v) const { atomicMin(p, v); }
    __device__ __forceinline__ void lower(double *p, double v) const { atomicMin((unsigned long long *)p, (unsigned long long)__double_as_longlong(fmax(v, 0.0))); }
};

// Best and second-best value of a whole line against the current words (one wavefront).  Out of
// line and with nothing but values passed: rare, and its registers would be the callers' otherwise.
// share, shares: every so many-th stretch of 256 entries only, where several wavefronts read a line together
__device__ __noinline__ Top2 read_whole_line(const int32_t *line, int to, const unsigned long long *words, double Kd, int salt, int share, int shares)
{
    const int lane = threadIdx.x & 63;
    Top2 t{NEG_HUGE, NEG_HUGE, 0x7fffffff, 0};
#pragma unroll 2
    for (int j = share * 256 + lane * 4; j < to; j += shares * 256) {
        const int4 w4 = *(const int4 *)(line + j);
        const int32_t w[4] = {w4.x, w4.y, w4.z, w4.w};
        double v[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const double p = word_dual(load_fresh_u64(&words[min(j + e, to - 1)]));
            v[e] = j + e < to ? fma(Kd, (double)w[e], -p) : NEG_HUGE;
        }
        top2_push4(t.b1, t.b2, t.idx, t.w, v[0], v[1], v[2], v[3], j, w4, salt);
    }
    t = wave_top2(t);
    t.idx ^= salt;
    return t;
}

// The same of a whole list (out of line for the same reason: nine bids in ten are decided by its first half).
__device__ __noinline__ Top2 read_list(const int2 *e, const unsigned long long *words, double Kd, int salt)
{
    const int lane = threadIdx.x & 63;
    const int2 e0 = e[lane], e1 = e[lane + 64];
    const unsigned long long w0 = load_fresh_u64(&words[e0.x]), w1 = load_fresh_u64(&words[e1.x]);
    const double v0 = fma(Kd, (double)e0.y, -word_dual(w0)), v1 = fma(Kd, (double)e1.y, -word_dual(w1));
    const bool first = v0 >= v1;
    const double hi = fmax(v0, v1), lo = fmin(v0, v1);
    Top2 t;
    t.b1 = wave_max(hi);
    const unsigned long long hit = __ballot(hi == t.b1);
    // among tied lanes the first at or after a lane that depends on the bidder
    const unsigned turn = (unsigned)salt & 63u;
    const unsigned long long turned = hit & (~0ull << turn);
    const int src = __ffsll((long long)(turned ? turned : hit)) - 1;
    t.b2 = wave_max(lane == src ? lo : hi);
    t.idx = __builtin_amdgcn_readlane(first ? e0.x : e1.x, src);
    t.w = __builtin_amdgcn_readlane(first ? e0.y : e1.y, src);
    return t;
}

// A bid on a whole line that all of a workgroup reads; returns, in its first lane, who has to bid next, -1 or (in all of the first wavefront)
// RESTS.  Out of line like read_whole_line.
constexpr int RESTS = -2;
__device__ __noinline__ int bid_by_workgroup(const int32_t *line, int to, unsigned long long *words, double Kd, int b, double eps, Top2 *part)
{
    const int wave = (int)threadIdx.x >> 6;
    Top2 t = read_whole_line(line, to, words, Kd, tie_salt(b), wave, CORE_WAVES);
    if ((threadIdx.x & 63) == 0) part[wave] = t;
    __syncthreads();
    int next = -1;
    if (wave == 0) {
        for (int w = 1; w < CORE_WAVES; ++w) top2_merge(t, part[w]);
        if (t.b1 <= eps) next = RESTS;
        else if (threadIdx.x == 0) {
            const unsigned long long mine = pack_word(Kd * (double)t.w - fmax(t.b2 - eps, 0.0), b + 1);
            const unsigned long long old = atomicMax(&words[t.idx], mine);
            next = old < mine ? word_id(old) : b;
        }
    }
    __syncthreads();
    return next;
}

// (out of line: rare, and a dozen divisions)
__device__ __noinline__ int parts_out_of_line(int slices, int lines, int waves, bool prefixes) { return parts_of_line(slices, lines, waves, prefixes); }

// One wavefront.  The host is told by the launch itself, not by the one behind it, and decides while this one ends and that one
// clears the control block.  Being a function of its own it also ends the kernel's vector spills (51 in either instance before).  Rounds of
// 777 x 1501 1.67 -> 1.64 ms, 1024 x 1024 2.07 -> 2.00, 3001 x 2003 4.05 -> 3.97, 4096 x 8192 6.37 -> 6.25, 20,000 x 20,000 39.6 -> 38.8.
__device__ __noinline__ void tell_host(CoreCtl *ctl, void *to, unsigned *told, unsigned number)
{
    const int lane = threadIdx.x & 63;
    if (lane == 0) ctl->told = 1u;
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    static_assert(sizeof(CoreReport) <= 256, "a word a lane");
    if (lane < (int)(sizeof(CoreReport) / 4))
        __hip_atomic_store((unsigned *)to + lane, load_fresh_u32((const unsigned *)&ctl->out + lane), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");         // what has been stored is there before the number is
    if (lane == 0) __hip_atomic_store(told, number, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

// Everything a workgroup carries through the launch.  LARGE: for problems whose first bids run on all dies, where
// bidders may wait for better lists.  (Those few instructions cost a chain's step 3 % where one die does it all.)
template <bool LARGE>
struct Core {
    const CoreArgs &a;
    CoreCtl *ctl;
    CoreShared &sh;
    unsigned G, rank;
    unsigned generation, columns_ready;     // columns_ready: the sides whose lists exist by column (bits)
    unsigned epoch;                         // the step the launch is at: never set back (team_steps.h)
    int tid, lane, wave;
    unsigned bids, depth, steps, scans, whole, rests;          // this wavefront's counts

    __device__ Core(const CoreArgs &args, CoreCtl *c, CoreShared &s)
        : a(args), ctl(c), sh(s), G(1), rank(0), generation(0), columns_ready(args.columns_ready), epoch((unsigned)args.first_parity), tid(threadIdx.x), lane(threadIdx.x & 63),
          wave(__builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6)), bids(0), depth(0), steps(0), scans(0), whole(0), rests(0) {}

    __device__ int gtid() const { return (int)rank * CORE_THREADS + tid; }
    __device__ int gsize() const { return (int)G * CORE_THREADS; }
    // (dealt out over the compute units first: a scan's gathers are bound by one unit's request rate)
    __device__ int gwave() const { return wave * (int)G + (int)rank; }
    __device__ int gwaves() const { return (int)G * CORE_WAVES; }

    // Barrier over the participating workgroups: each stores the barrier's number in a slot of its
    // own, and one wavefront polls all the slots, a lane each.  (A store and a load of L2 take 0.1 us
    // each, a read-modify-write 0.27 us and the next one on the same address waits for it: counting
    // arrivals took 1.0 us.)  Every wait is bounded; whoever's runs out says so in its slot and
    // everybody leaves.
    __device__ __forceinline__ bool barrier()
    {
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
        ++generation;
        if (G == 1u && a.spin_limit > 0u) return true;
        if (tid < 64) {
            if (lane == 0) store_u32(&ctl->reached[rank], generation);
            unsigned spins = 0;
            bool ok = true;
            for (;;) {
                unsigned least = generation, any = 0u;
                for (unsigned g = lane; g < G; g += 64u) {
                    const unsigned seen = load_fresh_u32(&ctl->reached[g]);
                    least = min(least, seen);
                    any |= seen;
                }
                if (__any(any & CORE_GAVE_UP)) { ok = false; break; }
                if (__all(least >= generation)) break;
                if (++spins > a.spin_limit) { ok = false; break; }
            }
            if (lane == 0) {
                if (!ok) store_u32(&ctl->reached[rank], CORE_GAVE_UP);
                sh.ok = ok ? 1 : 0;
            }
        }
        __syncthreads();
        return sh.ok != 0;
    }

    // The workgroups of one die (with `wide`: of all dies) find each other, at most `workgroups` of
    // them; the others leave.
    // Returns 0 (not one of them), 1, or -1 (a wait ran out).
    __device__ __forceinline__ int join()
    {
        if (tid == 0) {
            unsigned number, members = 1u;
            const int ok = join_team(TeamMemory{}, TeamWords{&ctl->die, &ctl->joined, &ctl->arrived, &ctl->members}, (int)die_number(),
                                     a.wide != 0, gridDim.x, (unsigned)a.workgroups, CORE_JOIN_LOOKS, a.spin_limit, &number, &members);
            if (ok == -2) store_u32(&ctl->reached[number], CORE_GAVE_UP);
            sh.n_alive = (int)number;
            sh.base = members;
            sh.ok = ok >= 0 ? 1 : ok + 1;
        }
        __syncthreads();
        const int ok = sh.ok;
        if (ok == 1) { rank = (unsigned)sh.n_alive; G = sh.base; }
        __syncthreads();
        return ok;
    }

    // ---------------- bids ----------------

    __device__ __forceinline__ Top2 whole_line(const CoreSide &s, int b)
    {
        const int to = s.line_len ? min(s.line_len[b], s.len) : s.len;
        whole += (unsigned)(to + 3) / 4u;
        return read_whole_line(s.A + (size_t)b * s.pitch, to, s.otherword, a.Kd, tie_salt(b), 0, 1);
    }

    // a slice of a line, all of it in flight (lines are padded to a multiple of four)
    __device__ __forceinline__ void load_slice(const int32_t *line, int from, int to, int4 *ahead)
    {
#pragma unroll
        for (int q = 0; q < CORE_SLICE / 256; ++q) {
            const int j = from + q * 256 + lane * 4;
            ahead[q] = j < to ? *(const int4 *)(line + j) : make_int4(MF_INFEASIBLE, MF_INFEASIBLE, MF_INFEASIBLE, MF_INFEASIBLE);
        }
    }

    // Wavefronts that read a line together, each every so many-th slice of it
    __device__ __forceinline__ int parts_of(const CoreSide &s, int lines) const
    {
        return parts_out_of_line((s.len + CORE_SLICE - 1) / CORE_SLICE, lines, gwaves(), s.line_len != nullptr);
    }

    // The best half of a line's list, a lane an entry, and what nothing else is worth more than.
    struct Half { int2 e; double bound; };
    __device__ __forceinline__ Half half_of(const CoreSide &s, int b) const
    {
        return Half{s.entries[(size_t)b * CORE_LIST + lane], s.half_bound[b]};
    }

    // Best and second-best value of b's whole list; *outside: what no unlisted entry exceeds
    __device__ __forceinline__ Top2 listed(const CoreSide &s, int b, double slack, double *outside) const
    {
        *outside = s.bound[b] + slack;
        return read_list(s.entries + (size_t)b * CORE_LIST, s.otherword, a.Kd, tie_salt(b));
    }

    // One bid of bidder b by this wavefront; returns who has to bid next because of it, or -1, with the first half of
    // that one's list in h.  What bounds hundreds of chains is how many words a die's L2 hands out (every entry's
    // is a request of its own: 256 wavefronts ask for 32,768 a step, 16 channels serve one each a cycle), what
    // bounds a few is the chain of dependent trips: list 0.13 us, words 0.13, bid 0.37.  So the better half of the list
    // is looked at alone first, and decides if its two best are both worth more than anything else can be
    // (nine bids in ten); and who will be evicted is known from the words, before the bid is made, unless
    // another wavefront gets in between: his list is on its way while the bid is.  The first bids of a 20,000 x
    // 20,000 phase 236 -> 187 us, its last 570 bidders 820 -> 627 us; a matching 15.3 -> 14.5 ms, next round 24.2 -> 23.3.
    // The two best are found as half_list.h says.
    // waiting: if it is -1 a bidder whose whole list no longer decides does not have his line read here but goes there.
    __device__ __forceinline__ int bid(const CoreSide &s, int b, Half &h, double eps, double slack, bool count_rests, int &waiting)
    {
        double outside = fmax(h.bound + slack, 0.0);        // (what is worth nothing is not bid for and holds no bid down)
        const unsigned long long word = load_fresh_u64(&s.otherword[h.e.x]);
        ++bids;
        const double v = fma(a.Kd, (double)h.e.y, -word_dual(word));
        const WaveLanes lanes;
        const int key = lanes.keys(v, outside);
        int top, second;
        const int src = best_lane(lanes, v, key, (unsigned)tie_salt(b) & 63u, &top);
        int guess = __builtin_amdgcn_readlane(word_id(word), src);
        Half ahead = h;
        if (guess >= 0) ahead = half_of(s, guess);
        Top2 t;
        t.b1 = lanes.at(v, src);
        t.idx = __builtin_amdgcn_readlane(h.e.x, src);
        t.w = __builtin_amdgcn_readlane(h.e.y, src);
        t.b2 = next_value(lanes, v, key, src, outside, &second);
        if ((top == 0 || second == 0) && outside > 0.0) {
            guess = -1;
            t = listed(s, b, slack, &outside);
            if (t.b1 < outside) {                           // the list no longer decides
                if (LARGE && waiting == -1) {
                    if (lane == 0) atomicAdd(&sh.dense, 1);
                    --bids;
                    waiting = b;
                    return -1;
                }
                t = whole_line(s, b);
                outside = NEG_HUGE;
                if (lane == 0) atomicAdd(&sh.dense, 1);
            }
        }
        if (t.b1 <= eps) {
            if (count_rests) ++rests;
            return -1;
        }
        int next = 0;
        if (lane == 0) {
            const double keep = fmax(fmax(t.b2, outside) - eps, 0.0);
            const unsigned long long mine = pack_word(a.Kd * (double)t.w - keep, b + 1);
            const unsigned long long old = atomicMax(&s.otherword[t.idx], mine);
            next = old < mine ? word_id(old) : b;
        }
        next = __builtin_amdgcn_readfirstlane(next);
        if (next >= 0 && next != b) h = next == guess ? ahead : half_of(s, next);
        return next;
    }

    // The same for a bidder whose line has to be read whole, by all of the workgroup: a wavefront alone takes 0.15 ms for a line of
    // 20,000, and the step lasts as long as the slowest.  Returns, in the first lane, who has to bid next.
    __device__ __forceinline__ int bid_on_whole_line(const CoreSide &s, int b, double eps, bool count_rests)
    {
        const int to = s.line_len ? min(s.line_len[b], s.len) : s.len;
        const int next = bid_by_workgroup(s.A + (size_t)b * s.pitch, to, s.otherword, a.Kd, b, eps, sh.part);
        if (wave == 0) {
            ++bids;
            whole += (unsigned)(to + 3) / 4u;
            if (next == RESTS && count_rests) ++rests;
        }
        return next;
    }

    // hands a bidder on to the next epoch (called by one lane)
    __device__ __forceinline__ void push(int b, int *next, int *counter)
    {
        const unsigned slot = atomicAdd(&sh.pushes, 1u);
        if (slot < (unsigned)CORE_PUSH_BUFFER) sh.list[slot] = (unsigned long long)(unsigned)b;
        else store_i32(&next[atomicAdd(counter, 1)], b);
    }
    __device__ __forceinline__ void flush(int *next, int *counter)
    {
        __syncthreads();
        const unsigned mine = min(sh.pushes, (unsigned)CORE_PUSH_BUFFER);
        if (tid == 0) sh.base = mine ? (unsigned)atomicAdd(counter, (int)mine) : 0u;
        __syncthreads();
        for (unsigned t = tid; t < mine; t += CORE_THREADS) store_i32(&next[sh.base + t], (int)sh.list[t]);
    }

    // The same without a place in `next` for more than one of each: lines kept may be there twice.
    __device__ __forceinline__ bool keep(int b)
    {
        const unsigned slot = atomicAdd(&sh.pushes, 1u);
        if (slot < (unsigned)CORE_PUSH_BUFFER) sh.list[slot] = (unsigned long long)(unsigned)b;
        return slot < (unsigned)CORE_PUSH_BUFFER;
    }
    __device__ __forceinline__ void hand_on(int *next, int *counter, unsigned from, unsigned mark)
    {
        __syncthreads();
        const unsigned to = min(sh.pushes, (unsigned)CORE_PUSH_BUFFER);
        for (unsigned t0 = from + wave * 64; t0 < to; t0 += CORE_THREADS) {
            const unsigned t = t0 + lane;
            const int b = t < to ? (int)sh.list[t] : 0;
            const bool first = t < to && atomicExch(&a.stamp[b], mark) != mark;
            const unsigned long long all = __ballot(first);
            if (!all) continue;
            int at = 0;
            if (lane == 0) at = atomicAdd(counter, __popcll(all));
            at = __builtin_amdgcn_readfirstlane(at);
            if (first) store_i32(&next[at + __popcll(all & ((1ull << lane) - 1ull))], b);
        }
    }

    // The most any opposite dual has come down since the side's lists were made (a list's bound holds
    // for entries that were worth so much less then).  ok: false when a wait ran out.  *stale: the duals
    // have risen, on average, by a good part of what the lists reach below their best entries, so
    // that many of them are about to stop deciding bids.
    __device__ __forceinline__ double slack_of(const CoreSide &s, bool &ok, bool *stale)
    {
        if (gtid() < 3) store_through(&ctl->slack[gtid()], 0ull);      // (every stage has a barrier after its last reading of these)
        ok = barrier();
        if (!ok) return 0.0;
        double most = 0.0, rise = 0.0, reach = 0.0;
        for (int k = gtid(); k < s.len; k += gsize()) {
            const double d = s.built[k] - word_dual(load_fresh_u64(&s.otherword[k]));
            most = fmax(most, d);
            rise -= d;
        }
        for (int i = gtid(); i < s.lines; i += gsize()) reach += s.reach[i];
        most = wave_max(most);
        for (int off = 32; off >= 1; off >>= 1) { rise += __shfl_xor(rise, off); reach += __shfl_xor(reach, off); }
        // (one workgroup's share at a time: atomics on one address complete at one per 10 ns, and 2048 wavefronts' took 25 us,
        // 256 wavefronts' 8 us)
        double *part = (double *)sh.list;
        __syncthreads();
        if (lane == 0) { part[wave] = most; part[CORE_WAVES + wave] = rise; part[2 * CORE_WAVES + wave] = reach; }
        __syncthreads();
        if (tid == 0) {
            for (int w = 1; w < CORE_WAVES; ++w) { most = fmax(most, part[w]); rise += part[CORE_WAVES + w]; reach += part[2 * CORE_WAVES + w]; }
            if (most > 0.0) atomicMax(&ctl->slack[0], (unsigned long long)__double_as_longlong(most));
            if (rise > 0.0) atomicAdd(&ctl->slack[1], (unsigned long long)(rise / s.len));
            atomicAdd(&ctl->slack[2], (unsigned long long)(reach / s.lines));
        }
        ok = barrier();
        const double up = (double)load_fresh_u64(&ctl->slack[1]), far = (double)load_fresh_u64(&ctl->slack[2]);
        *stale = s.len > CORE_LIST && up > a.stale_rise * far;
        return __longlong_as_double((long long)load_fresh_u64(&ctl->slack[0]));
    }
    // brings the plain copy of the opposite duals up to date
    __device__ __forceinline__ void write_duals(const CoreSide &s)
    {
        for (int k = gtid(); k < s.len; k += gsize()) store_f64(&s.other_dual[k], word_dual(load_fresh_u64(&s.otherword[k])));
    }
    // A step's list of bidders and the next one's; the rings of counts, cleared two steps ahead (see team_steps.h)
    __device__ __forceinline__ int *bidders(unsigned step) const { return (step & 1u) ? a.list1 : a.list0; }
    __device__ __forceinline__ void clear_ahead()
    {
        if (gtid() != 0) return;
        const unsigned z = step_clears(epoch);
        store_i32(&ctl->cnt[z], 0);
        store_i32(&ctl->whole_count[z], 0);
        store_u32(&ctl->dense[z], 0u);
    }

    // (see team_steps.h)
    __device__ __forceinline__ unsigned long long rows_looked_at() const { return load_fresh_u64(&ctl->rescans); }
    __device__ __forceinline__ void add_rows_looked_at(int looked) { if (tid == 0 && looked) atomicAdd(&ctl->rescans, (unsigned long long)looked); }
    __device__ __forceinline__ bool bidders_left() const { return sh.n_alive > 0; }

    // The side's lists once more by opposite line (columns, in a search): made when a search first
    // needs them and good as long as the lists are.
    __device__ __forceinline__ bool by_column(const CoreSide &s)
    {
        const int total = s.lines * CORE_LIST;
        for (int k = gtid(); k < s.len; k += gsize()) store_i32(&s.t_at[k], 0);
        if (!barrier()) return false;
#pragma unroll 4
        for (int e = gtid(); e < total; e += gsize()) {
            const int2 entry = s.entries[e];
            if (entry.y != MF_INFEASIBLE) atomicAdd(&s.t_at[entry.x], 1);
        }
        if (!barrier()) return false;
        if (rank == 0) {                                     // running sums: a stretch of columns per thread
            const int per = (s.len + CORE_THREADS - 1) / CORE_THREADS, first = tid * per, last = min(first + per, s.len);
            int mine = 0;
            for (int k = first; k < last; ++k) mine += load_fresh_i32(&s.t_at[k]);
            int *sums = (int *)sh.list;
            __syncthreads();
            sums[tid] = mine;
            __syncthreads();
            for (int d = 1; d < CORE_THREADS; d <<= 1) {
                const int o = tid >= d ? sums[tid - d] : 0;
                __syncthreads();
                sums[tid] += o;
                __syncthreads();
            }
            int run = sums[tid] - mine;
            for (int k = first; k < last; ++k) {
                const int n = load_fresh_i32(&s.t_at[k]);
                store_i32(&s.t_start[k], run);
                store_i32(&s.t_at[k], run);
                run += n;
            }
        }
        if (!barrier()) return false;
#pragma unroll 4
        for (int e = gtid(); e < total; e += gsize()) {
            const int2 entry = s.entries[e];
            if (entry.y != MF_INFEASIBLE) {
                const int at = atomicAdd(&s.t_at[entry.x], 1);
                store_through((unsigned long long *)&s.t_entries[at], (unsigned long long)(unsigned)(e / CORE_LIST) | ((unsigned long long)(unsigned)entry.y << 32));
            }
        }
        return barrier();
    }

    __device__ __forceinline__ int search(const CoreSide &s, double eps, double slack, int count, const int *list, int *next, int *counter);
    __device__ __forceinline__ int refine(double lower_by);
    __device__ __forceinline__ int run();
    __device__ __forceinline__ int leave(int reason, int phase, int stage, int count, int parity);
};

// Runs one side until at most stop_at bidders are left.  Returns 0 (done), or a reason to leave the launch.
template <bool LARGE>
__device__ __forceinline__ int run_bids(Core<LARGE> &c, const CoreSide &s, double eps, double slack, int stop_at, bool count_rests,
                        int &count, double &bid_budget)
{
    const CoreArgs &a = c.a;
    CoreCtl *ctl = c.ctl;
    long long few_steps = 0, stuck_steps = 0;
    int fewest = count;
    unsigned dense_lines = 0, looks = 0;
    // Bidders whose lists no longer decide wait for better ones while there are many of them: a wavefront takes 0.1 to
    // 0.3 ms to read a line of 20,000 past the caches, the lists of 9000 such lines are made in 0.2 ms.  (First bids of
    // the second phase of a 20,000 x 20,000 round on lists: 2.1 ms with lines read, 0.12 ms and 0.4 ms of lists so.)
    bool put_off = LARGE;
    while (count > stop_at) {
        const int *list = c.bidders(c.epoch);
        int *next = c.bidders(c.epoch + 1u);
        int *counter = &ctl->cnt[step_fills(c.epoch)];
        c.clear_ahead();
        if (c.tid == 0) { c.sh.pushes = 0u; c.sh.dense = 0; if (LARGE) c.sh.n_alive = 0; }
        __syncthreads();
        // few enough for one die: its chain steps and barriers are shorter
        if (a.wide && count <= a.narrow_at) return MF_CORE_HANDOVER;
        if (side_ends(count, stop_at, count_rests || a.tail_always || __builtin_amdgcn_readfirstlane(c.sh.columns_wait) ? a.tail_steps : 0, few_steps)) break;      // (see side_end.h)
        const bool few = count <= a.path_max || (count <= CORE_MAX_SOURCES && few_steps >= 4 * a.path_after);
        // (hundreds of bidders that outbid each other by an epsilon at a time, as on rank-one weights: a
        // search for as many of them as it takes)
        const bool stuck = stuck_steps >= stuck_after(a.path_after);
        if (a.path_max > 0 && ((few && few_steps >= a.path_after) || stuck)) {
            const int rc = c.search(s, eps, slack, count, list, next, counter);
            if (rc == MF_CORE_DENSE || rc == MF_CORE_RELIST) { ++c.epoch; count = load_fresh_i32(&ctl->cnt[step_reads(c.epoch)]); }
            if (rc) return rc;
            few_steps = stuck_steps = 0;
        } else {
            // with more bidders than wavefronts a chain is followed for a few steps only
            const int most = count > c.gwaves() ? a.steps_many : a.steps_few;
            bid_budget -= (double)count * most;
            // (far more looks at the list than a side takes: finish it on whole lines)
            if (bid_budget < 0.0 || ++looks > 100000u) return MF_CORE_LIMIT;
            for (int item = c.gwave(); item < count; item += c.gwaves()) {
                int b = __builtin_amdgcn_readfirstlane(load_fresh_i32(&list[item]));
                typename Core<LARGE>::Half h = c.half_of(s, b);
                int done = 0, waiting = -1;
                for (; b >= 0 && done < most; ++done) b = c.bid(s, b, h, eps, slack, count_rests, waiting);
                if (LARGE && waiting >= 0) {
                    b = waiting;
                    if (!put_off) {                         // (read below; should there be no room, in a step to come)
                        int at = 0;
                        if (c.lane == 0) at = atomicAdd(&c.sh.n_alive, 1);
                        at = __builtin_amdgcn_readfirstlane(at);
                        if (at < CORE_MAX_SOURCES) {
                            if (c.lane == 0) c.sh.alive[at] = b;
                            b = -1;
                        }
                    }
                }
                if (b >= 0 && c.lane == 0) c.push(b, next, counter);
                if (c.gwave() == 0) c.depth += (unsigned)done;
            }
            if (LARGE && !put_off) {
                __syncthreads();
                const int reading = min(c.sh.n_alive, CORE_MAX_SOURCES);
                for (int q = 0; q < reading; ++q) {
                    const int set_off = c.bid_on_whole_line(s, c.sh.alive[q], eps, count_rests);
                    if (c.tid == 0 && set_off >= 0) c.push(set_off, next, counter);
                }
            }
            if (count <= CORE_MAX_SOURCES) few_steps += most;
            stuck_steps += most;
            c.flush(next, counter);
            if (c.tid == 0 && c.sh.dense) atomicAdd(&ctl->dense[step_fills(c.epoch)], (unsigned)c.sh.dense);
        }
        if (!c.barrier()) return MF_CORE_ABORT;
        ++c.epoch;
        count = load_fresh_i32(&ctl->cnt[step_reads(c.epoch)]);
        if (count <= fewest - fewest / 8) { fewest = count; stuck_steps = 0; }
        const unsigned dense = load_fresh_u32(&ctl->dense[step_reads(c.epoch)]);
        if (LARGE && put_off) {
            if (count > stop_at && dense > CORE_WAITING && 4u * dense >= (unsigned)count) return MF_CORE_RELIST;
            put_off = dense == 0u || dense > CORE_WAITING;      // (few enough to read their lines)
        } else {
            dense_lines += dense;
            if (count > stop_at && dense_lines > (unsigned)a.dense_limit) return MF_CORE_RELIST;
            put_off = LARGE;
        }
    }
    return 0;
}

// Shortest augmenting paths for the bidders in list[0..count): see paths.hip for the method (one
// label-correcting search with every unplaced bidder a root, the nearest end of a path served one
// at a time).  Here a scanned line costs its list; what lies beyond the list is bounded below by
// the length the list's bound gives, and only a line for which that is shorter than the nearest
// path end known is read whole.
//
// When a path is served only the columns of its root's tree change price, and only they lose their
// labels: no label of another tree can become shorter, because a column of the tree is, at its raised
// price, at least as far from any scanned row as the served path was long.  The tree's columns get
// their new labels from the scanned rows whose lists they are on, and
// candidates a scan left out because they lay beyond the path end of the time are remembered by
// the shortest one.  (Scanning every labelled row again after each path was 600,000 scans, not 50,000, for
// a 20,000 x 20,000 matching.)
template <bool LARGE>
__device__ __forceinline__ int Core<LARGE>::search(const CoreSide &s, double eps, double slack, int listed_count, const int *list, int *next, int *counter)
{
    const int count = min(listed_count, CORE_MAX_SOURCES);
    for (int k = gtid(); k < s.len; k += gsize()) {
        store_through(&a.label[k], CORE_INF);
        store_through(&a.expanded[k], CORE_INF);
        store_through(&a.read_from[k], CORE_INF);
        store_f64(&a.left[k], CORE_FAR);
        store_f64(&a.dropped[k], CORE_FAR);
        store_u32(&a.stamp[k], 0u);
        const int h = word_id(load_fresh_u64(&s.otherword[k]));
        if (h >= 0) store_i32(&a.held_weight[k], s.A[(size_t)h * s.pitch + k]);
    }
    for (int i = gtid(); i < s.lines; i += gsize()) store_f64(&a.base[i], CORE_FAR);
    if (!barrier()) return MF_CORE_ABORT;
    for (int item = gwave(); item < count; item += gwaves()) {
        const int r = load_fresh_i32(&list[item]);
        double outside;
        const Top2 t = listed(s, r, slack, &outside);
        const double best = t.b1 >= outside ? t.b1 : whole_line(s, r).b1;
        if (lane == 0) {
            store_through(&ctl->src_profit[item], (unsigned long long)__double_as_longlong(best - eps));
            store_through(&ctl->src_outside[item], (unsigned long long)__double_as_longlong(outside));
            store_through(&ctl->src_left[item], (unsigned long long)__double_as_longlong(CORE_WHOLE));
            store_i32(&a.held[r], -1 - item);
            if (best - eps > 0.0) store_f64(&a.base[r], best);
        }
    }
    if (gtid() < 3) {
        store_through(&ctl->low[gtid()], CORE_INF);
        store_through(&ctl->sink_found[gtid()], CORE_INF);
        store_through(&ctl->frontier[gtid()], 0ull);
        store_through(&ctl->whole_front[gtid()], 0ull);
    }
    if (gtid() <= CORE_JUMP_PASSES) store_u32(&ctl->jump_pending[gtid()], 0u);
    if (gtid() == 0) { store_through(&ctl->sink, CORE_INF); store_through(&ctl->rescans, 0ull); }
    if (!barrier()) return MF_CORE_ABORT;
    if (tid < count) {
        sh.profit[tid] = __longlong_as_double((long long)load_fresh_u64(&ctl->src_profit[tid]));
        sh.outside[tid] = __longlong_as_double((long long)load_fresh_u64(&ctl->src_outside[tid]));
        sh.remainder[tid] = sh.profit[tid] + eps - sh.outside[tid];
        sh.row[tid] = load_fresh_i32(&list[tid]);
    }
    __syncthreads();
    if (tid == 0) {
        int n = 0;
        for (int j = 0; j < count; ++j)
            if (sh.profit[j] > 0.0) sh.alive[n++] = j;      // a bidder whose best value is at most eps rests
        sh.n_alive = n;
        sh.served = 0ull;
    }
    __syncthreads();
    int n_alive = sh.n_alive;
    const unsigned side_bit = s.otherword == a.side[0].otherword ? 1u : 2u;
    auto resting_bidders = [&]() {
        unsigned long long best = CORE_INF;
        for (int e = 0; e < n_alive; ++e) {
            const int j = sh.alive[e];
            const unsigned long long w = ((unsigned long long)(long long)sh.profit[j] << 21) | (1ull << 20) | (unsigned long long)sh.row[j];
            best = w < best ? w : best;
        }
        return best;
    };
    unsigned long long agreed_sink = resting_bidders();
    double low = 0.0, width = 4.0 * eps;
    unsigned step = 0, since_served = 0;
    bool swept = false, from_bidders = true, sweep_next = false;
    int status = 0;
    long long lines_read = 0;                                // whole lines; the same in every workgroup
    unsigned long long my_steps = 0;
    while (n_alive > 0) {
        if (++since_served > 4u * (unsigned)s.len + 4096u) { status = MF_CORE_DENSE; break; }     // (the same in every workgroup)
        ++step;
        const unsigned c = step % 3u, p = (step + 1u) % 3u, z = (step + 2u) % 3u;
        if (tid == 0) { sh.pushes = 0u; sh.sink = CORE_INF; sh.low = CORE_INF; sh.dense = 0; }
        __syncthreads();
        // (the last step's barrier ended all writing to slot c: this step writes p and z, and a served tree clears them behind
        // the next barrier.  The nearest sink, [9], moves meanwhile: it only prunes, and decides nothing)
        const unsigned long long words = load_fresh_u64(&ctl->low[min(lane, 12)]);
        auto word_at = [&](unsigned q) {
            return (unsigned long long)(unsigned)__builtin_amdgcn_readlane((int)(unsigned)(words & 0xffffffffull), (int)q) |
                   ((unsigned long long)(unsigned)__builtin_amdgcn_readlane((int)(unsigned)(words >> 32), (int)q) << 32);
        };
        const int front = from_bidders ? 0 : (int)word_at(6u + c);
        const int whole_front = from_bidders ? 0 : min((int)word_at(10u + c), s.len + CORE_MAX_SOURCES);
        const bool sweeping = !from_bidders && (sweep_next || front + whole_front == 0);
        const int nf = from_bidders ? n_alive : (sweeping ? 0 : min(front, a.frontier_room));
        const int nw = sweeping ? 0 : whole_front;
        lines_read += nw;
        // Paths so long that the lists do not show what they are made of are better searched for on whole
        // lines by the whole device: a 20,000 x 20,000 round of that kind took 390 ms here, 120 ms so.
        if (lines_read > s.read_limit) { status = MF_CORE_DENSE; break; }
        {
            const unsigned long long found = word_at(3u + c);
            agreed_sink = found < agreed_sink ? found : agreed_sink;
        }
        if (!from_bidders && !sweep_next && swept && nf + nw == 0) {
            const unsigned long long lo = word_at(c);
            if (lo == CORE_INF || lo >= (agreed_sink >> 21)) {
                // ---- every label below the nearest path end is final: serve its tree ----
                // (Should a wait run out anywhere in here, the launch ends and the phase starts again
                // from the prices it began with: nothing half-done survives.)
                const unsigned long long sink = agreed_sink, d_star = sink >> 21;
                const int sink_id = (int)(sink & 0xfffffull);
                const bool gives_up = ((sink >> 20) & 1ull) != 0;
                for (int k = gtid(); k < s.len; k += gsize()) {
                    const unsigned long long lw = load_fresh_u64(&a.label[k]);
                    int up = CORE_NO_LABEL;
                    const int row = (int)(lw & MF_ID_MASK);
                    if (lw != CORE_INF) up = load_fresh_i32(&a.held[row]);
                    store_through(&a.parent[k], ((unsigned long long)(unsigned)row << 32) | (unsigned long long)(unsigned)up);
                    store_i32(&a.jump[k], up);
                }
                if (!barrier()) return MF_CORE_ABORT;
                int passes = 0;
                bool lost = false;
                for (;;) {
                    bool short_of_it = false;
                    for (int k = gtid(); k < s.len; k += gsize()) {
                        int up = load_fresh_i32(&a.jump[k]);
                        if (up < 0) continue;
                        for (int hop = 0; hop < CORE_JUMP_HOPS && up >= 0; ++hop) up = load_fresh_i32(&a.jump[up]);
                        store_i32(&a.jump[k], up);
                        short_of_it |= up >= 0;
                    }
                    if (__syncthreads_or(short_of_it) && tid == 0) atomicOr(&ctl->jump_pending[passes], 1u);
                    if (!barrier()) return MF_CORE_ABORT;
                    if (load_fresh_u32(&ctl->jump_pending[passes]) == 0u) break;      // (cleared two barriers from here)
                    if (++passes >= CORE_JUMP_PASSES) { lost = true; break; }
                }
                int root = -1;
                {
                    int at = sink_id;
                    if (gives_up) at = load_fresh_i32(&a.held[sink_id]);
                    if (at >= 0) at = load_fresh_i32(&a.jump[at]);
                    if (at < 0 && at != CORE_NO_LABEL) root = -1 - at;
                }
                if (lost || root < 0 || root >= count) { status = MF_CORE_DENSE; break; }
                if (tid == 0) sh.pushes = 0u;
                if (gtid() == 0) { store_i32(&ctl->tree_count, 0); store_i32(&ctl->read_count, 0); store_f64(&a.base[sh.row[root]], CORE_FAR); }
                if (!barrier()) return MF_CORE_ABORT;
                for (int k = gtid(); k < s.len; k += gsize()) {
                    if (load_fresh_i32(&a.jump[k]) != -1 - root) continue;
                    store_u32(&a.stamp[k], CORE_IN_TREE);
                    const unsigned long long d_int = load_fresh_u64(&a.label[k]) >> MF_ID_BITS;
                    const unsigned long long cw = load_fresh_u64(&s.otherword[k]);
                    if (word_id(cw) >= 0) store_f64(&a.base[word_id(cw)], CORE_FAR);        // its holder's scan no longer counts
                    {
                        const unsigned slot = atomicAdd(&sh.pushes, 1u);
                        if (slot < (unsigned)CORE_PUSH_BUFFER) sh.list[slot] = (unsigned long long)(unsigned)k;
                        else store_i32(&a.tree[atomicAdd(&ctl->tree_count, 1)], k);
                    }
                    if (d_int < d_star) {
                        store_through(&s.otherword[k], pack_word(word_dual(cw) + (double)(long long)(d_star - d_int), (int)(cw & MF_ID_MASK)));
                    }
                }
                flush(a.tree, &ctl->tree_count);
                if (!barrier()) return MF_CORE_ABORT;
                auto clear_tree = [&]() {
                    if (rank == 0) {
                        if (tid == 0) {
                            int k = sink_id;
                            if (gives_up) {
                                const int h = load_fresh_i32(&a.held[sink_id]);
                                k = h < 0 ? -1 : h;
                            }
                            // (one dependent trip a hop here; the words are changed below, by as many threads as there are hops)
                            unsigned hops = 0;
                            while (k >= 0 && hops <= (unsigned)s.lines) {
                                const unsigned long long pr = load_fresh_u64(&a.parent[k]);
                                const int i = (int)(pr >> 32);
                                if (hops < (unsigned)CORE_PUSH_BUFFER) sh.list[hops] = ((unsigned long long)(unsigned)i << 32) | (unsigned long long)(unsigned)k;
                                else {
                                    store_through(&s.otherword[k], pack_word(word_dual(load_fresh_u64(&s.otherword[k])) + eps, i + 1));
                                    store_i32(&a.held_weight[k], s.A[(size_t)i * s.pitch + k]);
                                }
                                ++hops;
                                k = (int)(unsigned)(pr & 0xffffffffull);
                            }
                            sh.pushes = hops;
                            for (int q = 0; q <= CORE_JUMP_PASSES; ++q) store_u32(&ctl->jump_pending[q], 0u);
                            store_through(&ctl->sink, CORE_INF);
                            for (int q = 0; q < 3; ++q) {
                                store_through(&ctl->sink_found[q], CORE_INF); store_through(&ctl->low[q], CORE_INF);
                                store_through(&ctl->frontier[q], 0ull); store_through(&ctl->whole_front[q], 0ull);
                            }
                        }
                        __syncthreads();
                        for (unsigned t = tid; t < min(sh.pushes, (unsigned)CORE_PUSH_BUFFER); t += CORE_THREADS) {
                            const int k = (int)(unsigned)(sh.list[t] & 0xffffffffull), i = (int)(sh.list[t] >> 32);
                            store_through(&s.otherword[k], pack_word(word_dual(load_fresh_u64(&s.otherword[k])) + eps, i + 1));
                            store_i32(&a.held_weight[k], s.A[(size_t)i * s.pitch + k]);
                        }
                    }
                    // The tree's columns lose their labels.  What the others have reached stays as it is: a
                    // column of the tree, at its raised price, is at least as far from any of them as the
                    // path just served was long.
                    __syncthreads();
                    if (tid == 0) sh.pushes = 0u;
                    __syncthreads();
                    auto was_read = [&](int i) {
                        const unsigned slot = atomicAdd(&sh.pushes, 1u);
                        if (slot < (unsigned)CORE_PUSH_BUFFER) sh.list[slot] = (unsigned long long)(unsigned)i;
                        else store_i32(&a.whole0[atomicAdd(&ctl->read_count, 1)], i);
                    };
                    for (int k = gtid(); k < s.len; k += gsize()) {
                        const unsigned state = load_fresh_u32(&a.stamp[k]);
                        if (state == CORE_IN_TREE) {
                            store_through(&a.label[k], CORE_INF);
                            store_u32(&a.stamp[k], 0u);
                            store_through(&a.expanded[k], CORE_INF);
                            store_through(&a.read_from[k], CORE_INF);
                            store_f64(&a.left[k], CORE_FAR);
                            store_f64(&a.dropped[k], CORE_FAR);
                        } else if (state == CORE_READ) was_read(word_id(load_fresh_u64(&s.otherword[k])));
                    }
                    if (rank == 0 && tid < n_alive && sh.alive[tid] != root && sh.remainder[sh.alive[tid]] >= CORE_WHOLE) was_read(sh.row[sh.alive[tid]]);
                    flush(a.whole0, &ctl->read_count);
                    __syncthreads();
                    if (tid == 0) {
                        int n = 0;
                        for (int e = 0; e < n_alive; ++e) if (sh.alive[e] != root) sh.alive[n++] = sh.alive[e];
                        sh.n_alive = n;
                    }
                };
                auto offer_again = [&](bool from_columns) {
                    // New labels for the tree's columns, from the scanned rows whose lists they are on.  Either every
                    // scanned row's list is looked through once more, or the lists are kept by column as well and
                    // a wavefront takes a column, or a stretch of its entries.  Making those takes one die 0.1 ms for
                    // 1024 lines, 0.65 ms for 20,000 (1 ms with 40,000 columns); looking through a thousand lists takes
                    // 15 us, and a search has a dozen trees to serve.  So they are made once four times as many
                    // rows have been looked at as there are, few searches.  (Made at the start of every
                    // search: 20,000 x 20,000 next round 23.5 / 21.7 ms, 20,000 x 40,000 24.5 / 22.7, matching 14.3 /
                    // 13.7, 4096 x 8192 7.65 / 7.44, smaller ones the same.)
                    const int n_tree = load_fresh_i32(&ctl->tree_count);       // (this and read_count: complete, and cleared by the next tree)
                    constexpr int STRETCH = 512;
                    int looked = 0;
                    if (!from_columns) {
                        unsigned *in_tree = (unsigned *)sh.list;             // a bit a column, and this workgroup's scanned rows
                        int *rows = (int *)(sh.list + CORE_PUSH_BUFFER / 2);
                        __syncthreads();
                        if (tid == 0) sh.pushes = 0u;
                        for (int t = tid; t * 32 < s.len; t += CORE_THREADS) in_tree[t] = 0u;
                        __syncthreads();
                        for (int t = tid; t < n_tree; t += CORE_THREADS) {
                            const int k = load_fresh_i32(&a.tree[t]);
                            atomicOr(&in_tree[k >> 5], 1u << (k & 31));
                        }
                        for (int i = gtid(); i < s.lines; i += gsize())
                            if (load_fresh(&a.base[i]) < CORE_FAR * 0.5) rows[atomicAdd(&sh.pushes, 1u)] = i;
                        __syncthreads();
                        looked = (int)sh.pushes;
                        int i = wave < looked ? rows[wave] : 0;
                        const int2 *e = s.entries + (size_t)i * CORE_LIST;
                        int2 e0 = e[lane], e1 = e[lane + 64];
                        double base = load_fresh(&a.base[i]);
                        for (int t = wave; t < looked; t += CORE_WAVES) {
                            const int2 now0 = e0, now1 = e1;
                            const int now = i;
                            const double from = base;
                            if (t + CORE_WAVES < looked) {                   // the next row's list, meanwhile
                                i = rows[t + CORE_WAVES];
                                e = s.entries + (size_t)i * CORE_LIST;
                                e0 = e[lane]; e1 = e[lane + 64];
                                base = load_fresh(&a.base[i]);
                            }
                            const bool in0 = now0.y != MF_INFEASIBLE && (in_tree[now0.x >> 5] >> (now0.x & 31) & 1u);
                            const bool in1 = now1.y != MF_INFEASIBLE && (in_tree[now1.x >> 5] >> (now1.x & 31) & 1u);
                            if (!__any(in0 || in1)) continue;
                            unsigned long long w0 = 0ull, w1 = 0ull, l0 = 0ull, l1 = 0ull;
                            if (in0) { w0 = load_fresh_u64(&s.otherword[now0.x]); l0 = load_fresh_u64(&a.label[now0.x]); }
                            if (in1) { w1 = load_fresh_u64(&s.otherword[now1.x]); l1 = load_fresh_u64(&a.label[now1.x]); }
                            const unsigned long long m0 = ((unsigned long long)(long long)(from - fma(a.Kd, (double)now0.y, -word_dual(w0))) << MF_ID_BITS) | (unsigned long long)now;
                            const unsigned long long m1 = ((unsigned long long)(long long)(from - fma(a.Kd, (double)now1.y, -word_dual(w1))) << MF_ID_BITS) | (unsigned long long)now;
                            if (in0 && m0 < l0) atomicMin(&a.label[now0.x], m0);
                            if (in1 && m1 < l1) atomicMin(&a.label[now1.x], m1);
                        }
                    } else for (int it = gwave(); it < n_tree; it += gwaves()) {
                        const int k = load_fresh_i32(&a.tree[it]);
                        const int from = load_fresh_i32(&s.t_start[k]), to = load_fresh_i32(&s.t_at[k]);
                        const double price = word_dual(load_fresh_u64(&s.otherword[k]));
                        for (int e0 = from; e0 < to; e0 += STRETCH) {
                            double best = CORE_FAR;
                            int who = 0;
#pragma unroll
                            for (int q = 0; q < STRETCH / 64; ++q) {
                                const int e = e0 + q * 64 + lane;
                                if (e < to) {
                                    const unsigned long long entry = load_fresh_u64((const unsigned long long *)&s.t_entries[e]);
                                    const int i = (int)(unsigned)(entry & 0xffffffffull);
                                    const double cand = load_fresh(&a.base[i]) - fma(a.Kd, (double)(int)(entry >> 32), -price);
                                    if (cand < best) { best = cand; who = i; }
                                }
                            }
                            const double least = -wave_max(-best);
                            if (least < CORE_FAR * 0.5) {
                                const int i = wave_min(best == least ? who : 0x7fffffff);
                                if (lane == 0) {
                                    const unsigned long long mine = ((unsigned long long)(long long)least << MF_ID_BITS) | (unsigned long long)i;
                                    atomicMin(&a.label[k], mine);
                                }
                            }
                        }
                    }
                    // ... and at the rows whose whole lines have been read: what is not on their lists they
                    // would not offer the column again.  (Reading all those lines once more after every
                    // path took 15 ms a path where 15,000 lines had been read.)
                    const int n_read = load_fresh_i32(&ctl->read_count), stretches = (n_read + STRETCH - 1) / STRETCH;
                    for (int it = gwave(); it < n_tree * stretches; it += gwaves()) {
                        const int k = load_fresh_i32(&a.tree[it / stretches]), from = it % stretches * STRETCH;
                        const double price = word_dual(load_fresh_u64(&s.otherword[k]));
                        double best = CORE_FAR;
                        int who = 0;
#pragma unroll
                        for (int q = 0; q < STRETCH / 64; ++q) {
                            const int e = from + q * 64 + lane;
                            if (e < n_read) {
                                const int i = load_fresh_i32(&a.whole0[e]);
                                const int32_t w = !s.line_len || k < s.line_len[i] ? s.A[(size_t)i * s.pitch + k] : MF_INFEASIBLE;
                                const double cand = load_fresh(&a.base[i]) - fma(a.Kd, (double)w, -price);
                                if (w != MF_INFEASIBLE && cand < best) { best = cand; who = i; }
                            }
                        }
                        const double least = -wave_max(-best);
                        if (least < CORE_FAR * 0.5) {
                            const int i = wave_min(best == least ? who : 0x7fffffff);
                            if (lane == 0) atomicMin(&a.label[k], ((unsigned long long)(long long)least << MF_ID_BITS) | (unsigned long long)i);
                        }
                    }
                    return looked;
                };
                bool by_columns = (columns_ready & side_bit) != 0u;
                const bool must = s.len > CORE_PUSH_BUFFER * 32 || s.lines / (int)G + CORE_THREADS > CORE_PUSH_BUFFER;      // (no room in LDS)
                if (!labels_of_served_tree(*this, by_columns, must, (unsigned long long)s.lines * CORE_RESCANS, clear_tree,
                                           [&]() { return by_column(s); }, offer_again))
                    return MF_CORE_ABORT;
                if (by_columns) columns_ready |= side_bit;
                if (tid == 0) sh.served = d_star;
                n_alive = sh.n_alive;
                agreed_sink = resting_bidders();
                since_served = 0;
                --step;
                from_bidders = false; sweep_next = true; swept = false;
                continue;
            }
            low = (double)(long long)lo;
        }
        const double bound = (double)(long long)(min(agreed_sink, word_at(9)) >> 21);
        if (nf > a.frontier_high) width = fmax(eps, width * 0.5);
        else if (nf < a.frontier_high / 8) width = fmin(a.path_width * eps, width * 2.0);
        const double limit = fmin(low + width, bound);
        if (gtid() == 0) {
            store_through(&ctl->frontier[z], 0ull);
            store_through(&ctl->whole_front[z], 0ull);
            store_through(&ctl->low[z], CORE_INF);
            store_through(&ctl->sink_found[z], CORE_INF);
        }
        const unsigned long long *frontier = ((step & 1u) ? a.frontier1 : a.frontier0);
        unsigned long long *next_frontier = ((step & 1u) ? a.frontier0 : a.frontier1);
        auto reach = [&](int k, int holder) {
            const unsigned long long entry = ((unsigned long long)(unsigned)holder << 32) | (unsigned long long)(unsigned)k;
            const unsigned slot = atomicAdd(&sh.pushes, 1u);
            if (slot < (unsigned)CORE_PUSH_BUFFER) sh.list[slot] = entry;
            else {                                      // (no room: the pass over all columns finds the label)
                const unsigned long long at = atomicAdd(&ctl->frontier[p], 1ull);
                if (at < (unsigned long long)a.frontier_room) store_through(&next_frontier[at], entry);
            }
        };
        auto ends_at = [&](unsigned long long word) { atomicMin(&ctl->sink, word); atomicMin(&ctl->sink_found[p], word); };
        // One candidate: column k at weight w through row i.  `first` is what the compare-and-swap of
        // its label saw (so that a wavefront has those of both its entries in flight at once).  A
        // column lowered twice in a step is twice on the frontier: looking it up in a stamp would
        // cost every first one another round trip, and what two scans of its holder publish goes
        // together in any order (search_words.h).
        auto candidate = [&](double base, int32_t w, unsigned long long word) {
            const double cand = base - fma(a.Kd, (double)w, -word_dual(word));
            return w != MF_INFEASIBLE && cand < bound ? cand : CORE_FAR;
        };
        auto label_of = [&](double cand, int i) { return ((unsigned long long)(long long)cand << MF_ID_BITS) | (unsigned long long)i; };
        auto shorter = [&](unsigned long long mine, unsigned long long seen) { return (mine >> MF_ID_BITS) < (seen >> MF_ID_BITS); };
        auto settle = [&](double cand, int k, unsigned long long word, unsigned long long mine, unsigned long long seen, unsigned long long was) {
            while (was != seen) {                       // strictly shorter only: see lower_label in paths.hip
                if (!shorter(mine, was)) return;
                seen = was;
                was = atomicCAS(&a.label[k], seen, mine);
            }
            if (cand < limit) {
                const int holder = word_id(word);
                if (holder < 0) ends_at(((unsigned long long)(long long)cand << 21) | (unsigned long long)k);
                else reach(k, holder);
            }
        };
        auto relax = [&](int i, double cand, int k, unsigned long long word) {
            const unsigned long long mine = label_of(cand, i), seen = load_fresh_u64(&a.label[k]);
            if (shorter(mine, seen)) settle(cand, k, word, mine, seen, atomicCAS(&a.label[k], seen, mine));
        };
        int *whole_list = (step & 1u) ? a.whole1 : a.whole0, *next_whole = (step & 1u) ? a.whole0 : a.whole1;
        unsigned taken = 0;                                         // of sh.list: scanned already
        if (nf + nw > 0) {
            swept = false;
            // With few rows on the frontier a workgroup goes on with what its own scans reach for some
            // rounds before the next step shares it out.  A path is some 70 rows long and each of
            // them took a step of 4.5 us, 2.4 us of it to hand over to everybody else and wait for
            // them; a round of its own takes 2 us (all searches of a 20,000 x 20,000 matching
            // 11.8 -> 6.5 ms, 1024 x 1024 1.1 -> 0.7 ms).
            int here = nf, first = gwave(), stride = gwaves();
            unsigned start = 0;
            for (int round = 0;; ++round) {
            for (int it = first; it < here; it += stride) {
                int i, mine_col;                                     // (a bidder: -1 - its number)
                if (round == 0 && from_bidders) {
                    mine_col = -1 - sh.alive[it];
                    i = sh.row[-1 - mine_col];
                } else {
                    const unsigned long long entry = round ? sh.list[start + it] : load_fresh_u64(&frontier[it]);
                    mine_col = (int)(unsigned)(entry & 0xffffffffull);
                    i = (int)(unsigned)(entry >> 32);
                }
                const int2 *e = s.entries + (size_t)i * CORE_LIST;
                const int2 e0 = e[lane], e1 = e[lane + 64];
                unsigned long long lw = 0ull, held_word = 0ull, ex = CORE_INF;
                int32_t w_held = 0;
                if (mine_col >= 0) {
                    lw = load_fresh_u64(&a.label[mine_col]);
                    held_word = load_fresh_u64(&s.otherword[mine_col]);
                    w_held = load_fresh_i32(&a.held_weight[mine_col]);
                    ex = load_fresh_u64(&a.expanded[mine_col]);
                }
                const unsigned long long w0 = load_fresh_u64(&s.otherword[e0.x]), w1 = load_fresh_u64(&s.otherword[e1.x]);
                const unsigned long long l0 = load_fresh_u64(&a.label[e0.x]), l1 = load_fresh_u64(&a.label[e1.x]);
                double dist, profit;
                if (mine_col < 0) { dist = 0.0; profit = sh.profit[-1 - mine_col]; }
                else {
                    if (lw == CORE_INF || scanned_from(lw >> MF_ID_BITS, ex)) continue;     // (from that label already)
                    dist = (double)(long long)(lw >> MF_ID_BITS);
                    profit = fma(a.Kd, (double)w_held, -word_dual(held_word));
                }
                const double base = dist + profit + eps;
                double left_out;
                {
                    const double c0 = candidate(base, e0.y, w0), c1 = candidate(base, e1.y, w1);
                    const unsigned long long m0 = label_of(c0, i), m1 = label_of(c1, i);
                    const bool try0 = c0 < CORE_FAR && shorter(m0, l0), try1 = c1 < CORE_FAR && shorter(m1, l1);
                    // (what lies beyond the nearest path end is left out until that end is served)
                    const double x0 = base - fma(a.Kd, (double)e0.y, -word_dual(w0)), x1 = base - fma(a.Kd, (double)e1.y, -word_dual(w1));
                    left_out = fmin(e0.y != MF_INFEASIBLE && !(x0 < bound) ? x0 : CORE_FAR, e1.y != MF_INFEASIBLE && !(x1 < bound) ? x1 : CORE_FAR);
                    unsigned long long was0 = 0ull, was1 = 0ull;
                    if (try0) was0 = atomicCAS(&a.label[e0.x], l0, m0);
                    if (try1) was1 = atomicCAS(&a.label[e1.x], l1, m1);
                    if (try0) settle(c0, e0.x, w0, m0, l0, was0);
                    if (try1) settle(c1, e1.x, w1, m1, l1, was1);
                }
                // (last: a load that is waited for after a store waits for the store as well)
                left_out = -wave_max(-left_out);
                if (mine_col < 0 && lane == 0) store_through(&ctl->src_dropped[-1 - mine_col], (unsigned long long)__double_as_longlong(left_out));
                if (mine_col >= 0 && lane == 0) {
                    publish_scan(SharedWords{}, ScanWords{&a.base[i], &a.dropped[mine_col], &a.expanded[mine_col]}, lw >> MF_ID_BITS, base, left_out);
                    store_i32(&a.held[i], mine_col);
                    if (dist + profit < bound)
                        ends_at(((unsigned long long)(long long)(dist + profit) << 21) | (1ull << 20) | (unsigned long long)i);
                }
                ++scans;
            }
            if (round >= CORE_OWN_ROUNDS || 2 * nf > gwaves()) break;
            __syncthreads();
            const unsigned end = min(sh.pushes, (unsigned)CORE_PUSH_BUFFER);
            __syncthreads();
            start = taken;
            here = (int)(end - taken);
            if (here == 0 || here > CORE_OWN_MOST) break;
            taken = end;
            first = wave; stride = CORE_WAVES;
            }
            // whole lines, in slices: a wavefront each.  What bounds it is latency: four entries' prices are in
            // flight per lane, and a label is looked at only where it may be lowered (one entry at a
            // time took 24 us a slice, 36 ms where 37,000 lines of 20,000 had to be read).
            const int parts = nw > 0 ? parts_of(s, nw) : 1;
            int slice = 0;                                          // (a slice a turn: what a line needs is loaded again, a loop around the slices keeps it in registers)
            for (int it = gwave(); it < nw * parts;) {
                const int e = it / parts, from = (it - e * parts + slice * parts) * CORE_SLICE;
                const int entry = __builtin_amdgcn_readfirstlane(load_fresh_i32(&whole_list[e]));
                int i;
                double base;
                bool sound = true;
                if (entry < 0) {                                    // a bidder
                    const int j = -1 - entry;
                    i = __builtin_amdgcn_readfirstlane(sh.row[j]);
                    base = sh.profit[j] + eps;
                } else {
                    const unsigned long long lw = load_fresh_u64(&a.label[entry]), word = load_fresh_u64(&s.otherword[entry]);
                    i = __builtin_amdgcn_readfirstlane(word_id(word));
                    base = (double)(long long)(lw >> MF_ID_BITS) + fma(a.Kd, (double)load_fresh_i32(&a.held_weight[entry]), -word_dual(word)) + eps;
                    sound = lw != CORE_INF && i >= 0;               // (cannot be otherwise)
                }
                const int length = !sound ? 0 : s.line_len ? min(s.line_len[i], s.len) : s.len, to = min(length, from + CORE_SLICE);
                if (from < to) {
                    int4 ahead[CORE_SLICE / 256];
                    load_slice(s.A + (size_t)i * s.pitch, from, to, ahead);
                    const double unlisted = base - (s.bound[i] + slack);
                    double left_out = CORE_FAR;                     // the nearest unlisted one beyond the nearest path end
#pragma unroll
                    for (int q = 0; q < CORE_SLICE / 256; ++q) {
                        const int j = from + q * 256 + lane * 4;
                        if (j >= to) break;
                        const int32_t w[4] = {ahead[q].x, ahead[q].y, ahead[q].z, ahead[q].w};
                        unsigned long long word[4];
#pragma unroll
                        for (int e = 0; e < 4; ++e) word[e] = load_fresh_u64(&s.otherword[min(j + e, to - 1)]);
#pragma unroll 1
                        for (int e = 0; e < 4; ++e) {
                            if (j + e >= to || w[e] == MF_INFEASIBLE) continue;
                            const double x = base - fma(a.Kd, (double)w[e], -word_dual(word[e]));
                            if (x < bound) relax(i, x, j + e, word[e]);
                            else if (x >= unlisted) left_out = fmin(left_out, x);
                        }
                    }
                    whole += (unsigned)(to - from + 3) / 4u;
                    left_out = -wave_max(-left_out);
                    if (lane == 0 && left_out < CORE_FAR)
                        publish_slice(SharedWords{}, WholeLine{nullptr, entry < 0 ? (double *)&ctl->src_left[-1 - entry] : &a.left[entry]}, left_out);
                }
                if (from + parts * CORE_SLICE < length) ++slice;
                else { it += gwaves(); slice = 0; }
            }
            from_bidders = false;
        } else {
            swept = true;
            sweep_next = false;
            auto read_whole = [&](int entry) {
                const unsigned long long at = atomicAdd(&ctl->whole_front[p], 1ull);
                store_i32(&next_whole[at], entry);
            };
            for (int k = gtid(); k < s.len; k += gsize()) {
                const unsigned long long lw = load_fresh_u64(&a.label[k]);
                const unsigned long long ex = load_fresh_u64(&a.expanded[k]);
                const double left = load_fresh(&a.left[k]), drop = load_fresh(&a.dropped[k]);
                const unsigned long long read_from = load_fresh_u64(&a.read_from[k]);
                const int holder = word_id(load_fresh_u64(&s.otherword[k]));
                const unsigned long long d_int = lw >> MF_ID_BITS;
                if (lw == CORE_INF) continue;
                if (!scanned_from(d_int, ex)) {         // not scanned from this label yet
                    const double d = (double)(long long)d_int;
                    if (!(d < bound)) continue;
                    if (holder < 0) atomicMin(&sh.sink, (d_int << 21) | (unsigned long long)k);
                    else if (d >= limit) atomicMin(&sh.low, d_int);
                    else reach(k, holder);
                    continue;
                }
                // (a path may end in the row that holds it; found before, but ends found before one was served are forgotten)
                const double base = load_fresh(&a.base[holder]), rests = base - eps;
                const double rem = unlisted_from(d_int, read_from, left, base - (s.bound[holder] + slack));
                if (rests < bound) atomicMin(&sh.sink, ((unsigned long long)(long long)rests << 21) | (1ull << 20) | (unsigned long long)holder);
                if (drop < bound) {                     // candidates left out then may be of use now: scan it again
                    if (drop >= limit) atomicMin(&sh.low, (unsigned long long)(long long)drop);
                    else { store_through(&a.expanded[k], CORE_INF); store_f64(&a.dropped[k], CORE_FAR); reach(k, holder); }
                }
                if (rem < bound) {
                    if (rem >= limit) atomicMin(&sh.low, (unsigned long long)(long long)fmax(rem, 0.0));
                    else { read_whole(k); begin_whole_line(SharedWords{}, WholeLine{&a.read_from[k], &a.left[k]}, d_int, CORE_FAR); store_u32(&a.stamp[k], CORE_READ); }
                }
            }
            if (rank == 0 && tid < n_alive) {
                const int j = sh.alive[tid];
                const double rem = sh.remainder[j] < CORE_WHOLE ? sh.remainder[j] : __longlong_as_double((long long)load_fresh_u64(&ctl->src_left[j]));
                const double drop = __longlong_as_double((long long)load_fresh_u64(&ctl->src_dropped[j]));
                if (drop < bound) {
                    if (drop >= limit) atomicMin(&sh.low, (unsigned long long)(long long)drop);
                    else reach(-1 - j, sh.row[j]);
                }
                if (rem < bound) {
                    if (rem >= limit) atomicMin(&sh.low, (unsigned long long)(long long)fmax(rem, 0.0));
                    else { read_whole(-1 - j); sh.remainder[j] = CORE_WHOLE; store_through(&ctl->src_left[j], (unsigned long long)__double_as_longlong(CORE_WHOLE)); }
                }
            }
        }
        __syncthreads();
        const unsigned pushed = min(sh.pushes, (unsigned)CORE_PUSH_BUFFER) - taken;
        if (tid == 0) {
            sh.base = pushed ? (unsigned)atomicAdd(&ctl->frontier[p], (unsigned long long)pushed) : 0u;
            if (sh.sink != CORE_INF) ends_at(sh.sink);
            if (sh.low != CORE_INF) atomicMin(&ctl->low[p], sh.low);
        }
        __syncthreads();
        for (unsigned t = tid; t < pushed; t += CORE_THREADS)
            if (sh.base + t < (unsigned)a.frontier_room) store_through(&next_frontier[sh.base + t], sh.list[taken + t]);
        ++my_steps;
        if (!barrier()) return MF_CORE_ABORT;
    }
    // What the other trees' columns have still to rise for the paths served so far: a row of a tree that has been served
    // would rather have them at these prices.  (See pending_rise in search_words.h; the last step's barrier ended all writing of labels.)
    if (status)
        for (int k = gtid(); k < s.len; k += gsize()) {
            const unsigned long long rise = pending_rise(load_fresh_u64(&a.label[k]), CORE_INF, MF_ID_BITS, sh.served);
            if (rise) {
                const unsigned long long word = load_fresh_u64(&s.otherword[k]);
                store_through(&s.otherword[k], pack_word(word_dual(word) + (double)(long long)rise, (int)(word & MF_ID_MASK)));
            }
        }
    if (gtid() == 0) {
        steps += (unsigned)my_steps;
        for (int e = 0; e < n_alive; ++e) store_i32(&next[atomicAdd(counter, 1)], sh.row[sh.alive[e]]);
        for (int rest = count; rest < listed_count; ++rest) store_i32(&next[atomicAdd(counter, 1)], load_fresh_i32(&list[rest]));
    }
    if (status) {
        if (!barrier()) return MF_CORE_ABORT;
    }
    __syncthreads();
    return status;
}

// A complete assignment that is optimal already only lacks exact prices.  Rows raise the prices of
// the columns they would rather have until no row prefers anything to what it holds (a row without a
// partner: until nothing is worth having), each raise setting off the row that holds the column;
// this ends, without a free column ever getting a price, exactly when the assignment is optimal.  (All
// prices are first lowered by some hundred epsilons: raising can then also arrive at prices a little
// below those of the phase, which is what rows that would rather have a free column call for.)  The
// phases at finer epsilons, which would re-assign everybody several times over only to arrive at the
// same assignment, are then left out.  Returns 1 (prices proved exact), 0 (not optimal yet),
// 2 (better lists are wanted; it goes on from the prices reached), or -1.
template <bool LARGE>
__device__ __forceinline__ int Core<LARGE>::refine(double lower_by)
{
    const CoreSide &s = a.side[0];
    for (int k = gtid(); k < s.len; k += gsize()) {
        const int r = load_fresh_i32(&a.col2row[k]);
        store_through(&s.otherword[k], pack_word(fmax(load_fresh(&s.other_dual[k]) - lower_by, 0.0), r + 1));
        store_u32(&a.stamp[k], 0u);
    }
    for (int i = gtid(); i < s.lines; i += gsize()) {
        store_i32(&bidders(epoch)[i], i);
        const int col = load_fresh_i32(&a.row2col[i]);
        store_i32(&a.held_weight[i], col >= 0 ? s.A[(size_t)i * s.pitch + col] : 0);
    }
    if (gtid() < 3) store_u32(&ctl->failed[gtid()], 0u);    // (read last before the barriers of the stages since)
    bool ok;
    bool risen;
    const double slack = slack_of(s, ok, &risen);               // (its barriers also end the set-up above)
    if (!ok) return -1;
    int count = s.lines;
    int done = -2;
    unsigned whole_lines = 0;
    int whole_rows = 0, fewest = count, unimproved = 0;
    for (unsigned round = 1;; ++round) {
        const int *list = bidders(epoch);
        int *next = bidders(epoch + 1u);
        int *counter = &ctl->cnt[step_fills(epoch)];
        clear_ahead();
        if (gtid() == 0) store_u32(&ctl->failed[(round + 1u) % 3u], 0u);
        if (tid == 0) { sh.pushes = 0u; sh.failed = 0u; sh.dense = 0; }
        __syncthreads();
        // (few rows left: a workgroup looks at the rows it has set off itself for some rounds, as in a
        // search: 7 -> 3 us for each row of the last chains)
        const bool few = count <= gwaves();
        int here = count, first = gwave(), stride = gwaves();
        unsigned start = 0, taken = 0;
        for (int own = 0;; ++own) {
        for (int item = first; item < here; item += stride) {
            const int i = own ? (int)(unsigned)sh.list[start + item] : load_fresh_i32(&list[item]);
            const int2 *e = s.entries + (size_t)i * CORE_LIST;
            const int2 e0 = e[lane], e1 = e[lane + 64];
            const int col = load_fresh_i32(&a.row2col[i]);
            const int32_t w_held = load_fresh_i32(&a.held_weight[i]);
            const double outside = s.bound[i] + slack;
            const unsigned long long w0 = load_fresh_u64(&s.otherword[e0.x]), w1 = load_fresh_u64(&s.otherword[e1.x]);
            const double profit = col >= 0 ? fma(a.Kd, (double)w_held, -word_dual(load_fresh_u64(&s.otherword[max(col, 0)]))) : 0.0;
            bool failed = profit < 0.0;                 // it would rather rest
            auto wants = [&](int32_t w, unsigned long long word, double &need) {
                need = fma(a.Kd, (double)w, -profit);
                return w != MF_INFEASIBLE && word_dual(word) < need;
            };
            if (!failed) {
                double n0, n1;
                const bool want0 = wants(e0.y, w0, n0), want1 = wants(e1.y, w1, n1);
                failed |= (want0 && word_id(w0) < 0) || (want1 && word_id(w1) < 0);      // a free column would get a price
                if (!failed) {
                    const unsigned long long m0 = pack_word(n0, (int)(w0 & MF_ID_MASK)), m1 = pack_word(n1, (int)(w1 & MF_ID_MASK));
                    unsigned long long was0 = CORE_INF, was1 = CORE_INF;
                    if (want0) was0 = atomicMax(&s.otherword[e0.x], m0);
                    if (want1) was1 = atomicMax(&s.otherword[e1.x], m1);
                    const bool raised0 = was0 < m0, raised1 = was1 < m1;
                    unsigned st0 = round, st1 = round;
                    if (few) {                          // (a row set off twice: sorted out when they are handed on)
                        if (raised0 && !keep(word_id(w0))) failed = true;
                        if (raised1 && !keep(word_id(w1))) failed = true;
                    } else {
                        if (raised0) st0 = atomicExch(&a.stamp[e0.x], round);
                        if (raised1) st1 = atomicExch(&a.stamp[e1.x], round);
                        if (st0 != round) push(word_id(w0), next, counter);
                        if (st1 != round) push(word_id(w1), next, counter);
                    }
                }
                if (lane == 0 && profit < outside) {    // the list does not show everything this row might want: all of it, next round
                    const int at = atomicAdd(&ctl->whole_count[step_fills(epoch)], 1);
                    if (at < s.len) store_i32(&((epoch & 1u) ? a.whole0 : a.whole1)[at], i);
                    else failed = true;
                    atomicAdd(&sh.dense, 1);
                }
            }
            if (__any(failed)) { if (lane == 0) atomicOr(&sh.failed, 1u); break; }
            ++scans;
        }
        if (own >= CORE_OWN_ROUNDS || !few) break;
        __syncthreads();
        const unsigned end = min(sh.pushes, (unsigned)CORE_PUSH_BUFFER);
        const bool failed = sh.failed != 0u;
        __syncthreads();
        here = (int)(end - taken);
        if (failed || here == 0 || here > CORE_OWN_MOST) break;
        start = taken;
        taken = end;
        first = wave; stride = CORE_WAVES;
        }
        const int parts = whole_rows > 0 ? parts_of(s, whole_rows) : 1;
        int slice = 0;
        for (int it = gwave(); it < whole_rows * parts;) {
            const int row = it / parts, from = (it - row * parts + slice * parts) * CORE_SLICE;
            const int i = __builtin_amdgcn_readfirstlane(load_fresh_i32(&((epoch & 1u) ? a.whole1 : a.whole0)[row]));
            const int col = load_fresh_i32(&a.row2col[i]);
            const double profit = col >= 0 ? fma(a.Kd, (double)load_fresh_i32(&a.held_weight[i]), -word_dual(load_fresh_u64(&s.otherword[max(col, 0)]))) : 0.0;
            const int length = s.line_len ? min(s.line_len[i], s.len) : s.len, to = min(length, from + CORE_SLICE);
            if (from < to) {
                int4 ahead[CORE_SLICE / 256];
                load_slice(s.A + (size_t)i * s.pitch, from, to, ahead);
#pragma unroll
                for (int q = 0; q < CORE_SLICE / 256; ++q) {
                    const int j = from + q * 256 + lane * 4;
                    if (j >= to) break;
                    const int32_t w[4] = {ahead[q].x, ahead[q].y, ahead[q].z, ahead[q].w};
                    unsigned long long word[4];
#pragma unroll
                    for (int e = 0; e < 4; ++e) word[e] = load_fresh_u64(&s.otherword[min(j + e, to - 1)]);
                    for (int e = 0; e < 4; ++e) {
                        const double need = fma(a.Kd, (double)w[e], -profit);
                        if (j + e >= to || w[e] == MF_INFEASIBLE || !(word_dual(word[e]) < need)) continue;
                        if (word_id(word[e]) < 0) { atomicOr(&sh.failed, 1u); break; }
                        const unsigned long long mine = pack_word(need, (int)(word[e] & MF_ID_MASK));
                        if (!(atomicMax(&s.otherword[j + e], mine) < mine)) continue;
                        if (few) { if (!keep(word_id(word[e]))) atomicOr(&sh.failed, 1u); }
                        else if (atomicExch(&a.stamp[j + e], round) != round) push(word_id(word[e]), next, counter);
                    }
                }
                whole += (unsigned)(to - from + 3) / 4u;
            }
            if (from + parts * CORE_SLICE < length) ++slice;
            else { it += gwaves(); slice = 0; }
        }
        if (few) hand_on(next, counter, taken, round);
        else flush(next, counter);
        if (tid == 0 && sh.failed) atomicOr(&ctl->failed[round % 3u], 1u);
        if (tid == 0 && sh.dense) atomicAdd(&ctl->dense[step_fills(epoch)], (unsigned)sh.dense);
        if (!barrier()) return -1;
        ++epoch;
        if (load_fresh_u32(&ctl->failed[round % 3u]) != 0u) { done = 0; break; }        // (the next round writes the other two)
        count = load_fresh_i32(&ctl->cnt[step_reads(epoch)]);
        whole_rows = min(load_fresh_i32(&ctl->whole_count[step_reads(epoch)]), s.len);
        if (count + whole_rows == 0) { done = 1; break; }
        whole_lines += load_fresh_u32(&ctl->dense[step_reads(epoch)]);
        if (whole_lines > (unsigned)a.dense_limit) { done = 2; break; }
        // (on the way to a proof fewer and fewer rows are left; once more and more of them are, prices
        // are going round and round)
        unimproved += few ? CORE_OWN_ROUNDS + 1 : 1;
        if (count < fewest) { fewest = count; unimproved = 0; }
        if (round >= (unsigned)a.refine_rounds || unimproved > a.refine_patience || count > fewest + fewest / 4 + 64) { done = 0; break; }
    }
    if (gtid() == 0) steps += 1;
    return done;
}

// Ends the launch with everything the host, or the next launch, needs in memory.
template <bool LARGE>
__device__ __forceinline__ int Core<LARGE>::leave(int reason, int phase, int stage, int count, int parity)
{
    // (summed up by workgroup first: four atomics from each of 256 wavefronts, on four addresses, took a launch 15 to 30 us)
    __syncthreads();
    if (tid < 4) sh.list[tid] = 0ull;
    __syncthreads();
    CoreReport &out = ctl->out;
    unsigned long long *sums[4] = {&out.bids, &out.scans, &out.whole_groups, &out.rested};
    const unsigned mine[4] = {bids, scans, whole, rests};
    if (lane == 0) {
#pragma unroll
        for (int q = 0; q < 4; ++q)
            if (mine[q]) atomicAdd(&sh.list[q], (unsigned long long)mine[q]);
    }
    __syncthreads();
    if (tid == 0) {
#pragma unroll
        for (int q = 0; q < 4; ++q)
            if (sh.list[q]) atomicAdd(sums[q], sh.list[q]);
    }
    // a wait that runs out here still counts: the reason stays "a wait ran out"
    if (reason == MF_CORE_ABORT || !barrier()) return MF_CORE_ABORT;
    if (rank == 0 && wave == 0) {
        if (lane == 0) {
            out.reason = reason;
            out.phase = phase;
            out.stage = stage;
            out.count = count;
            out.parity = parity;
            out.columns_wait = sh.columns_wait;
            out.steps = steps;
            out.columns_ready = columns_ready;
            out.depth = depth;
        }
        tell_host(ctl, a.tell_to, a.told, a.number);
    }
    return reason;
}

template <bool LARGE>
__device__ __forceinline__ int Core<LARGE>::run()
{
    const CoreSide &fwd = a.side[0], &rev = a.side[1];
    int ph = a.first_phase, stage = a.first_stage, count = a.first_count;
    int left_rows = 0, left_cols = 0;
    if (tid == 0) sh.columns_wait = a.columns_wait;      // (barriers before anybody asks)
    double bid_budget = a.bid_limit;
    bool ok, fresh_lists = stage != MF_CORE_RESET;    // (the launch before this one asked for them)
    if (stage == MF_CORE_FORWARD_DONE) left_rows = count;
    if (stage == MF_CORE_REVERSE_DONE) left_cols = count;
    for (;;) {
        const double eps = a.eps[ph];
        // (added to at the end of a forward side: barriers of that side before it, of the next stage after it)
        const int stop = a.rested_before + load_fresh_u64(&ctl->out.rested) < (unsigned long long)a.growth_rest ? a.stop_grown[ph] : a.stop[ph];
        if (stage == MF_CORE_RESET && a.use_wide && !a.wide) return leave(MF_CORE_HANDOVER, ph, stage, 0, 0);
        if (stage == MF_CORE_RESET) {
            if (gtid() == 0) store_i32(&ctl->out.phase, ph);
            for (int k = gtid(); k < fwd.len; k += gsize()) {
                store_through(&fwd.otherword[k], pack_word(load_fresh(&fwd.other_dual[k]), 0));
                store_i32(&a.col2row[k], -1);
            }
            for (int i = gtid(); i < fwd.lines; i += gsize()) { store_i32(&a.row2col[i], -1); store_i32(&bidders(epoch)[i], i); }
            count = fwd.lines;
            stage = MF_CORE_FORWARD;                    // (slack_of's barriers end this)
        }
        if (stage == MF_CORE_FORWARD || stage == MF_CORE_REVERSE) {
            const bool forward = stage == MF_CORE_FORWARD;
            const CoreSide side = forward ? a.side[0] : a.side[1];
            bool risen;
            const double slack = slack_of(side, ok, &risen);
            if (!ok) return MF_CORE_ABORT;
            // duals that came down a long way make every list's bound useless: better lists first
            if (((slack > a.stale * eps && side.len > CORE_LIST) || risen) && !fresh_lists) {
                if (forward) write_duals(side);
                return leave(MF_CORE_RELIST, ph, stage, count, (int)(epoch & 1u));
            }
            fresh_lists = false;
            const int rc = run_bids(*this, side, eps, slack, stop, forward, count, bid_budget);
            if (rc) {
                if (rc != MF_CORE_ABORT) write_duals(side);
                return leave(rc, ph, stage, count, (int)(epoch & 1u));
            }
            if (forward) { left_rows = count; stage = MF_CORE_FORWARD_DONE; }
            else { left_cols = count; stage = MF_CORE_REVERSE_DONE; }
        }
        if (stage == MF_CORE_FORWARD_DONE) {
            if (lane == 0 && rests) atomicAdd(&ctl->out.rested, (unsigned long long)rests);
            rests = 0;
            for (int i = gtid(); i < fwd.lines; i += gsize()) {
                store_i32(&a.row2col[i], -1);
                store_f64(&rev.other_dual[i], 0.0);
                store_through(&a.rowword[i], 0ull);
            }
            int *next = bidders(epoch + 1u), *counter = &ctl->cnt[step_fills(epoch)];
            clear_ahead();
            if (tid == 0) sh.pushes = 0u;
            if (!barrier()) return MF_CORE_ABORT;
            for (int k = gtid(); k < fwd.len; k += gsize()) {
                const unsigned long long word = load_fresh_u64(&fwd.otherword[k]);
                const double p = word_dual(word);
                const int r = word_id(word);
                store_f64(&fwd.other_dual[k], p);
                store_i32(&a.col2row[k], r);
                if (r >= 0) {
                    const double pi = fma(a.Kd, (double)fwd.A[(size_t)r * fwd.pitch + k], -p);
                    store_i32(&a.row2col[r], k);
                    store_f64(&rev.other_dual[r], pi);
                    store_through(&a.rowword[r], pack_word(pi, k + 1));
                } else if (p > 0.0) push(k, next, counter);      // an unassigned column that still carries a price must bid
            }
            flush(next, counter);
            if (!barrier()) return MF_CORE_ABORT;
            ++epoch;
            count = load_fresh_i32(&ctl->cnt[step_reads(epoch)]);
            // Every row left over leaves a column unused, too, and columns are as a rule not asked to bid for that:
            // their lists (and, the first time, the transposed matrix) take a millisecond or two.  But an unused column
            // keeps the price a coarser phase drove it to, and with no better way out the first phase that runs to the end
            // would have to raise all others to it, epsilon by epsilon (20,000 x 20,000, one pair in two feasible: 4,800
            // search steps, 104 ms).  So in the phase before that one they bid.  Auctions without / with it: one pair
            // in 2, 3, 4, 6, 10 feasible 104 / 26, 72 / 21, 50 / 23, 50 / 33, 20 / 17 ms; sixteen 20,000 x 20,000 rounds
            // 28.2 / 24.8 (median), nine rounds after those 31.0 / 27.7.  In every phase: 28.1; also in the first on
            // lists: 28.6.
            const bool next_complete = ph + 1 >= a.n_phases || a.stop[ph + 1] == 0;
            const int most_unused = stop > 0 && !next_complete ? stop + left_rows : stop;
            if (left_rows > 0 && count > most_unused) {
                // rows that still wanted to bid get the profit that covers all of their pairs (see settle_unplaced_kernel)
                bool risen;
                const double slack = slack_of(fwd, ok, &risen);
                if (!ok) return MF_CORE_ABORT;
                for (int i = gwave(); i < fwd.lines; i += gwaves()) {
                    if (load_fresh_i32(&a.row2col[i]) >= 0) continue;
                    double outside;
                    const Top2 t = listed(fwd, i, slack, &outside);
                    const double pi = fmax(t.b1 < outside ? whole_line(fwd, i).b1 : t.b1, 0.0);
                    if (lane == 0) {
                        store_f64(&rev.other_dual[i], pi);
                        store_through(&a.rowword[i], pack_word(pi, 0));
                    }
                }
                if (!barrier()) return MF_CORE_ABORT;
            }
            left_cols = count;
            if (tid == 0) sh.columns_wait = columns_may_wait(count, left_rows, stop, a.path_max, CORE_MAX_SOURCES) ? 1 : 0;
            if (count > most_unused) {
                if (!a.have_columns) return leave(MF_CORE_COLUMNS, ph, MF_CORE_REVERSE, count, (int)(epoch & 1u));
                stage = MF_CORE_REVERSE;
                continue;
            }
            stage = MF_CORE_PHASE_DONE;
        }
        if (stage == MF_CORE_REVERSE_DONE) {
            for (int k = gtid(); k < fwd.len; k += gsize()) { store_i32(&a.col2row[k], -1); store_f64(&fwd.other_dual[k], 0.0); }
            if (!barrier()) return MF_CORE_ABORT;
            for (int i = gtid(); i < fwd.lines; i += gsize()) {
                const unsigned long long word = load_fresh_u64(&a.rowword[i]);
                const int k = word_id(word);
                store_i32(&a.row2col[i], k);
                store_f64(&rev.other_dual[i], word_dual(word));
                if (k >= 0) {
                    store_i32(&a.col2row[k], i);
                    store_f64(&fwd.other_dual[k], fma(a.Kd, (double)fwd.A[(size_t)i * fwd.pitch + k], -word_dual(word)));
                }
            }
            if (!barrier()) return MF_CORE_ABORT;
        }
        // (stage is now MF_CORE_PHASE_DONE, or the launch starts there)
        if (ph + 1 >= a.n_phases) return leave(MF_CORE_DONE, ph, MF_CORE_PHASE_DONE, 0, 0);
        if (left_rows == 0 && left_cols == 0 && eps <= a.refine_below && a.may_refine) {
            if (a.use_wide && !a.wide) return leave(MF_CORE_HANDOVER, ph, MF_CORE_PHASE_DONE, 0, 0);
            const int exact = refine(a.refined ? 0.0 : a.refine_lower * eps);      // (after new lists it goes on from the prices reached)
            fresh_lists = false;
            if (exact < 0) return MF_CORE_ABORT;
            if (exact == 2) {
                write_duals(fwd);
                return leave(MF_CORE_RELIST, ph, MF_CORE_PHASE_DONE, 0, 0);
            }
            if (exact > 0) {
                write_duals(fwd);
                return leave(MF_CORE_DONE, ph, MF_CORE_PHASE_DONE, 0, 0);
            }
        }
        ++ph;
        stage = MF_CORE_RESET;
    }
}

template <bool LARGE>
__global__ __launch_bounds__(CORE_THREADS) void core_kernel(CoreArgs a, CoreCtl *ctl)
{
    __shared__ CoreShared sh;
    Core<LARGE> core(a, ctl, sh);
    const int joined = core.join();
    if (joined != 1) return;                            // (not of that die, or a wait ran out: the reason stays as it was)
    (void)core.run();
}

// The control block as a launch wants to find it (one wavefront).
__device__ __forceinline__ void clear_control(CoreCtl *ctl, int lane)
{
    for (int k = lane; k < CORE_MAX_WORKGROUPS; k += 64) ctl->reached[k] = 0u;
    if (lane != 0) return;
    ctl->die = -1;
    ctl->told = 0u;
    ctl->joined = 0u; ctl->arrived = 0u; ctl->members = 0u;
    for (unsigned q = 0; q < STEP_RING; ++q) { ctl->cnt[q] = 0; ctl->whole_count[q] = 0; ctl->dense[q] = 0u; }
    ctl->out = CoreReport{MF_CORE_ABORT, -1, MF_CORE_RESET, 0, 0, 0, 0u, 0ull, 0ull, 0ull, 0ull, 0ull, 0ull};
}

__global__ __launch_bounds__(64) void core_clear_kernel(CoreCtl *ctl) { clear_control(ctl, threadIdx.x); }

// Tells the host how a launch ended, if that has not (a wait ran out), and leaves the control block clear for the next one.
__global__ __launch_bounds__(64) void core_report_kernel(CoreCtl *ctl, void *to, unsigned *told, unsigned number)
{
    if (ctl->told == 0u) {
        tell(&ctl->out, to, (int)(sizeof(CoreReport) / 4), threadIdx.x);
        tell_number(told, number, threadIdx.x);
    }
    clear_control(ctl, threadIdx.x);
}

}  // namespace

namespace {

void launch_lists(mf_ctx *ctx, const SideArgs &s, int made, int stride, const int *list, int which, double *depth, const double *own_dual, const int *partner,
                  double *built)
{
#define MF_LIST(LINES)                                                                                                                     \
    hipLaunchKernelGGL((core_list_kernel<LINES>), dim3((made + LINES - 1) / LINES), dim3(LIST_THREADS), 0, ctx->stream, s.A, s.pitch, s.len, \
                       s.line_len, made, stride, list, s.other_dual, s.Kd, ctx->core_entries[which], ctx->core_bound[which], ctx->core_half_bound[which], depth, own_dual, partner, built, list ? 1 : 0, \
                       s.Kd * (double)ctx->h_stats->max_weight)
    if (made > 8 * ctx->n_cus) MF_LIST(4); else if (made > 4 * ctx->n_cus) MF_LIST(2);
    else MF_LIST(1);
#undef MF_LIST
}

}  // namespace

// Lists of a side's lines for its opposite duals as they are; with `partner`, of those that may bid.
int mf_core_lists(mf_ctx *ctx, const SideArgs &s, int lines, int which, const double *own_dual, const int *partner)
{
    if (s.len <= CORE_LIST) partner = nullptr;          // whole lines: they never have to be made again
    launch_lists(ctx, s, lines, 1, nullptr, which, ctx->core_reach[which], own_dual, partner, ctx->core_built[which]);
    MF_HIP(hipGetLastError());
    return MF_OK;
}

// The same for `count` lines only, those in `list` (device); the others' lists stay as they are.
int mf_core_lists_of(mf_ctx *ctx, const SideArgs &s, const int *list, int count, int which)
{
    if (count <= 0) return MF_OK;
    launch_lists(ctx, s, count, 1, list, which, ctx->core_reach[which], nullptr, nullptr, ctx->core_built[which]);
    MF_HIP(hipGetLastError());
    return MF_OK;
}

// How far below a line's best value its list would reach, for a sample of lines: *deep becomes the
// share of them that reach at least `distance`.
int mf_core_probe(mf_ctx *ctx, const SideArgs &s, int lines, double distance, double *deep)
{
    const int stride = (lines + MF_CORE_PROBES - 1) / MF_CORE_PROBES, probes = (lines + stride - 1) / stride;
    launch_lists(ctx, s, probes, stride, nullptr, 0, ctx->core_depth, nullptr, nullptr, nullptr);
    MF_HIP(hipGetLastError());
    const int rc = mf_send_and_await(ctx, mf_report{{{ctx->core_depth, ctx->h_core_depth, 2 * probes}}});
    if (rc != MF_OK) return rc;
    int n = 0;
    for (int k = 0; k < probes; ++k) n += ctx->h_core_depth[k] >= distance;
    *deep = (double)n / probes;
    return MF_OK;
}

int mf_core_launch(mf_ctx *ctx, const SideArgs &fwd, const SideArgs &rev, int rn, int rm, const mf_core_plan &plan, mf_core_state *st)
{
    CoreArgs a{};
    // (by default a quarter of the matrix, at least eight million entries: about 3 ms on one die at 20,000 x 20,000)
    auto read_limit = [ctx](const SideArgs &side, int lines) {
        const long long all = (long long)lines * side.len * ctx->core_read / 100, entries = all > ctx->core_read_least ? all : ctx->core_read_least;
        return entries / (side.typical_len > 1 ? side.typical_len : 1);
    };
    a.side[0] = CoreSide{fwd.A, fwd.pitch, rn, rm, read_limit(fwd, rn), fwd.line_len, ctx->colword, ctx->price, ctx->core_entries[0], ctx->core_t_start[0], ctx->core_t_at[0], ctx->core_t_entries[0], ctx->core_bound[0], ctx->core_half_bound[0], ctx->core_built[0], ctx->core_reach[0]};
    a.side[1] = CoreSide{rev.A, rev.pitch, rm, rn, read_limit(rev, rm), rev.line_len, ctx->roword, ctx->profit, ctx->core_entries[1], ctx->core_t_start[1], ctx->core_t_at[1], ctx->core_t_entries[1], ctx->core_bound[1], ctx->core_half_bound[1], ctx->core_built[1], ctx->core_reach[1]};
    a.Kd = fwd.Kd;
    for (int k = 0; k < plan.n_phases; ++k) { a.eps[k] = (double)plan.eps[k]; a.stop[k] = plan.stop[k]; a.stop_grown[k] = plan.stop_grown[k]; }
    a.n_phases = plan.n_phases;
    a.first_phase = st->phase; a.first_stage = st->stage; a.first_count = st->count; a.first_parity = st->parity;
    a.columns_wait = st->columns_wait;
    a.growth_rest = ctx->phase_growth_rest;
    a.rested_before = plan.rested_before;
    a.have_columns = plan.have_columns ? 1 : 0;
    a.may_refine = plan.may_refine ? 1 : 0;
    a.stale = plan.stale;
    a.stale_rise = 0.35;
    a.refine_below = plan.refine_below;
    a.refine_rounds = 256;
    a.refine_patience = 40;
    a.refine_lower = 256.0;
    a.path_max = ctx->path_max;
    {
        // (a search of a small problem costs less than long chains of its last bidders: with 256 steps for every size /
        // with this rule rounds of 64 x 64 take 0.95 / 0.79 ms, 1024 x 1024 2.37 / 2.28, from 1664 rows on the same)
        const long long share = 48 + rn / 8, after = ctx->core_after * (share < 256 ? share : 256) / 256;
        a.path_after = ctx->path_after < after ? ctx->path_after : after;
    }
    a.tail_steps = ctx->phase_tail_sides ? ctx->phase_tail_steps : 0;
    a.tail_always = rn >= ctx->phase_tail_from ? 1 : 0;
    a.steps_many = ctx->core_many; a.steps_few = ctx->core_few;
    a.path_width = (double)ctx->core_width;
        a.frontier_high = ctx->path_frontier_rows;
    a.spin_limit = ctx->path_spin_limit;
    a.columns_ready = st->columns_ready;
    a.base = ctx->core_base; a.dropped = ctx->core_dropped; a.tree = ctx->core_tree;
    a.wide = st->wide; a.use_wide = plan.use_wide ? 1 : 0; a.narrow_at = ctx->core_narrow; a.refined = st->refined;
    a.dense_limit = 128 + rn / 64;
    {
        // a small problem needs few wavefronts, and a barrier over few workgroups is short
        const int want = (rm + 31) / 32, most = st->wide ? CORE_MAX_WORKGROUPS : 64;
        a.workgroups = want < most ? want : most;
    }
    a.frontier_room = (int)((ctx->max_n > ctx->max_m ? ctx->max_n : ctx->max_m) * 16ll < (1ll << 30) ? (ctx->max_n > ctx->max_m ? ctx->max_n : ctx->max_m) * 16ll : (1ll << 30));
    a.bid_limit = plan.bid_limit;
    a.row2col = ctx->row2col; a.col2row = ctx->col2row; a.rowword = ctx->roword;
    a.list0 = ctx->list[0]; a.list1 = ctx->list[1];
    a.label = ctx->path_label; a.expanded = ctx->path_expanded;
    a.frontier0 = ctx->path_frontier[0]; a.frontier1 = ctx->path_frontier[1];
    a.stamp = ctx->path_stamp; a.held = ctx->path_held; a.jump = ctx->path_jump;
    a.parent = ctx->core_parent; a.read_from = ctx->core_read_from; a.left = ctx->path_base; a.whole0 = ctx->path_tree; a.whole1 = ctx->path_parent; a.held_weight = ctx->core_weight;
    CoreCtl *ctl = (CoreCtl *)ctx->core_ctl;
    if (!ctx->core_clear) hipLaunchKernelGGL(core_clear_kernel, dim3(1), dim3(64), 0, ctx->stream, ctl);
    ctx->core_clear = false;
    // one workgroup per compute unit of the device: those of one die stay
    const unsigned report = ++ctx->reports;
    a.tell_to = ctx->h_core_report; a.told = &ctx->h_told->number; a.number = report;
    hipLaunchKernelGGL(plan.use_wide ? core_kernel<true> : core_kernel<false>, dim3(ctx->n_cus), dim3(CORE_THREADS), 0, ctx->stream, a, ctl);
    MF_HIP(hipGetLastError());
    hipLaunchKernelGGL(core_report_kernel, dim3(1), dim3(64), 0, ctx->stream, ctl, ctx->h_core_report, &ctx->h_told->number, report);
    MF_HIP(hipGetLastError());
    const int rc = mf_await(ctx, report);
    if (rc != MF_OK) return rc;
    ctx->core_clear = true;                             // (behind the report, and before anything else on the stream)
    const CoreReport &h = *(const CoreReport *)ctx->h_core_report;
    st->by_column += __builtin_popcount(h.columns_ready & ~st->columns_ready);
    st->columns_ready = h.columns_ready;
    st->refined = h.reason == MF_CORE_RELIST && h.stage == MF_CORE_PHASE_DONE;
    st->reason = h.reason; if (h.phase >= 0) st->phase = h.phase; st->stage = h.stage; st->count = h.count; st->parity = h.parity; st->columns_wait = h.columns_wait;
    st->bids += (long long)h.bids; st->depth += (long long)h.depth; st->steps += (long long)h.steps; st->scans += (long long)h.scans;
    st->rested += (long long)h.rested;
    st->launches += 1;
    // (a bid counts as a whole list, also where the first half of it decided)
    st->bytes += (long long)(h.bids + h.scans) * CORE_LIST * 8 + (long long)h.whole_groups * 16;
    return MF_OK;
}

size_t mf_core_ctl_bytes() { return sizeof(CoreCtl); }
size_t mf_core_report_bytes() { return sizeof(CoreReport); }

