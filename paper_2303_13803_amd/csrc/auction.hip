// Maximum-weight bipartite matching of the scored graph (paper: Algorithm
// "Scheduling algorithm", GetMatching; Section "Matching-based scheduling"
// states the problem and asks for the optimal matching).
//
// The paper solves it with the sequential Kuhn-Munkres algorithm.  Here the
// same optimum is reached by an epsilon-scaling forward/reverse auction, whose
// unit of work - "scan one line of the weight matrix against the current duals
// and keep the best two" - is a coalesced streaming read, and whose updates are
// 64-bit atomic maxima.  Weights are multiplied by K = min(n, m) + 1 so that the final
// epsilon = 1 is below 1/min(n, m) of a weight unit: the matching is then exactly
// optimal, and the duals it leaves behind prove it (see certificate_kernel).
//
// Formulation.  maximise sum W_ij x_ij, every row and column used at most
// once.  Dual: minimise sum pi_i + sum p_j with pi_i + p_j >= K W_ij, pi, p >= 0.
// The auction keeps, for the current epsilon,
//   (I1) pi_i + p_j >= K W_ij - eps on every feasible pair,
//   (I2) pi_i + p_j  = K W_ij      on every assigned pair,
// and stops a phase when every unassigned row has pi_i = 0 and every
// unassigned column has p_j = 0; then the assignment is within min(n, m)*eps of the
// optimum.  A forward round lets unassigned rows raise prices p; a reverse
// round lets unassigned columns that still carry a positive price raise
// profits pi (and lower their own price).  Both are the same computation with
// the roles of rows and columns exchanged, so one pair of kernels serves both,
// reading W for forward rounds and its transpose for reverse rounds.
//
// All dual values are integers below 2^43; the scans evaluate K*w - dual in
// double precision, where such integers and their differences are exact, so
// that they run at the full rate of the FP64 vector units.
#include "scan.h"
#include "report.h"

namespace {

// One round for many bidders: a workgroup per bidder, bids taking effect at
// once.  Later bidders of the same round may already see them (or a slightly
// older dual): the auction tolerates both because duals only move one way and a
// bid computed from an outdated dual simply fails to win.  The counters form a
// ring: launch r reads cnt[r], fills cnt[r+1] and clears cnt[r+2].
//
// A bid sets off at most one bidder (the holder it displaced, or itself), who takes its place in the next round's list: no
// counter is touched.  Places where nobody has to go on hold -1, and compact_kernel takes them out before the
// host, or any other kernel, looks at the list; what a place has cost since it was last full (its bids, its words read) adds up
// in `work` until then.  (Handing bidders over by atomics on one counter, one a workgroup, bounded these rounds: 10 ns each, and
// the workgroups that started meanwhile waited 7 us to read the count on the same line.  Rounds of 3000, 2000 and 1200 bidders
// on lines of 6001 to 9007 entries 45 -> 26, 36 -> 24 and 26 -> 15 us; compact_kernel takes 5 us, once for three of them.)
__device__ __forceinline__ unsigned long long work_of(unsigned long long words) { return (1ull << MF_WORK_WORDS) + words; }

template <int NT, int RB>
__global__ __launch_bounds__(NT, 3) void round_kernel(SideArgs s, const int *__restrict__ list,
                                                   int *__restrict__ next, mf_device_stats *stats,
                                                   int ring, unsigned long long *__restrict__ work, int full)
{
    __shared__ Top2 red[RB + RB * (NT / 64)];
    const int count = stats->cnt[ring & 3];
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        stats->cnt[(ring + 1) & 3] = count;
        stats->cnt[(ring + 2) & 3] = 0;
        stats->head = 0;
        stats->round_at = device_time();
        if (count > 0) stats->rounds += 1ull;
    }
    for (int item = blockIdx.x * RB; item < count; item += gridDim.x * RB) {
        int salt[RB], len = s.len;                          // (lines of different lengths go one by one)
        const int32_t *rows[RB];
        bool any = false;
#pragma unroll
        for (int r = 0; r < RB; ++r) {
            const int b = list[min(item + r, count - 1)];   // a short last group repeats its last line
            any |= b >= 0;
            rows[r] = s.A + (size_t)max(b, 0) * s.pitch;
            salt[r] = tie_salt(max(b, 0));
            if (RB == 1) len = line_length(s, max(b, 0));
        }
        if (!any) {                                         // (the same in the whole workgroup)
            if (threadIdx.x < RB && item + (int)threadIdx.x < count) next[item + threadIdx.x] = -1;
            continue;
        }
        block_scan_rows<NT, RB>(rows, salt, s.other_dual, len, s.Kd, red);
        if (threadIdx.x < RB && item + (int)threadIdx.x < count) {      // one lane bids per line
            const int place = item + threadIdx.x, b = list[place];
            int again = -1;
            if (b >= 0) {
                Top2 t = red[threadIdx.x];
                t.idx ^= tie_salt(b);
                again = decide_and_bid<true>(s, b, t);
                work[place] = (full ? 0ull : work[place]) + work_of((unsigned long long)len);
            }
            next[place] = again;
        }
    }
}

// The bidders left by the rounds since the list was last full, one behind the other, and what those rounds have cost.
constexpr int COMPACT_THREADS = 1024;

__global__ __launch_bounds__(COMPACT_THREADS) void compact_kernel(const int *__restrict__ list, int *__restrict__ next,
                                                                  mf_device_stats *stats, int ring, const unsigned long long *__restrict__ work)
{
    constexpr int WAVES = COMPACT_THREADS / 64;
    __shared__ int s_count[WAVES], s_base;
    __shared__ unsigned long long s_bids[WAVES], s_words[WAVES];
    const int count = stats->cnt[ring & 3], lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        stats->cnt[(ring + 2) & 3] = 0;
        stats->round_end = device_time();
    }
    for (int first = blockIdx.x * COMPACT_THREADS; first < count; first += gridDim.x * COMPACT_THREADS) {
        const int item = first + threadIdx.x;
        const int b = item < count ? list[item] : -1;
        const unsigned long long done = item < count ? work[item] : 0ull, going = __ballot(b >= 0);
        unsigned long long bids = done >> MF_WORK_WORDS, words = done & ((1ull << MF_WORK_WORDS) - 1ull);
        for (int off = 32; off >= 1; off >>= 1) { bids += __shfl_xor(bids, off); words += __shfl_xor(words, off); }
        if (lane == 0) { s_count[wave] = __popcll(going); s_bids[wave] = bids; s_words[wave] = words; }
        __syncthreads();
        if (threadIdx.x == 0) {
            int total = 0;
            for (int w = 0; w < WAVES; ++w) { const int c = s_count[w]; s_count[w] = total; total += c; }
            for (int w = 1; w < WAVES; ++w) { bids += s_bids[w]; words += s_words[w]; }
            s_base = total ? atomicAdd(&stats->cnt[(ring + 1) & 3], total) : 0;
            atomicAdd(&stats->bids, bids);
            atomicAdd(&stats->round_bytes, words * 4ull);
        }
        __syncthreads();
        if (b >= 0) next[s_base + s_count[wave] + __popcll(going & ((1ull << lane) - 1ull))] = b;
        __syncthreads();                                    // before the next stretch overwrites the counts
    }
}

// The tail of a run.  When few bidders are left, rounds are bound by launch
// latency and the work is a handful of chains: a bid evicts a holder, who bids
// next, and so on.  Each workgroup takes a pending bidder and then follows its
// chain - after every bid it goes on with whoever has to bid because of it -
// so no workgroup creates work for another, none waits for another, and each
// stops as soon as the list is used up.  `stats->active` counts the workgroups
// still following a chain; once it is at most `hand_back_at` the rest hand their
// bidders back, so that the host can put several workgroups on each chain.
constexpr int CHAIN_THREADS = 1024;

__global__ __launch_bounds__(CHAIN_THREADS) void chain_kernel(SideArgs s, const int *__restrict__ list,
                                                              int *__restrict__ out_list,
                                                              mf_device_stats *stats, int ring,
                                                              long long step_cap, int hand_back_at)
{
    __shared__ Top2 red[CHAIN_THREADS / 64];
    __shared__ int s_next, s_active;
    if (threadIdx.x == 0) s_active = 0x7fffffff;
    const int count = stats->cnt[ring & 3];
    unsigned long long steps = 0, retries = 0, scanned = 0;
    bool handing_back = false;              // block-uniform
    for (;;) {
        __syncthreads();
        if (threadIdx.x == 0) s_next = atomicAdd(&stats->head, 1);
        __syncthreads();
        const int item = s_next;
        if (item >= count) break;
        int b = list[item];
        if (handing_back) {                 // pass on what nobody will bid for in this launch
            if (threadIdx.x == 0) out_list[atomicAdd(&stats->cnt[(ring + 1) & 3], 1)] = b;
            continue;
        }
        bool fresh = false;                 // re-read the duals past the caches after a bid that lost
        while (b >= 0) {
            if ((steps & 3) == 0) {         // now and then: how many workgroups still follow a chain?
                __syncthreads();
                if (threadIdx.x == 0)
                    s_active = __hip_atomic_load(&stats->active, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                __syncthreads();
            }
            if ((long long)steps >= step_cap || s_active <= hand_back_at) {
                if (threadIdx.x == 0) out_list[atomicAdd(&stats->cnt[(ring + 1) & 3], 1)] = b;
                handing_back = true;
                break;
            }
            ++steps;
            const int len = line_length(s, b);
            scanned += (unsigned long long)len;
            Top2 t = block_scan<CHAIN_THREADS>(s.A + (size_t)b * s.pitch, s.other_dual, len, s.Kd, fresh, red,
                                               0, tie_salt(b));
            t.idx ^= tie_salt(b);
            if (threadIdx.x == 0) s_next = decide_and_bid(s, b, t);
            __syncthreads();
            fresh = (s_next == b);
            if (fresh && threadIdx.x == 0) ++retries;
            b = s_next;
        }
        // handed back: follow no further chain, but keep emptying the list - if every workgroup
        // stopped here, entries nobody had claimed yet would never reach the next launch
    }
    if (threadIdx.x == 0) {
        atomicAdd(&stats->active, -1);      // this workgroup follows no chain any more
        if (steps) {
            atomicAdd(&stats->bids, steps);
            atomicAdd(&stats->chain_bids, steps);
            atomicAdd(&stats->bytes, scanned * 4ull);
            atomicMax(&stats->launch_max, steps);
            if (retries) atomicAdd(&stats->chain_retries, retries);
        }
    }
}

__global__ void chain_begin_kernel(mf_device_stats *stats, int ring, int workgroups)
{
    stats->head = 0;
    stats->active = workgroups;
    stats->cnt[(ring + 1) & 3] = 0;
    stats->cnt[(ring + 2) & 3] = 0;
    stats->rounds += 1ull;
    stats->chain_depth += stats->launch_max;     // of the previous chain kernel
    stats->launch_max = 0;
}

// The last few chains.  One compute unit cannot keep enough memory requests in
// flight to read a 100 KB line in much under ten microseconds, and with one
// or two chains left that latency is all there is.  Here TEAM_SIZE workgroups
// (on as many compute units) share each step of one chain: the leader
// publishes the bidder, every member scans its slice of the line and posts
// its top-2, the leader merges them, bids and publishes the next bidder.
// Members only ever wait for their leader and the leader for its members;
// every wait is bounded, and a wait that runs out raises `abort` so that all
// workgroups leave and the host falls back to chain_kernel.
constexpr int TEAM_SIZE_MAX = 32;        // workgroups per chain (run-time choice up to this)
constexpr int TEAM_MAX = 64;             // chains served at once
constexpr int TEAM_WIDE_MIN_LINE = 8192; // shortest line for which many small teams pay
constexpr unsigned TEAM_SPIN_LIMIT = 1u << 21;

struct alignas(128) TeamCtl {
    unsigned long long cmd;             // sequence << 32 | fresh << 31 | (bidder + 1); bidder + 1 == 0: stop
    unsigned int abort;
    unsigned int pad0;
    unsigned long long pad[14];
    // a member's result: three words, each carrying the low 8 bits of the step's sequence number,
    // so that the leader can tell a word of this step from the previous one without any fence:
    // best << 8 | tag, second << 8 | tag, index << 40 | (weight & 0xffffffff) << 8 | tag
    unsigned long long partial[TEAM_SIZE_MAX][4];
};

__device__ inline unsigned long long tag_value(double v, unsigned tag)
{
    const double c = fmin(fmax(v, -4.0e15), 4.0e15);        // integers up to 2^52 in magnitude
    return ((unsigned long long)(long long)c << 8) | (unsigned long long)(tag & 0xffu);
}
__device__ inline double untag_value(unsigned long long w)
{
    return (double)((long long)w >> 8);
}

__global__ void team_begin_kernel(mf_device_stats *stats, TeamCtl *ctl, int ring)
{
    const int t = threadIdx.x;
    if (t < TEAM_MAX) {
        ctl[t].cmd = 0ull; ctl[t].abort = 0u;
        for (int k = 0; k < TEAM_SIZE_MAX; ++k) { ctl[t].partial[k][0] = 0ull; ctl[t].partial[k][1] = 0ull; ctl[t].partial[k][2] = 0ull; }
    }
    if (t == 0) {
        stats->head = 0;
        stats->cnt[(ring + 1) & 3] = 0;
        stats->cnt[(ring + 2) & 3] = 0;
        stats->rounds += 1ull;
        stats->chain_depth += stats->launch_max;
        stats->launch_max = 0;
    }
}

template <int NT>
__global__ __launch_bounds__(NT) void team_kernel(SideArgs s, const int *__restrict__ list,
                                                  int *__restrict__ out_list, mf_device_stats *stats,
                                                  TeamCtl *ctl_all, int ring, long long step_cap,
                                                  int TEAM_SIZE)
{
    __shared__ Top2 red[NT / 64];
    __shared__ long long s_word;
    TeamCtl *ctl = ctl_all + blockIdx.x / TEAM_SIZE;
    const int member = blockIdx.x % TEAM_SIZE;
    const int count = stats->cnt[ring & 3];
    // the members share a line in equal slices of what has to be read of it
    auto slice_of = [&](int b, int &off) {
        const int len = line_length(s, b);
        const int slice = (((len + TEAM_SIZE - 1) / TEAM_SIZE) + 3) & ~3;
        off = member * slice;
        return max(0, min(slice, len - off));
    };

    if (member != 0) {
        // ---- member: wait for the leader's next command, scan, post ----
        unsigned expect = 1;
        for (;;) {
            __syncthreads();
            if (threadIdx.x == 0) {
                unsigned long long c = 0ull;
                unsigned spins = 0;
                for (;;) {
                    c = load_fresh_u64(&ctl->cmd);
                    if ((unsigned)(c >> 32) == expect) break;
                    ++spins;
                    if (spins > TEAM_SPIN_LIMIT || ((spins & 255u) == 0u && load_fresh_u32(&ctl->abort))) { c = 0ull; break; }
                }
                if (c == 0ull) atomicExch(&ctl->abort, 1u);
                s_word = (long long)c;
            }
            __syncthreads();
            const unsigned long long c = (unsigned long long)s_word;
            const int b = (int)(c & 0x7fffffffull) - 1;
            if (b < 0) break;                                   // stop (or abort)
            // a slice is small enough to stay in this compute unit's cache from step to step, so the
            // duals are always read past the caches here
            int off;
            const int my_len = slice_of(b, off);
            const Top2 t = block_scan<NT>(s.A + (size_t)b * s.pitch + off, s.other_dual + off, my_len, s.Kd,
                                          true, red, off, tie_salt(b));
            if (threadIdx.x == 0) {
                const int idx = t.idx == 0x7fffffff ? 0 : t.idx;      // already a key on the global index
                store_through(&ctl->partial[member][0], tag_value(t.b1, expect));
                store_through(&ctl->partial[member][1], tag_value(t.b2, expect));
                store_through(&ctl->partial[member][2], ((unsigned long long)(unsigned)idx << 40) |
                                                            ((unsigned long long)(unsigned)t.w << 8) | (expect & 0xffu));
            }
            ++expect;
        }
        return;
    }

    // ---- leader: follow chains, one command per step ----
    unsigned seq = 0;
    unsigned long long steps = 0, retries = 0, scanned = 0;
    bool dead = false;
    while (!dead) {
        __syncthreads();
        if (threadIdx.x == 0) s_word = atomicAdd(&stats->head, 1);
        __syncthreads();
        const int item = (int)s_word;
        if (item >= count) break;
        int b = list[item];
        bool fresh = false;
        while (b >= 0) {
            if ((long long)steps >= step_cap) {
                if (threadIdx.x == 0) out_list[atomicAdd(&stats->cnt[(ring + 1) & 3], 1)] = b;
                dead = true;
                break;
            }
            ++steps;
            ++seq;
            if (threadIdx.x == 0)
                store_through(&ctl->cmd, ((unsigned long long)seq << 32) | (fresh ? 0x80000000ull : 0ull) |
                                             (unsigned long long)(b + 1));
            int off;
            const int my_len = slice_of(b, off);                       // member 0: off == 0
            scanned += (unsigned long long)line_length(s, b);
            const Top2 t = block_scan<NT>(s.A + (size_t)b * s.pitch, s.other_dual, my_len, s.Kd, true, red, 0,
                                          tie_salt(b));
            if (threadIdx.x < 64) {                         // first wavefront: one lane per member
                const int k = threadIdx.x;
                Top2 mine = t;                              // lane 0: the leader's own slice
                int ok = 1;
                if (k >= TEAM_SIZE) {
                    mine = Top2{NEG_HUGE, NEG_HUGE, 0x7fffffff, 0};
                } else if (k >= 1) {                        // wait for member k's three words of this step
                    const unsigned tag = seq & 0xffu;
                    unsigned long long w0, w1, w2;
                    unsigned spins = 0;
                    for (;;) {
                        w0 = load_fresh_u64(&ctl->partial[k][0]);
                        w1 = load_fresh_u64(&ctl->partial[k][1]);
                        w2 = load_fresh_u64(&ctl->partial[k][2]);
                        if ((w0 & 0xffu) == tag && (w1 & 0xffu) == tag && (w2 & 0xffu) == tag) break;
                        ++spins;
                        if (spins > TEAM_SPIN_LIMIT || ((spins & 255u) == 0u && load_fresh_u32(&ctl->abort))) { ok = 0; break; }
                    }
                    mine.b1 = untag_value(w0);
                    mine.b2 = untag_value(w1);
                    mine.idx = (int)(w2 >> 40);
                    mine.w = (int)(unsigned)((w2 >> 8) & 0xffffffffull);
                }
                ok = __all(ok);
                if (ok) {
                    mine = wave_top2(mine);
                    mine.idx ^= tie_salt(b);
                    if (threadIdx.x == 0) s_word = decide_and_bid(s, b, mine);
                } else if (threadIdx.x == 0) {
                    atomicExch(&ctl->abort, 1u);
                    out_list[atomicAdd(&stats->cnt[(ring + 1) & 3], 1)] = b;
                    s_word = -2;
                }
            }
            __syncthreads();
            const int next = (int)s_word;
            if (next == -2) { dead = true; break; }
            fresh = (next == b);
            retries += fresh;
            b = next;
        }
    }
    if (threadIdx.x == 0) {
        store_through(&ctl->cmd, (unsigned long long)(seq + 1) << 32);      // stop
        if (load_fresh_u32(&ctl->abort)) atomicExch(&stats->team_abort, 1);
        if (steps) {
            atomicAdd(&stats->bids, steps);
            atomicAdd(&stats->chain_bids, steps);
            atomicAdd(&stats->team_bids, steps);
            atomicAdd(&stats->bytes, scanned * 4ull);
            atomicMax(&stats->launch_max, steps);
            if (retries) atomicAdd(&stats->chain_retries, retries);
        }
    }
}

// Start of an epsilon phase: drop the assignment, keep the duals, all rows bid.
__global__ void reset_kernel(int n, int m, const double *__restrict__ price,
                             unsigned long long *colword, int *row2col, int *col2row, int *list,
                             mf_device_stats *stats, unsigned long long *times)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i == 0 && times[AT_PREPARED] == 0ull) times[AT_PREPARED] = device_time();
    if (i < n) { row2col[i] = -1; list[i] = i; }
    if (i < m) { col2row[i] = -1; colword[i] = pack_word(price[i], 0); }
    if (i == 0) { stats->cnt[0] = n; stats->cnt[1] = 0; stats->cnt[2] = 0; stats->cnt[3] = 0; }
}

// After the forward rounds the price words name every column's holder, and a
// row's profit is whatever its column leaves it (0 for a row that rests).
__global__ void forward_done_rows_kernel(int n, double *__restrict__ profit,
                                         unsigned long long *roword, int *row2col, mf_device_stats *stats)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i == 0) { stats->cnt[0] = 0; stats->cnt[1] = 0; stats->cnt[2] = 0; stats->cnt[3] = 0; }
    if (i < n) { row2col[i] = -1; profit[i] = 0.0; roword[i] = 0ull; }
}

__global__ void forward_done_cols_kernel(int m, const int32_t *__restrict__ W, int64_t ldw, double Kd,
                                         const unsigned long long *__restrict__ colword,
                                         const double *__restrict__ price, double *__restrict__ profit,
                                         unsigned long long *roword, int *row2col, int *col2row,
                                         int *list, mf_device_stats *stats)
{
    const int j = blockIdx.x * blockDim.x + threadIdx.x;
    if (j >= m) return;
    const unsigned long long word = colword[j];
    const int r = word_id(word);
    col2row[j] = r;
    if (r >= 0) {
        const double pi = Kd * (double)W[(size_t)r * ldw + j] - word_dual(word);
        row2col[r] = j;
        profit[r] = pi;
        roword[r] = pack_word(pi, j + 1);
    } else if (price[j] > 0.0) {
        list[atomicAdd(&stats->cnt[0], 1)] = j;    // an unassigned column that still carries a price must bid
    }
}

// A forward side that was stopped early leaves rows that still wanted to bid.  Before the other
// side runs, each gets the profit that covers all of its pairs at the current prices (its best
// value, or 0), held by nobody: then pi_i + p_j >= K W_ij - eps holds on every feasible pair
// again, which the bids and searches of the other side rely on.
__global__ __launch_bounds__(BID_THREADS) void settle_unplaced_kernel(
    const int32_t *__restrict__ W, int64_t ldw, int n, int m, const double *__restrict__ price,
    const int *__restrict__ row2col, double Kd, double *__restrict__ profit, unsigned long long *roword,
    const int *__restrict__ line_len)
{
    __shared__ Top2 red[BID_THREADS / 64];
    for (int i = blockIdx.x; i < n; i += gridDim.x) {
        if (row2col[i] >= 0) continue;                               // block-uniform
        const int len = line_len ? min(line_len[i], m) : m;
        const Top2 t = block_scan<BID_THREADS>(W + (size_t)i * ldw, price, len, Kd, false, red, 0, 0);
        if (threadIdx.x == 0) {
            const double pi = fmax(t.b1, 0.0);
            profit[i] = pi;
            roword[i] = pack_word(pi, 0);
        }
        __syncthreads();
    }
}

// After the reverse rounds the profit words name every row's holder; a column's
// price is whatever its row leaves it (0 for a column that rests).
__global__ void reverse_done_cols_kernel(int m, double *__restrict__ price, int *col2row)
{
    const int j = blockIdx.x * blockDim.x + threadIdx.x;
    if (j < m) { col2row[j] = -1; price[j] = 0.0; }
}

__global__ void reverse_done_rows_kernel(int n, const int32_t *__restrict__ W, int64_t ldw, double Kd,
                                         const unsigned long long *__restrict__ roword,
                                         double *__restrict__ price, int *row2col, int *col2row)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const unsigned long long word = roword[i];
    const int c = word_id(word);
    row2col[i] = c;
    if (c >= 0) {
        col2row[c] = i;
        price[c] = Kd * (double)W[(size_t)i * ldw + c] - word_dual(word);
    }
}

// W^T (for the reverse rounds' coalesced column scans) and the largest weight.
// 64 x 64 tiles through LDS, 16-byte loads and stores on both sides.
// len_rows / len_cols (null: whole lines): entries of row i at or beyond len_rows[i] are infeasible and not read, and
// entries of column j at or beyond len_cols[j], which does not grow with j, will not be: tiles of nothing else are
// left out (20,000 x 40,000 with prefixes of a tenth: 1.24 -> 0.12 ms).
__global__ __launch_bounds__(256) void transpose_kernel(const int32_t *__restrict__ W, int n, int m, int64_t ldw,
                                                        int32_t *__restrict__ WT, int64_t ldt,
                                                        const int *__restrict__ len_rows, const int *__restrict__ len_cols,
                                                        mf_device_stats *stats)
{
    __shared__ int32_t tile[64][65];
    const int bx = blockIdx.x * 64, by = blockIdx.y * 64;
    if (len_cols && by >= len_cols[bx]) return;
    const int q4 = (threadIdx.x & 15) * 4, rr = threadIdx.x >> 4;       // 16 threads per line, 16 lines per pass
    int mx = 0;
#pragma unroll
    for (int p = 0; p < 4; ++p) {
        const int r = p * 16 + rr, i = by + r, j = bx + q4;
        int32_t w[4] = {MF_INFEASIBLE, MF_INFEASIBLE, MF_INFEASIBLE, MF_INFEASIBLE};
        const int to = i < n ? (len_rows ? min(len_rows[i], m) : m) : 0;
        if (j < to) {
            const int32_t *src = W + (size_t)i * ldw + j;
            if (j + 3 < to) { const int4 v = *(const int4 *)src; w[0] = v.x; w[1] = v.y; w[2] = v.z; w[3] = v.w; }
            else {
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (j + e < to) w[e] = src[e];
            }
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) { tile[r][q4 + e] = w[e]; mx = max(mx, w[e]); }
    }
    __syncthreads();
#pragma unroll
    for (int p = 0; p < 4; ++p) {
        const int r = p * 16 + rr, j = bx + r, i = by + q4;
        if (j < m && i < n) {
            int32_t *dst = WT + (size_t)j * ldt + i;
            if (i + 3 < n) *(int4 *)dst = make_int4(tile[q4][r], tile[q4 + 1][r], tile[q4 + 2][r], tile[q4 + 3][r]);
            else {
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (i + e < n) dst[e] = tile[q4 + e][r];
            }
        }
    }
    for (int off = 32; off >= 1; off >>= 1) mx = max(mx, __shfl_xor(mx, off));
    // the maximum only grows, so an outdated (smaller) cached value at worst costs a redundant atomic
    if ((threadIdx.x & 63) == 0 && mx > stats->max_weight) atomicMax(&stats->max_weight, mx);
}

__global__ void set_count_kernel(mf_device_stats *stats, int count)
{
    stats->cnt[0] = count; stats->cnt[1] = 0; stats->cnt[2] = 0; stats->cnt[3] = 0;
}
__global__ void fill_counter_kernel(unsigned long long *counter) { *counter = 0ull; }

// The largest weight alone (it sets the first epsilon), for solves that may never need W^T.
__global__ __launch_bounds__(256) void max_weight_kernel(const int32_t *__restrict__ W, int n, int m, int64_t ldw,
                                                         mf_device_stats *stats)
{
    int mx = 0;
    for (int i = blockIdx.y; i < n; i += gridDim.y) {
        const int32_t *row = W + (size_t)i * ldw;
        for (int j = (blockIdx.x * 256 + threadIdx.x) * 4; j < m; j += gridDim.x * 1024) {
            const int4 v = *(const int4 *)(row + j);            // the pitch is a multiple of four
            mx = max(mx, v.x);
            if (j + 1 < m) mx = max(mx, v.y);
            if (j + 2 < m) mx = max(mx, v.z);
            if (j + 3 < m) mx = max(mx, v.w);
        }
    }
    for (int off = 32; off >= 1; off >>= 1) mx = max(mx, __shfl_xor(mx, off));
    if ((threadIdx.x & 63) == 0 && mx > stats->max_weight) atomicMax(&stats->max_weight, mx);
}

__global__ void zero_listed_kernel(double *price, const int32_t *__restrict__ which, int count, int m)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < count && which[i] >= 0 && which[i] < m) price[which[i]] = 0.0;
}

// known, known_pairs (or null): largest weight and feasible pairs of the matrix, noted while it was scored.  scored: this
// launch is the first after the scoring pass.
__global__ void init_solver_kernel(int n, int m, double *price, double *profit, mf_device_stats *stats,
                                   int keep_prices, const int *known, const unsigned long long *known_pairs,
                                   unsigned long long *times, int scored)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i == 0) {
        times[AT_SOLVE] = device_time();
        if (scored) times[AT_SCORED] = times[AT_SOLVE];
        times[AT_PREPARED] = 0ull;
    }
    if (i < n + 4) profit[i] = 0.0;
    if (i < m + 4 && (!keep_prices || i >= m)) price[i] = 0.0;
    if (i == 0) {
        stats->rounds = 0; stats->bids = 0; stats->bytes = 0; stats->round_bytes = 0; stats->head = 0;
        stats->chain_bids = 0; stats->chain_depth = 0; stats->launch_max = 0; stats->chain_retries = 0; stats->team_bids = 0; stats->path_steps = 0; stats->path_scans = 0; stats->team_abort = 0; stats->rested = 0; stats->active = 0; stats->max_weight = known ? *known : 0;
        stats->feasible_pairs = known_pairs ? *known_pairs : ~0ull;
        stats->cnt[0] = 0; stats->cnt[1] = 0; stats->cnt[2] = 0; stats->cnt[3] = 0;
    }
}

template <int NT, int RB>
void launch_round_shape(mf_ctx *ctx, const SideArgs &s, int count, int ring, bool full)
{
    int grid = (count + RB - 1) / RB;
    if (grid > MAX_GRID) grid = MAX_GRID;
    // ten workgroups per compute unit read a matrix faster than one per group of lines: those that
    // finish early take another group
    const int cap = ctx->bulk_grid > 0 ? ctx->bulk_grid : 10 * (ctx->n_cus > 0 ? ctx->n_cus : 256);
    if (grid > cap) grid = cap;
    hipLaunchKernelGGL((round_kernel<NT, RB>), dim3(grid), dim3(NT), 0, ctx->stream, s, ctx->list[ring & 1],
                       ctx->list[(ring + 1) & 1], ctx->stats, ring, ctx->path_label, full ? 1 : 0);
}

// full: nobody is missing from the list
void launch_round(mf_ctx *ctx, const SideArgs &s, int count, int ring, bool full)
{
    if (s.edge_start && count >= 2048) { mf_launch_list_round(ctx, s, count, ring, ctx->path_label, full); return; }
    // Lines in groups per wavefront read the matrix fastest, and that is what counts when (nearly)
    // every line bids: the first round of a phase.  In the rounds after it, one line per workgroup
    // does better although it reads more slowly: bids land sooner, later bidders of the same round
    // see them, and fewer bids are wasted (measured on cluster-scale rounds: a fifth fewer bids).  Two lines
    // a group, not four, for the same reason, since rounds hand bidders over without atomics, which the more workgroups the
    // longer queued up: six seeds of 20,000 x 20,000 rounds 40.5 / 39.9 ms, of the rounds after them 17.9 / 17.3, one pair in two of
    // 15,000 x 15,000 15.1 / 11.2, 4096 x 8192 6.69 / 6.59 (one line and 256 threads there, too: 39.4, 17.4, 13.3, 6.53).
    // Feasible prefixes differ in length from nothing to the whole line, and one wavefront on the four longest
    // is what a grouped round then waits for (20,000 x 40,000, a tenth feasible: 207 us, 130 to 174 one by one).
    const bool grouped = !s.line_len && count >= 2048 && (long long)count * 100 >= (long long)ctx->bulk_share * (long long)s.len_t;
    switch (grouped ? ctx->bulk_shape : 0) {
    case 1: launch_round_shape<64, 4>(ctx, s, count, ring, full); break;
    case 2: launch_round_shape<64, 2>(ctx, s, count, ring, full); break;
    case 3: launch_round_shape<128, 4>(ctx, s, count, ring, full); break;
    case 4: launch_round_shape<256, 4>(ctx, s, count, ring, full); break;
    default: launch_round_shape<256, 1>(ctx, s, count, ring, full); break;
    }
}

// Runs one side until at most `stop_at` bidders are left (0: until nobody is left to bid).
// list[0] / cnt[0] hold the first bidders (`count` of them).  Returns MF_OK or an error;
// *left_over is the number of bidders still unplaced.  search_now: at most so many bidders (0: none)
// are searched for at once, without following their chains first, with a label window of search_width.
int run_side(mf_ctx *ctx, const SideArgs &s, int count, bool time_first, int stop_at, long long tail_budget, int *left_over,
             int search_now = 0, int search_width = 0)
{
    int ring = 0;
    // Short chains are cheapest followed step by step; a chain that is still going after
    // `path_after` steps is ended by shortest-path searches instead.
    long long team_steps = 0;
    long long stuck_steps = 0;              // chain steps, and rounds, since there were an eighth more bidders
    long long until_stuck = 0;              // ... of which so many may come
    int fewest = count;
    int idle_launches = 0;
    long long tail_steps = 0;               // dependent steps of the chain kernels of this run, longest workgroup of each
    *left_over = count;
    // Bulk rounds do not wait for their own outcome: the next round is launched for at most as many
    // bidders as the last count the host has seen (a round never leaves more bidders than it
    // found: each bid displaces at most one holder), the kernel reads the true count on the
    // device, and the host reads the count of a round while the one after it runs.  `unread` says
    // that such a round is in flight; every other kind of launch waits for the exact count first.
    bool unread = false;
    int unread_ring = 0, unread_slot = 0, slot = 0;
    unsigned unread_report = 0;
    bool counted_teams = false, chained = false, unstuck = false;
    unsigned long long bids_before = ctx->h_stats->bids;
    // takes in the statistics copied after the launch that left the lists at position `at`
    auto absorb = [&](int at) -> int {
        if ((long long)ctx->h_stats->bids == (long long)bids_before && ctx->h_stats->cnt[at & 3] >= count) {
            // a launch that neither evaluated a bid nor placed anybody must not repeat for ever
            if (++idle_launches > 64) return MF_ERR_NOT_CONVERGED;
        } else idle_launches = 0;
        bids_before = ctx->h_stats->bids;
        count = ctx->h_stats->cnt[at & 3];
        if (counted_teams) team_steps += (long long)ctx->h_stats->launch_max;     // the longest any leader went
        if (chained) {
            // (a launch that ended because its chains are stuck leaves hundreds of bidders: a search first, and chains again)
            if ((long long)ctx->h_stats->launch_max < until_stuck) tail_steps += (long long)ctx->h_stats->launch_max;
            stuck_steps += (long long)ctx->h_stats->launch_max;
        }
        if (count < fewest - fewest / 8) { fewest = count; stuck_steps = 0; }
        // (a step of a search takes as long as four of a chain: no more time goes into such searches than into chains)
        if (unstuck) stuck_steps = -4 * (long long)ctx->h_stats->launch_max;
        // a bounded wait ran out: one workgroup per chain, or no more searches, for the rest of this solve
        if (ctx->h_stats->team_abort == 1) { ctx->team_off = true; ctx->fallbacks |= MF_FALLBACK_TEAMS; }
        if (ctx->h_stats->team_abort == 2) { ctx->path_off = true; ctx->fallbacks |= MF_FALLBACK_SEARCHES; }
        *left_over = count;
        return MF_OK;
    };
    auto read_unread = [&]() -> int {
        const int rc = mf_await(ctx, unread_report);
        if (rc != MF_OK) return rc;
        *ctx->h_stats = *ctx->h_stats_slot[unread_slot];
        unread = false;
        return absorb(unread_ring);
    };
    while (!side_ends(count, stop_at, tail_budget, tail_steps)) {
        const bool paths_ok = ctx->path_max > 0 && !ctx->path_off && ctx->n_cus > 0;
        until_stuck = paths_ok ? stuck_after(ctx->path_after) - stuck_steps : ctx->max_rounds;
        const bool stuck = until_stuck <= 0, bulk = count > ctx->tail_max && !stuck;
        if (unread && !bulk) {
            // chains, teams and searches are laid out for the exact number of bidders
            const int rc = read_unread();
            if (rc != MF_OK) return rc;
            continue;
        }
        bool timed = false;
        counted_teams = false; chained = false; unstuck = false;
        const unsigned long long bytes_before = ctx->h_stats->bytes + ctx->h_stats->round_bytes;
        const bool teams_ok = ctx->team_max > 0 && !ctx->team_off;
        const int cus = ctx->n_cus > 0 ? ctx->n_cus : 256;
        // chains at or below which teams take over from one workgroup per chain
        // (lines short enough for one compute unit to read in a couple of microseconds gain nothing
        // from being split: there the teams wait for the last few chains)
        int team_from = (ctx->team_wide > ctx->team_max && s.typical_len >= TEAM_WIDE_MIN_LINE) ? ctx->team_wide : ctx->team_max;
        if (team_from > TEAM_MAX) team_from = TEAM_MAX;
        if (team_from * 2 > cus) team_from = cus / 2;
        const long long left = ctx->max_rounds - (long long)ctx->h_stats->bids;
        if (left <= 0) return MF_ERR_NOT_CONVERGED;
        if (bulk) {
            const int batch = (count > 4096 || time_first) ? 1 : 3;     // the timed round stands alone
            stuck_steps += batch;
            for (int r = 0; r < batch; ++r) {
                timed = time_first;
                launch_round(ctx, s, count, ring, r == 0);
                ++ring;
            }
            hipLaunchKernelGGL(compact_kernel, dim3((count + COMPACT_THREADS - 1) / COMPACT_THREADS), dim3(COMPACT_THREADS), 0, ctx->stream,
                               ctx->list[ring & 1], ctx->list[(ring + 1) & 1], ctx->stats, ring, ctx->path_label);
            ++ring;
        } else if (paths_ok && (count <= search_now || stuck || (count <= ctx->path_max && (team_steps >= ctx->path_after || !teams_ok)))) {
            // few enough bidders, or chains long enough, to place each bidder by a shortest-path
            // search over the whole device
            int width = search_width > ctx->path_width ? search_width : ctx->path_width;
            if (stuck && width < ctx->core_width) width = ctx->core_width;
            const int rc = mf_launch_path_search(ctx, s, ring, width);
            if (rc != MF_OK) return rc;
            unstuck = stuck;
            ++ring;
        } else if (!teams_ok || count > team_from) {
            const int grid = count < ctx->chain_grid ? count : ctx->chain_grid;
            // Workgroups hand their bidders back once so few chains are left that teams (or searches)
            // do better.  Never at a count the grid starts below: then every workgroup would hand
            // back before its first bid and the same launch would repeat for ever.
            int hand_back = teams_ok ? team_from : (paths_ok ? ctx->path_max : -1);
            if (hand_back >= grid) hand_back = grid - 1;
            chained = true;
            hipLaunchKernelGGL(chain_begin_kernel, dim3(1), dim3(1), 0, ctx->stream, ctx->stats, ring, grid);
            // (the budget of a side that only prepares prices is checked between launches, not inside
            // this one: where rows that will end up unmatched fight over every column they fit
            // beside, cutting this launch short leaves hundreds of them to the finer phases, which
            // then take seconds - measured)
            hipLaunchKernelGGL(chain_kernel, dim3(grid), dim3(CHAIN_THREADS), 0, ctx->stream, s,
                               ctx->list[ring & 1], ctx->list[(ring + 1) & 1], ctx->stats, ring,
                               left / grid + 1 < until_stuck ? left / grid + 1 : until_stuck, hand_back);
            ++ring;
        } else {
            // every remaining chain gets a team: the fewer chains, the more workgroups on each
            const int teams = count;
            int size = cus / teams;
            size = size < 2 ? 2 : (size > ctx->team_size ? ctx->team_size : size);
            const bool before_paths = paths_ok && count <= ctx->path_max;
            long long team_cap = left / teams + 1;
            // many chains: stop after a while to regroup the ones still going into larger teams;
            // few: until the searches' turn
            const long long stop_after = before_paths ? ctx->path_after - team_steps
                                                      : (count > ctx->team_max ? ctx->team_regroup : team_cap);
            if (stop_after < team_cap) team_cap = stop_after;
            if (until_stuck < team_cap) team_cap = until_stuck;
            counted_teams = before_paths;
            chained = true;
            hipLaunchKernelGGL(team_begin_kernel, dim3(1), dim3(64), 0, ctx->stream, ctx->stats,
                               (TeamCtl *)ctx->team_ctl, ring);
            const dim3 grid(teams * size);
            using TeamKernel = void (*)(SideArgs, const int *, int *, mf_device_stats *, TeamCtl *, int, long long, int);
            const int threads = ctx->team_threads;
            const TeamKernel kernel = threads == 64 ? team_kernel<64> : threads == 128 ? team_kernel<128>
                                    : threads == 256 ? team_kernel<256> : threads == 512 ? team_kernel<512>
                                                                                         : team_kernel<1024>;
            hipLaunchKernelGGL(kernel, grid, dim3(threads == 64 || threads == 128 || threads == 256 || threads == 512 ? threads : 1024),
                               0, ctx->stream, s, ctx->list[ring & 1], ctx->list[(ring + 1) & 1], ctx->stats,
                               (TeamCtl *)ctx->team_ctl, ring, team_cap, size);
            ++ring;
        }
        MF_HIP(hipGetLastError());
        if (bulk && !timed && ctx->round_lag && count > 4096) {     // (smaller rounds go three to a read, above)
            unsigned report = 0;
            int rc = mf_send(ctx, mf_report_stats(ctx, ctx->h_stats_slot[slot]), &report);
            if (rc == MF_OK && unread) rc = read_unread();      // the round before this one, while this one runs
            if (rc != MF_OK) return rc;
            unread = true;
            unread_report = report;
            unread_ring = ring;
            unread_slot = slot;
            slot ^= 1;
            continue;
        }
        int rc = mf_send_and_await(ctx, mf_report_stats(ctx, ctx->h_stats));
        if (rc != MF_OK) return rc;
        unread = false;                                  // (a later report on the same stream: it covers the round in flight too)
        if (timed) {
            ctx->timings[T_BID_BULK] += mf_ms(ctx, ctx->h_stats->round_at, ctx->h_stats->round_end);
            ctx->timings[T_BID_BULK_LAUNCHES] += 1.0f;
            ctx->timings[T_BID_BULK_BYTES] += (float)((double)(ctx->h_stats->bytes + ctx->h_stats->round_bytes - bytes_before));
        }
        time_first = false;
        rc = absorb(ring);
        if (rc != MF_OK) return rc;
    }
    if (unread) {
        const int rc = read_unread();
        if (rc != MF_OK) return rc;
    }
    return MF_OK;
}

// Lists made for one side of one phase before it is finished on whole lines.  Where launches run on all dies most are made of
// the waiting lines alone, and a side of a round needs 10 to 20: with 4, 8, 12, 16, 24, 64 of them auctions of
// thirteen 20,000 x 20,000 rounds take 20.2, 19.8, 19.3, 17.9, 17.3, 17.5 ms.  Where one die does it all they are made of
// every line, and a side that wants a fifth wants dozens: 6000 rows that rank 6000 columns nearly alike take 42, 44, 51,
// 64, 139 ms with 2, 4, 8, 16, 64 (1500 of them 19, 22, 26, 39, 20), rounds and masked matrices of 100 to 6000 rows, which
// make fewer, the same with any.
constexpr int CORE_MOST_LISTS = 4, CORE_MOST_LISTS_WIDE = 24;

// The rest of a solve, from phase `ph`, on lists of every line's best entries (core.hip): one launch
// unless lists have to be made (again) or a side has to be finished on whole lines.  *after: n_phases
// when the solve is done, else the phase to go on from without this.
template <typename StopOf, typename MakeTranspose>
int run_core(mf_ctx *ctx, SideArgs &fwd, SideArgs &rev, int rn, int rm, const long long *ladder, int n_phases, int ph,
             const StopOf &stop_of, bool &have_transpose, const MakeTranspose &make_transpose, mf_core_state &st, int &after)
{
    mf_core_plan plan{};
    plan.n_phases = n_phases;
    for (int k = 0; k < n_phases; ++k) { plan.eps[k] = ladder[k]; plan.stop[k] = stop_of(k, 1); plan.stop_grown[k] = stop_of(k, ctx->phase_growth); }
    plan.refine_below = (double)ctx->core_refine * fwd.Kd;
    st.phase = ph; st.stage = MF_CORE_RESET; st.count = 0; st.parity = 0;
    plan.may_refine = true;
    // (launches over all dies pay from about 8000 rows on: figures at the top of core.hip)
    plan.use_wide = ctx->core_wide > 0 && rn >= ctx->core_wide;
    st.wide = plan.use_wide ? 1 : 0;
    plan.stale = 8.0;
    int rc = mf_core_lists(ctx, fwd, rn, 0, nullptr, nullptr);
    if (rc != MF_OK) return rc;
    st.lists_made += 1;
    if (rm > rn) {                      // unused columns are certain: they will have to bid
        if (!have_transpose) make_transpose();
    }
    int lists_made = 0, at_phase = -1, at_stage = -1;
    bool some_newer = false;
    for (;;) {
        plan.bid_limit = (double)ctx->max_rounds - (double)ctx->h_stats->bids - (double)st.bids;
        plan.rested_before = (unsigned long long)ctx->h_stats->rested + (unsigned long long)st.rested;
        rc = mf_core_launch(ctx, fwd, rev, rn, rm, plan, &st);
        if (rc != MF_OK) return rc;
        if (st.reason == MF_CORE_DONE) { after = n_phases; return MF_OK; }
        if (st.reason == MF_CORE_ABORT) {
            ctx->path_off = true;
            ctx->fallbacks |= MF_FALLBACK_SEARCHES;
            after = st.phase;
            return MF_OK;
        }
        const bool forward = st.stage != MF_CORE_REVERSE;
        if (st.reason == MF_CORE_HANDOVER) {
            if (st.wide && some_newer && (st.stage == MF_CORE_FORWARD || st.stage == MF_CORE_REVERSE)) {
                rc = forward ? mf_core_lists(ctx, fwd, rn, 0, nullptr, nullptr) : mf_core_lists(ctx, rev, rm, 1, nullptr, nullptr);
                if (rc != MF_OK) return rc;
                st.lists_made += 1;
                st.columns_ready &= ~(forward ? 1u : 2u);
            }
            some_newer = false;
            st.wide = !st.wide;
            continue;
        }
        if (st.phase != at_phase || st.stage != at_stage) { at_phase = st.phase; at_stage = st.stage; lists_made = 0; }
        if (st.reason == MF_CORE_COLUMNS || (st.reason == MF_CORE_RELIST && ++lists_made <= (plan.use_wide ? CORE_MOST_LISTS_WIDE : CORE_MOST_LISTS))) {
            if (!forward && !have_transpose) make_transpose();
            const int lines = forward ? rn : rm;
            if (st.reason == MF_CORE_RELIST && st.stage != MF_CORE_PHASE_DONE && st.wide && st.count < lines / 2) {
                // thousands of bidders wait for better lists: theirs alone (the others' still hold, and the lot is
                // made before one die takes over: a few hundred bidders would set off one row with an old list
                // after the other, and wait 0.1 ms each time)
                rc = forward ? mf_core_lists_of(ctx, fwd, ctx->list[st.parity], st.count, 0)
                             : mf_core_lists_of(ctx, rev, ctx->list[st.parity], st.count, 1);
                if (rc != MF_OK) return rc;
                st.lists_made += 1;
                some_newer = true;
                st.columns_ready &= ~(forward ? 1u : 2u);
                continue;
            }
            rc = forward ? mf_core_lists(ctx, fwd, rn, 0, nullptr, nullptr)
                         : mf_core_lists(ctx, rev, rm, 1, ctx->price, ctx->col2row);
            if (rc != MF_OK) return rc;
            st.lists_made += 1;
            st.columns_ready &= ~(forward ? 1u : 2u);
            if (!forward) plan.have_columns = true;
            continue;
        }
        if (st.stage == MF_CORE_PHASE_DONE) { plan.may_refine = false; continue; }       // (a refinement that lists do not help)
        // This side is finished on whole lines; where a search gave up, by one of the whole device's.  (At
        // an epsilon this fine the chains of a few dozen bidders would go on for seconds.)  Paths that made a
        // search give up are thousands of epsilons long, and the whole device's takes a step of 8 us for every
        // window of labels: it goes on with the window of searches on lists, not with path_width.  (The worst of a
        // hundred 20,000 x 20,000 rounds, auction: 160 ms with 1,024 epsilons, 118 with 8,192, 130 without
        // lists.  Wider windows help that round, 103 ms with 32,768, and scan more in others, 63 -> 70 ms.)
        if (st.parity == 1) { int *t = ctx->list[0]; ctx->list[0] = ctx->list[1]; ctx->list[1] = t; st.parity = 0; }
        hipLaunchKernelGGL(set_count_kernel, dim3(1), dim3(1), 0, ctx->stream, ctx->stats, st.count);
        if (!have_transpose) make_transpose();
        SideArgs side = forward ? fwd : rev;
        side.eps = (double)ladder[st.phase];
        int left_over = 0;
        rc = run_side(ctx, side, st.count, false, plan.stop[st.phase], 0, &left_over, st.reason == MF_CORE_DENSE ? 64 : 0,
                      st.reason == MF_CORE_DENSE ? ctx->core_width : 0);
        if (rc != MF_OK) return rc;
        st.sides_left += 1;
        if (ctx->path_off) { after = st.phase; return MF_OK; }      // (what a search left half-done may hold nobody to his epsilon: the phase once more)
        st.stage = forward ? MF_CORE_FORWARD_DONE : MF_CORE_REVERSE_DONE;
        st.count = left_over;
    }
}

// A problem that one compute unit holds (small.hip), from the caller's matrix.  *general: its weights are too large for that.
int run_small(mf_ctx *ctx, const int32_t *d_W, int n, int m, int64_t ldw, int32_t *d_row2col, int64_t *d_u, int64_t *d_v, mf_result *h_res,
              bool *general)
{
    int rc = mf_launch_small(ctx, d_W, n, m, ldw, d_row2col, d_u, d_v);
    if (rc != MF_OK) return rc;
    rc = mf_run_certificate(ctx, d_W, n, m, ldw, d_row2col, d_u, d_v, (int64_t)n + 1, h_res, true);
    if (rc != MF_OK) return rc;
    const mf_cert_out &c = *ctx->h_cert;
    *general = c.status == MF_SMALL_GENERAL;
    if (c.status != MF_OK) return c.status;
    ctx->timings[T_SOLVE] = mf_ms(ctx, ctx->h_times[AT_SOLVE], ctx->h_times[AT_CERT]);
    h_res->bids = h_res->chain_bids = c.bids;
    h_res->path_steps = h_res->path_scans = c.scans;
    h_res->chain_depth = (int64_t)c.bids + c.scans;
    h_res->bytes_scanned = 4ll * n * m;               // read once, into LDS
    h_res->phases = 1;
    h_res->ms_solve = ctx->timings[T_SOLVE];
    h_res->ms_certify = ctx->timings[T_CERT];
    return h_res->cert_ok ? MF_OK : MF_ERR_CERT;
}

}  // namespace

// `warm`: start from the prices the previous solve of the same shape left in
// the context (those of the columns listed in d_reset_cols set to 0) and from a
// small epsilon.  Any non-negative starting prices are valid - every phase
// drops the assignment and re-establishes its invariants - so this changes
// only how much work the phases have to do.
int mf_run_solver(mf_ctx *ctx, const int32_t *d_W, int n, int m, int64_t ldw,
                  int32_t *d_row2col, int64_t *d_u, int64_t *d_v, mf_result *h_res,
                  bool warm, const int32_t *d_reset_cols, int n_reset_cols, bool may_use_staged)
{
    // When the matrix was just scored here, the context still holds it with rows and columns in
    // order of memory fraction, where the pairs that can share are a prefix of every row and of
    // every column: the auction then runs on that copy and reads only the prefixes; the
    // certificate below is still evaluated on the caller's matrix, in the caller's coordinates.
    ctx->team_off = ctx->path_off = false;      // every solve starts with all of its kernels
    ctx->fallbacks = 0;
    const bool candidate = may_use_staged && ctx->fit_prefix && ctx->staged_n == n && ctx->staged_m == m;
    const bool flip = n > m;
    warm = warm && !flip && !candidate && ctx->warm_n == n && ctx->warm_m == m;
    ctx->warm_n = ctx->warm_m = 0;
    bool scored = true;                         // nothing has come between the scoring pass and the launches below
    if (mf_small_fits(ctx, n, m)) {
        bool general = false;
        const int rc = run_small(ctx, d_W, n, m, ldw, d_row2col, d_u, d_v, h_res, &general);
        if (!general) return rc;
        scored = false;
        *h_res = mf_result{};
    }
    const int64_t ldt = ((int64_t)n + 3) & ~3ll;
    const int rn = flip ? m : n, rm = flip ? n : m;
    const long long K = (long long)rn + 1;
    const double Kd = (double)K;
    const int nm = rm;

    // A matrix the caller brings (no memory-ordered copy, no prefixes) may still be mostly
    // infeasible pairs, in any pattern: its rows are then also kept as lists of feasible pairs.
    const bool lists_possible = !candidate && !flip && !warm && ctx->edge_lists_from > 0 && n >= ctx->edge_lists_from &&
                                ctx->fit_prefix_below > 0;
    {
        // the largest weight sets the first epsilon
        const bool known = candidate && ctx->largest_weight_known;
        const int chunks = (m + 4095) / 4096 < 4 ? (m + 4095) / 4096 : 4;
        hipLaunchKernelGGL(init_solver_kernel, dim3((nm + 4 + 255) / 256), dim3(256), 0, ctx->stream, rn, rm,
                           ctx->price, ctx->profit, ctx->stats, warm ? 1 : 0,
                           known ? ctx->largest_weight : nullptr, candidate ? ctx->feasible_pairs : nullptr, ctx->times, scored ? 1 : 0);
        if (lists_possible) {
            // the same pass also counts the feasible pairs of every row: with few of them the rounds read lists
            hipLaunchKernelGGL(fill_counter_kernel, dim3(1), dim3(1), 0, ctx->stream, ctx->feasible_pairs);
            const int rc = mf_count_edges(ctx, d_W, n, m, ldw);
            if (rc != MF_OK) return rc;
        } else if (!known)
            hipLaunchKernelGGL(max_weight_kernel, dim3(chunks, n < 1024 ? n : 1024), dim3(256), 0, ctx->stream, d_W, n,
                               m, ldw, ctx->stats);
        MF_HIP(hipGetLastError());
    }
    {
        mf_report r = mf_report_stats(ctx, ctx->h_stats);
        r.piece[1] = {ctx->feasible_pairs, ctx->h_feasible_pairs, 2};
        const int rc = mf_send_and_await(ctx, r);
        if (rc != MF_OK) return rc;
    }
    if (!lists_possible) *ctx->h_feasible_pairs = ctx->h_stats->feasible_pairs;
    const long long cmax = K * (long long)ctx->h_stats->max_weight;
    if (cmax >= MF_MAX_DUAL) return MF_ERR_RANGE;
    // ... worth it when most of the matrix can be left unread
    const bool staged = candidate && (double)*ctx->h_feasible_pairs * 100.0 < (double)ctx->fit_prefix_below * (double)n * (double)m;
    const int32_t *M = staged ? ctx->staged : d_W;
    const int64_t ldm = staged ? (((int64_t)m + 3) & ~3ll) : ldw;
    const int *len_rows = staged ? ctx->fit_len_on : nullptr, *len_cols = staged ? ctx->fit_len_off : nullptr;
    const int32_t *A = flip ? ctx->wt : M;
    const int64_t lda = flip ? ldt : ldm;
    const int32_t *At = flip ? M : ctx->wt;
    const int64_t ldat = flip ? ldm : ldt;
    if (warm && n_reset_cols > 0)
        hipLaunchKernelGGL(zero_listed_kernel, dim3((n_reset_cols + 255) / 256), dim3(256), 0, ctx->stream,
                           ctx->price, d_reset_cols, n_reset_cols, m);
    // W^T serves the second side of a phase (unassigned columns that still carry a price), which a
    // square, fully matched problem may never enter: it is made when first needed, unless the
    // transposed problem is the one being solved
    bool have_transpose = false;
    auto make_transpose = [&]() {
        hipLaunchKernelGGL(transpose_kernel, dim3((m + 63) / 64, (n + 63) / 64), dim3(256), 0, ctx->stream,
                           M, n, m, ldm, ctx->wt, ldt, len_rows, len_cols, ctx->stats);
        have_transpose = true;
    };
    if (flip) make_transpose();
    MF_HIP(hipGetLastError());

    // with per-line lengths a scan reads, on average, the pairs that can share divided by the lines
    const double feasible = staged ? (double)*ctx->h_feasible_pairs : (double)n * (double)m;
    SideArgs fwd{A, (long long)lda, rm, ctx->price, ctx->colword, 0.0, Kd, flip ? len_cols : len_rows,
                 (int)(feasible / (double)rn), nullptr, (long long)ldat, rn, flip ? len_rows : len_cols,
                 nullptr, nullptr, nullptr, &ctx->stats->rested};
    SideArgs rev{At, (long long)ldat, rn, ctx->profit, ctx->roword, 0.0, Kd, flip ? len_rows : len_cols,
                 (int)(feasible / (double)rm), A, (long long)lda, rm, flip ? len_cols : len_rows,
                 nullptr, nullptr, nullptr, nullptr};
    if (flip) fwd.T = At;                       // (the other copy of the matrix: made on demand unless it is the one solved on)
    if (lists_possible && (double)*ctx->h_feasible_pairs * 100.0 < (double)ctx->fit_prefix_below * (double)n * (double)m &&
        *ctx->h_feasible_pairs + 4ull * (unsigned long long)n <= (unsigned long long)mf_edge_capacity(ctx)) {
        const int rc = mf_build_edge_lists(ctx, d_W, n, m, ldw, &fwd);
        if (rc != MF_OK) return rc;
    }

    // The ladder of epsilons: divided by theta per phase down to 1.  Once epsilon is at most
    // final_jump weight units (final_jump * K in dual units) the next phase is the last one:
    // prices that good leave the phase at epsilon = 1 about one bid per row, and the phases in
    // between would each cost a full re-bid and a tail of their own.
    long long ladder[64];
    int n_phases = 0;
    {
        long long e = cmax / ctx->theta;
        if (warm && ctx->warm_eps_units * K < e) e = ctx->warm_eps_units * K;
        if (e < 1) e = 1;
        for (;;) {
            ladder[n_phases++] = e;
            if (e == 1 || n_phases == 64) break;
            long long next = e / ctx->theta;
            if (next < 1 || (ctx->final_jump > 0 && e <= ctx->final_jump * K) || n_phases == 63) next = 1;
            e = next;
        }
    }
    // A phase at a coarse epsilon only prepares prices for the later ones (each drops the
    // assignment anyway), so either of its sides may end while a few bidders are still
    // unplaced: their long chains of dependent bids, and the searches that would end them, are
    // then never run at that epsilon.  The last phase_keep phases run to the end: the first of
    // them settles what was left open, the last one is what makes the result exact.  The
    // second side runs whenever more columns than that are unused and still priced - skipping
    // it would carry their prices into ever finer phases, where taking them off costs far more.
    const int keep = phases_to_the_end(ctx->phase_keep, warm, n_phases);
    auto stop_of = [&](int ph, int growth) -> int {
        return bidders_left_over(n_phases - 1 - ph, keep, ctx->phase_stop, growth, ctx->path_off ? 0 : ctx->path_max, rn);
    };
    int phases = 0;
    mf_core_state core{};
    bool core_ok = ctx->core && ctx->n_cus > 0 && !ctx->path_off;
    for (int ph = 0; ph < n_phases; ++ph) {
        // From the phase on in which a list of each row's best columns reaches far enough below the
        // best (core_depth epsilons), the rest of the solve runs on such lists.  On problems whose first bids
        // run on all dies bidders whose lists have sunk wait there for better ones, a thousand and more at
        // once, and lists pay from a twentieth of that depth on: 20,000 x 20,000 next rounds 21.4 / 19.7 ms, one pair
        // in two of 15,000 x 15,000 19.4 / 13.8, others of 10,000 and more 0 to 4 % less.  Not with feasible
        // prefixes, whose lines cost little (20,000 x 40,000 20.3 / 22.3), and not where one die does it all (6001 x
        // 9007 13.2 / 14.2).
        if (core_ok && (ph > 0 || warm || rm <= MF_CORE_LIST)) {
            if (ph == 0) mf_note_time(ctx, AT_PREPARED);
            double deep = 1.0;
            if (rm > MF_CORE_LIST) {
                const bool all_dies = ctx->core_wide > 0 && rn >= ctx->core_wide && !fwd.line_len;
                const int rc = mf_core_probe(ctx, fwd, rn, (double)ctx->core_depth_eps * (double)ladder[ph] / (all_dies ? 20.0 : 1.0), &deep);
                if (rc != MF_OK) return rc;
            }
            if (deep >= 0.75) {
                int after = n_phases;
                const int rc = run_core(ctx, fwd, rev, rn, rm, ladder, n_phases, ph, stop_of, have_transpose, make_transpose, core, after);
                if (rc != MF_OK) return rc;
                if (after >= n_phases) { phases = core.phase + 1; break; }
                core_ok = false;                        // a wait ran out in there: on from that phase without it
                ph = after;
            }
        }
        const long long eps = ladder[ph];
        const bool searching = !ctx->path_off;
        // (a wait ran out in a search: what it left half-done may hold nobody to his epsilon, so the phase begins once more, without searches)
        const auto once_more = [&]() { return searching && ctx->path_off; };
        phases = ph + 1;
        fwd.eps = rev.eps = (double)eps;
        hipLaunchKernelGGL(reset_kernel, dim3((nm + 255) / 256), dim3(256), 0, ctx->stream, rn, rm, ctx->price,
                           ctx->colword, ctx->row2col, ctx->col2row, ctx->list[0], ctx->stats, ctx->times);
        int left_over = 0;
        // ... unless bidders have been giving up (best value at most epsilon) in this solve: then
        // workloads stay unmatched at the optimum, the bidders left over would be the ones that
        // end up resting, and the finer the epsilon at which they fight it out the longer it takes
        const int stop_at = stop_of(ph, ctx->h_stats->rested < ctx->phase_growth_rest ? ctx->phase_growth : 1);
        // a phase that runs to the end places its last bidders by a search, which re-labels the
        // columns of a served tree from the other copy of the matrix
        if (!have_transpose && stop_at == 0 && ctx->path_max > 1 && rn > 1) make_transpose();
        if (have_transpose) fwd.T = At;
        int rc = run_side(ctx, fwd, rn, true, stop_at, mf_tail_steps(ctx, 0, rn), &left_over);
        if (rc != MF_OK) return rc;
        if (once_more()) { core_ok = false; --ph; continue; }
        // who holds what after the forward rounds; unassigned priced columns go to list[0]
        hipLaunchKernelGGL(forward_done_rows_kernel, dim3((rn + 255) / 256), dim3(256), 0, ctx->stream, rn,
                           ctx->profit, ctx->roword, ctx->row2col, ctx->stats);
        hipLaunchKernelGGL(forward_done_cols_kernel, dim3((rm + 255) / 256), dim3(256), 0, ctx->stream, rm,
                           A, lda, Kd, ctx->colword, ctx->price, ctx->profit, ctx->roword, ctx->row2col,
                           ctx->col2row, ctx->list[0], ctx->stats);
        if (left_over > 0)
            hipLaunchKernelGGL(settle_unplaced_kernel, dim3(rn < MAX_GRID ? rn : MAX_GRID), dim3(BID_THREADS), 0,
                               ctx->stream, A, lda, rn, rm, ctx->price, ctx->row2col, Kd, ctx->profit, ctx->roword,
                               fwd.line_len);
        MF_HIP(hipGetLastError());
        rc = mf_send_and_await(ctx, mf_report_stats(ctx, ctx->h_stats));
        if (rc != MF_OK) return rc;
        const int rev_count = ctx->h_stats->cnt[0];
        if (rev_count > stop_at) {
            if (!have_transpose) make_transpose();
            rc = run_side(ctx, rev, rev_count, false, stop_at, mf_tail_steps(ctx, 1, rn), &left_over);
            if (rc != MF_OK) return rc;
            if (once_more()) { core_ok = false; --ph; continue; }
            hipLaunchKernelGGL(reverse_done_cols_kernel, dim3((rm + 255) / 256), dim3(256), 0, ctx->stream, rm,
                               ctx->price, ctx->col2row);
            hipLaunchKernelGGL(reverse_done_rows_kernel, dim3((rn + 255) / 256), dim3(256), 0, ctx->stream, rn,
                               A, lda, Kd, ctx->roword, ctx->price, ctx->row2col, ctx->col2row);
            MF_HIP(hipGetLastError());
        }
    }
    {
        const int rc = mf_extract_duals(ctx, A, lda, rn, rm, Kd, fwd.line_len, n, flip, staged, d_row2col, d_u, d_v);
        if (rc != MF_OK) return rc;
    }
    int rc = mf_run_certificate(ctx, d_W, n, m, ldw, d_row2col, d_u, d_v, K, h_res, false);
    if (rc != MF_OK) return rc;
    const unsigned long long *at = ctx->h_times;
    const float ms_solve = mf_ms(ctx, at[AT_SOLVE], at[AT_DUALS]), ms_duals = mf_ms(ctx, at[AT_DUALS], at[AT_CERT]), ms_cert = ctx->timings[T_CERT];
    ctx->timings[T_TRANSPOSE] = mf_ms(ctx, at[AT_SOLVE], at[AT_PREPARED]);
    ctx->timings[T_SOLVE] = ms_solve;
    ctx->timings[T_DUALS] = ms_duals;
    ctx->timings[T_LIST_LAUNCHES] = (float)core.launches;
    ctx->timings[T_LISTS_MADE] = (float)core.lists_made;
    ctx->timings[T_LIST_SIDES_LEFT] = (float)core.sides_left;
    ctx->timings[T_LISTS_BY_COLUMN] = (float)core.by_column;
    h_res->rounds = (int64_t)ctx->h_stats->rounds;
    // (the device's counts of bids include the searches' scans, which count against max_rounds)
    const int64_t searched = (int64_t)ctx->h_stats->path_scans;
    h_res->bids = (int64_t)ctx->h_stats->bids - searched + core.bids;
    h_res->bytes_scanned = (int64_t)(ctx->h_stats->bytes + ctx->h_stats->round_bytes) + core.bytes;
    h_res->chain_bids = (int64_t)ctx->h_stats->chain_bids - searched + core.bids;
    h_res->chain_retries = (int64_t)ctx->h_stats->chain_retries;
    h_res->team_bids = (int64_t)ctx->h_stats->team_bids;
    h_res->path_steps = (int64_t)ctx->h_stats->path_steps + core.steps;
    h_res->path_scans = searched + core.scans;
    h_res->chain_depth = (int64_t)(ctx->h_stats->chain_depth + ctx->h_stats->launch_max) + core.depth + core.steps;
    h_res->phases = phases;
    h_res->fallbacks = ctx->fallbacks;
    h_res->ms_solve = ms_solve;
    h_res->ms_certify = ms_duals + ms_cert;
    if (h_res->cert_ok && !staged) { ctx->warm_n = n; ctx->warm_m = m; }      // these prices may seed the next solve
    return h_res->cert_ok ? MF_OK : MF_ERR_CERT;
}
