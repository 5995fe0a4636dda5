// Internal declarations shared by the library's translation units (not installed).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <tuple>
#include "muxmatch.h"
#include "pair_tasks.h"
#include "side_end.h"

#define MF_HIP(call)                                                            \
    do {                                                                        \
        hipError_t e_ = (call);                                                 \
        if (e_ != hipSuccess) {                                                 \
            ctx->hip_error = e_;                                                \
            return MF_ERR_HIP;                                                  \
        }                                                                       \
    } while (0)

// A dual value and the index of the workload holding the other end share one
// 64-bit word so that a single atomicMax both raises the dual and records
// who raised it: word = dual << MF_ID_BITS | (id + 1), id + 1 == 0 meaning "nobody".
#define MF_ID_BITS 20
#define MF_ID_MASK ((1ull << MF_ID_BITS) - 1ull)
#define MF_MAX_DIM ((1 << MF_ID_BITS) - 2)
#define MF_MAX_DUAL (1ll << 43)
#define MF_MAX_TYPES 64

enum { T_PROJ = 0, T_PAIR, T_BID_BULK, T_BID_BULK_LAUNCHES, T_TRANSPOSE, T_DUALS, T_CERT, T_SOLVE,
       T_BID_BULK_BYTES, T_PAIR_EVALUATED, T_LIST_LAUNCHES, T_LISTS_MADE, T_LIST_SIDES_LEFT, T_LISTS_BY_COLUMN, T_COUNT = 16 };

// The matching on short lists (core.hip): entries per list, most phases of a solve, lines a probe
// looks at, why a launch ended and at which stage of a phase it (or the next one) starts.
#define MF_CORE_LIST 128
#define MF_CORE_PHASES 64
#define MF_CORE_PROBES 256
enum { MF_CORE_DONE = 1,        // the matching is complete and its prices are good
       MF_CORE_ABORT,           // a wait ran out: the phase starts again without this kernel
       MF_CORE_RELIST,          // many lines had to be read whole: the lists are due again
       MF_CORE_COLUMNS,         // columns have to bid and have no lists yet
       MF_CORE_DENSE,           // a search gave up: this side is finished on whole lines
       MF_CORE_LIMIT,           // the limit on bids may be reached: likewise
       MF_CORE_HANDOVER };      // on from here on all dies, or on one
enum { MF_CORE_RESET = 0, MF_CORE_FORWARD, MF_CORE_FORWARD_DONE, MF_CORE_REVERSE, MF_CORE_REVERSE_DONE, MF_CORE_PHASE_DONE };

// When a call's stages began (mf_ctx::times, ticks of the device's constant clock): noted by the first kernel of each.
enum { AT_SCORE = 0, AT_PAIRS, AT_PLACE, AT_SCORED, AT_SOLVE, AT_PREPARED, AT_DUALS, AT_CERT, AT_COUNT };

// Up to so many stretches of device memory stored into pinned memory (report.hip).
constexpr int MF_REPORT_PIECES = 4;
struct mf_report {
    struct { const void *from; void *to; int words; } piece[MF_REPORT_PIECES];      // of four bytes
};
struct mf_told {                    // pinned
    alignas(64) unsigned number;    // of the last report that is there
    alignas(64) unsigned long long at;      // when it was made
};

struct mf_device_stats {            // lives in device memory, cleared per solve
    unsigned long long rounds;      // bidding rounds
    unsigned long long bids;        // bids evaluated (one line scan each)
    unsigned long long bytes;       // weight bytes those scans read
    unsigned long long chain_bids;  // bids evaluated by chain kernels
    unsigned long long chain_depth; // sum over chain kernels of the most bids any one workgroup evaluated
    unsigned long long chain_retries; // chain bids that lost and were redone with uncached dual reads
    unsigned long long team_bids;   // chain bids evaluated by several workgroups together
    unsigned long long path_steps;  // super-steps of the shortest-path searches
    unsigned long long path_scans;  // line scans those searches made
    unsigned long long launch_max;  // scratch: that maximum for the chain kernel in flight
    unsigned long long feasible_pairs;      // of the matrix, where the scoring pass counted them (else ~0)
    unsigned long long round_at, round_end;     // when the last bidding round began, and when it was over
    int max_weight;
    int cnt[4];                     // ring of bidder-list lengths: round r reads cnt[r & 3]
    int head;                       // next unclaimed entry of the list a chain kernel works through
    int active;                     // workgroups of the running chain kernel still following a chain
    int team_abort;                 // a bounded wait between cooperating workgroups ran out (1: chain teams, 2: path search)
    int rested;                     // bidders of the side on which rows bid that gave up with best value <= eps, this solve
    unsigned long long round_bytes; // weight bytes the rounds with many bidders read
};

// What a place of a bidding round's list has cost: 4-byte words read, from this bit on bids (see round_kernel).
#define MF_WORK_WORDS 40

struct alignas(128) mf_cert_out {   // lives in device memory, cleared per check
    long long primal;
    long long dual;
    long long min_rc;
    int matched;
    int flags;                      // bit0 bad index/duplicate, bit1 infeasible pair, bit2 negative dual
    int bids, scans, status;        // of a matching by small_kernel, which begins the check in the same launch (in the first part)
};

// A check adds up in so many parts: workgroups that finish together would queue up behind atomics on one line.
constexpr int MF_CERT_PARTS = 16;
// (one thread clears a part)
__host__ __device__ inline void mf_clear_part(mf_cert_out *o) { o->primal = 0; o->dual = 0; o->min_rc = INT64_MAX; o->matched = 0; o->flags = 0; }
__host__ __device__ inline mf_cert_out mf_sum_parts(const mf_cert_out *o)
{
    mf_cert_out s = o[0];
    for (int p = 1; p < MF_CERT_PARTS; ++p) {
        s.primal += o[p].primal; s.dual += o[p].dual; s.matched += o[p].matched; s.flags |= o[p].flags;
        s.min_rc = o[p].min_rc < s.min_rc ? o[p].min_rc : s.min_rc;
    }
    return s;
}

// What mf_set_option sets, with the defaults.
struct mf_options {
    int64_t theta = 24;                         // epsilon divisor per phase
    int64_t max_rounds = 4000000000ll;          // limit on evaluated bids per solve
    int fit_prefix_below = 50;                  // percent of pairs that can share below which the solve uses the staged matrix
    int edge_lists_from = 4096;                 // rows from which a matrix the caller brought is turned into lists when few pairs are feasible (0: never)
    bool fit_prefix = true;                     // solve on the staged matrix, reading only the prefixes that can share
    bool fit_order = true;                      // score in memory order and skip pairs that cannot fit
    bool warm_reset_cols = true;                // start replaced columns at price 0 instead of their predecessor's price
    int64_t warm_eps_units = 0;                 // first epsilon of a warm-started solve, in weight units
    int phase_stop = 16;                        // unplaced bidders at or below which a phase that only prepares prices ends
    int phase_growth = 2;                       // ... times this for every phase further from the ones that run to the end
    int phase_growth_rest = 32;                 // bidders that may have given up before coarse phases stop leaving more
    int phase_keep = 0;                         // the last so many phases always run to the end (0: nobody has said how many, see side_end.h)
    long long phase_tail_steps = 64;            // dependent chain steps after which a side that only prepares prices ends (0: no limit)
    int phase_tail_from = 8192;                 // ... for problems with at least this many bidding lines
    int phase_tail_sides = 1;                   // ... on which sides: bit 0 the first (rows bid), bit 1 the second
    long long final_jump = 0;                   // epsilon (weight units) at or below which the next phase is the last (0: never)
    int tail_max = 1024;                        // bidder count at or below which chains are followed in one kernel
    int bulk_grid = 0;                          // most workgroups of a round with many bidders (0: one per group of lines, up to 8192)
    int bulk_shape = 2;                         // workgroup shape of rounds with many bidders (see launch_round)
    int bulk_share = 95;                        // ... "many": at least 2048 and this share (percent) of the side's lines
    int team_max = 8;                           // chains at or below which several workgroups share each chain (0: never)
    int team_size = 16, team_threads = 1024;    // most workgroups per chain, threads per such workgroup
    int team_wide = 64;                         // chains at or below which smaller teams already take over from chain_kernel
    long long team_regroup = 128;               // steps after which such teams stop so that the chains left can be regrouped
    int path_max = 16;                          // bidders at or below which shortest-path searches place them (0: never)
    long long path_after = 256;                 // chain steps per run after which the searches take over
    int path_grid = 0;                          // workgroups of a search (0: one per compute unit)
    int path_width = 1024;                      // label window of one super-step, in epsilons
    bool path_pull = false;                     // re-label a served tree's columns from the other copy of the matrix
    int path_frontier_rows = 1024;              // frontier above which the window is halved (doubled below an eighth of it)
    unsigned path_spin_limit = 1u << 22;        // polls a workgroup waits at a barrier of the search before it gives up
    int chain_grid = 256;                       // workgroups of chain_kernel
    int core = 1;                               // 0: no phases on short lists (core.hip)
    int core_depth_eps = 20;                    // how many epsilons the lists have to reach below a line's best value
    int core_many = 4, core_few = 32;           // chain steps between two looks at the list, with more / fewer bidders than wavefronts
    long long core_after = 256;                 // chain steps after which the last bidders are searched for
    int core_wide = 8192, core_narrow = 1024;   // lines from which the wide parts run on all dies; bidders at or below which one die takes over
    int core_read = 25;                         // percent of the matrix one search on lists may read whole, ...
    long long core_read_least = 8ll << 20;      // ... or so many entries if they are more
    int core_refine = 200;                      // epsilon (weight units) at or below which a complete phase is followed by a refinement
    int core_width = 8192;                      // label window of a search on lists, in epsilons
    int score_split = 1;                        // 1: the scorer's hidden layer multiplies fp16 pieces of its fp32 operands
    int round_lag = 1;                          // 1: bulk rounds are launched one ahead of the host's reads

    auto how_to_match() const
    {
        return std::tuple_cat(std::make_tuple(phase_keep ? phase_keep : PHASES_TO_THE_END), std::tie(theta, fit_prefix_below, edge_lists_from, fit_prefix, warm_reset_cols, warm_eps_units, phase_stop, phase_growth,
                        phase_growth_rest, phase_tail_steps, phase_tail_from, phase_tail_sides,
                        final_jump, tail_max, bulk_grid, bulk_shape, bulk_share, team_max, team_size, team_threads,
                        team_wide, team_regroup, path_max, path_after, path_grid, path_width, path_pull,
                        path_frontier_rows, path_spin_limit, chain_grid, core, core_depth_eps, core_many, core_few,
                        core_after, core_wide, core_narrow, core_read, core_read_least, core_refine, core_width,
                        round_lag));
    }
    // Whether one that says how to match differs from its default: small problems are then matched that way, too.
    bool as_told() const
    {
        const mf_options defaults;
        return how_to_match() != defaults.how_to_match();
    }
};

struct mf_ctx : mf_options {
    int device;
    hipStream_t stream;
    int max_n, max_m;
    hipError_t hip_error;
    unsigned kernels_configured;    // kernels whose dynamic shared memory limit has been raised on this device (bits)
    // scoring scratch
    float *proj_on, *proj_off;      // [max_n][H], [max_m][H]
    float *mem_on, *mem_off;        // [max_n], [max_m]
    float *sm_on, *sm_off;          // SM activity / SM demand features (pair-dependent SM input)
    int32_t *order_on, *order_off;  // workloads by ascending memory fraction (online: by type first)
    int32_t *rank_on, *rank_off;    // position of each workload in its order
    float *mem_on_sorted, *mem_off_sorted;
    int32_t *staged;                // [max_n][pad4(max_m)] the last scored matrix with rows and columns in memory order
    int32_t *fit_len_on, *fit_len_off;   // per staged row / column: how many entries from the start can share
    unsigned long long *feasible_pairs, *h_feasible_pairs;    // how many pairs of the staged matrix can share (device, pinned)
    int *edge_count;                // [max(max_n, max_m)] feasible pairs per row of a matrix the caller brought, padded to 4
    long long *edge_start;          // [max(max_n, max_m) + 1] where each row's list starts
    int staged_n, staged_m;         // shape of the staged matrix the solver may use (0: none)
    int *largest_weight;            // largest weight of the matrix just scored (device), noted while it was put in place
    bool largest_weight_known;      // ... and whether it is that of the matrix the staged copy belongs to
    int32_t *type_segment;          // [MF_MAX_TYPES + 1] first position of each type in order_on
    unsigned long long *pairs_evaluated, *h_pairs_evaluated;   // pairs the last scoring pass ran the MLP on (device, pinned)
    double pairs_total;             // ... out of this many
    // solver scratch
    int32_t *wt;                    // transposed weights [max_m][ldt]
    double *price, *profit;         // [max_m+4], [max_n+4]: exact integers held in doubles
    unsigned long long *colword, *roword;
    int *row2col, *col2row;
    int warm_n, warm_m;             // shape of the solve whose prices the context still holds (0: none)
    bool team_off;                  // set after a team wait ran out, for the rest of the solve
    int fallbacks;                  // MF_FALLBACK_* bits of the running solve
    void *team_ctl;                 // control blocks of the cooperating workgroups
    void *path_ctl;                 // control block of the shortest-path search
    unsigned long long *path_label, *path_expanded;   // [max(max_n, max_m)] each
    unsigned int *path_stamp;
    unsigned long long *path_frontier[2];   // 16 segments of max(max_n, max_m) entries (column, holder) each
    int *path_held;
    double *path_base;              // per bidding line: length of the shortest path to it plus what it would pay, or +inf
    int *path_tree;                 // columns of the tree being served
    int *path_parent, *path_jump;   // [max(max_n, max_m)] each: predecessor columns while a tree is served
    bool path_off;                  // set after a wait of the search ran out, for the rest of the solve
    int n_cus;                      // compute units of the device
    // phases on short lists (core.hip)
    int2 *core_entries[2];          // lists of the rows (of the side with fewer lines), of the columns
    double *core_bound[2], *core_half_bound[2], *core_built[2], *core_reach[2], *core_depth, *h_core_depth;
    int *core_t_start[2], *core_t_at[2], *core_tree;    // the lists by opposite line (searches)
    int2 *core_t_entries[2];
    double *core_base, *core_dropped;
    unsigned long long *core_parent, *core_read_from;
    int32_t *core_weight;
    void *core_ctl, *h_core_report;
    bool core_clear;                // the control block is as a launch wants to find it
    int *list[2];
    int *colmark;                   // [max_m]
    mf_device_stats *stats;
    mf_cert_out *cert;
    // pinned host mirrors
    mf_device_stats *h_stats;
    mf_device_stats *h_stats_slot[2];   // pinned: where the counts of bulk rounds land while the next round runs
    int32_t *h_type_first;              // pinned: where each type's rows start
    int *h_bad;                         // pinned: an index or a type was out of range
    mf_told *h_told;
    unsigned reports;                   // sent so far
    int *score_queue;                   // device: next tasks of the pair kernel's launches, one a type, MF_PAIR_QUEUES counters each
    unsigned *score_range;              // device: largest magnitudes the scorer's fp16 pieces are scaled by (project_kernel)
    mf_cert_out *h_cert;
    // timing
    unsigned long long *times, *h_times;        // [AT_COUNT] device, pinned
    double clock_khz;               // of the clock they are in
    hipEvent_t ev[2];               // (mf_measure_ceilings)
    float timings[T_COUNT];
    bool score_pending, score_placed;       // times of a scoring pass noted but not yet read; it put the scores in place
};

// One side of the auction as its kernels see it (rows bidding for columns, or the reverse).
struct SideArgs {
    const int32_t *A;                   // the bidding side's lines (W for rows, W^T for columns)
    long long pitch;
    int len;
    double *other_dual;                 // opposite duals as doubles, raised with atomicMax on the bits
    unsigned long long *otherword;      // opposite packed (dual, holder): the authoritative copy
    double eps, Kd;
    const int *line_len;                // optional: every entry of line b at or beyond line_len[b] is infeasible
    int typical_len;                    // what a scan reads on average (host-side choice of kernels only)
    // the same matrix by lines of the other side (line k of T is entry k of every line of A), when
    // that copy exists (else null): lets a search look at one entry of all bidding lines at once
    const int32_t *T;
    long long pitch_t;
    int len_t;                          // entries of a line of T = lines of A
    const int *line_len_t;              // optional, as line_len
    // optional: every line of A once more as a list of its feasible entries (position, weight),
    // list b at [edge_start[b], edge_start[b + 1]), both multiples of four, padding (0, infeasible)
    const long long *edge_start;
    const int *edge_col;
    const int32_t *edge_weight;
    int *rested;                        // optional: counts the bidders that rest (best value at most eps)
};

inline long long mf_tail_steps(const mf_ctx *ctx, int side, int lines) { return steps_of_side(side, ctx->phase_tail_sides, ctx->phase_tail_steps, ctx->phase_tail_from, lines); }

// report.hip
int mf_send(mf_ctx *ctx, const mf_report &r, unsigned *number);         // on the stream; *number says which it is
int mf_await(mf_ctx *ctx, unsigned number);                             // until that one is there
int mf_send_and_await(mf_ctx *ctx, const mf_report &r);
void mf_note_time(mf_ctx *ctx, int stage);                              // by a launch of its own
inline mf_report mf_report_stats(const mf_ctx *ctx, mf_device_stats *to) { return mf_report{{{ctx->stats, to, (int)(sizeof(mf_device_stats) / 4)}}}; }
inline float mf_ms(const mf_ctx *ctx, unsigned long long from, unsigned long long to) { return to > from ? (float)((double)(to - from) / ctx->clock_khz) : 0.0f; }
// score.hip
int mf_launch_score(mf_ctx *ctx, const mf_predictor *preds, int n_types, const int32_t *d_type,
                    const float *d_on, int n, const float *d_off, int m, int32_t *d_W, int64_t ldw,
                    float *d_sigma, bool as_it_comes);
int mf_launch_rescore(mf_ctx *ctx, const mf_predictor *pred, const float *d_on, int n, const float *d_off,
                      int m, int32_t *d_W, int64_t ldw, const int32_t *d_rows, int n_rows,
                      const int32_t *d_cols, int n_cols);
// auction.hip
int mf_run_solver(mf_ctx *ctx, const int32_t *d_W, int n, int m, int64_t ldw,
                  int32_t *d_row2col, int64_t *d_u, int64_t *d_v, mf_result *h_res,
                  bool warm, const int32_t *d_reset_cols, int n_reset_cols, bool may_use_staged);
// edges.hip
int mf_count_edges(mf_ctx *ctx, const int32_t *d_W, int n, int m, int64_t ldw);
int mf_build_edge_lists(mf_ctx *ctx, const int32_t *d_W, int n, int m, int64_t ldw, SideArgs *side);
void mf_launch_list_round(mf_ctx *ctx, const SideArgs &s, int count, int ring, unsigned long long *work, bool full);
inline size_t mf_edge_capacity(const mf_ctx *ctx)      // entries the lists may hold: half the staged copy's words each for columns and weights
{
    return ((size_t)ctx->max_n * ((((size_t)ctx->max_m + 3) & ~(size_t)3)) / 2) & ~(size_t)3;
}
// paths.hip
int mf_launch_path_search(mf_ctx *ctx, const SideArgs &s, int ring, int width);     // width: label window, in epsilons
// core.hip
struct mf_core_plan {
    int n_phases;
    long long eps[MF_CORE_PHASES];
    int stop[MF_CORE_PHASES], stop_grown[MF_CORE_PHASES];
    double refine_below, bid_limit;
    unsigned long long rested_before;
    bool have_columns, may_refine, use_wide;
    double stale;
};
struct mf_core_state {
    int reason, phase, stage, count, parity;
    int wide, refined;
    int columns_wait;                   // the columns that bid may be left to the next phase (side_end.h)
    unsigned columns_ready;             // the sides whose lists also exist by opposite line (bits)
    long long bids, depth, steps, scans, rested, bytes;      // summed over launches
    int launches, lists_made, sides_left, by_column;     // sides_left: finished on whole lines; by_column: lists that launches kept by opposite line, too
};
int mf_core_lists(mf_ctx *ctx, const SideArgs &s, int lines, int which, const double *own_dual, const int *partner);
int mf_core_lists_of(mf_ctx *ctx, const SideArgs &s, const int *list, int count, int which);
int mf_core_probe(mf_ctx *ctx, const SideArgs &s, int lines, double distance, double *deep);
int mf_core_launch(mf_ctx *ctx, const SideArgs &fwd, const SideArgs &rev, int rn, int rm, const mf_core_plan &plan, mf_core_state *st);
size_t mf_core_ctl_bytes(), mf_core_report_bytes();
// certificate.hip
int mf_extract_duals(mf_ctx *ctx, const int32_t *A, int64_t lda, int rn, int rm, double Kd, const int *line_len,
                     int n, bool flip, bool staged, int32_t *d_row2col, int64_t *d_u, int64_t *d_v);
int mf_run_certificate(mf_ctx *ctx, const int32_t *d_W, int n, int m, int64_t ldw,
                       const int32_t *d_row2col, const int64_t *d_u, const int64_t *d_v,
                       int64_t K, mf_result *h_res, bool begun);        // begun: ctx->cert and ctx->colmark are cleared
// small.hip
enum { MF_SMALL_GENERAL = 1 };           // status: left to the auction
bool mf_small_fits(const mf_ctx *ctx, int n, int m);
int mf_launch_small(mf_ctx *ctx, const int32_t *d_W, int n, int m, int64_t ldw, int32_t *d_row2col, int64_t *d_u, int64_t *d_v);
