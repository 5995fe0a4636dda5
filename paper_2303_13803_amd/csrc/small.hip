// The matching of problems of up to about a hundred rows, whose whole matrix fits into one compute unit's LDS (the
// paper's GetMatching on a handful of GPUs: Section "Matching-based scheduling").
//
// The auction's phases are made for matrices that many workgroups read at once; on 64 x 64 they are two dozen
// launches and 1 us for every bid of a chain, which goes through the L2 four times.  Here one workgroup puts the
// matrix into LDS and one wavefront of it solves: prices, holders and labels sit in registers, a lane having C
// neighbouring columns; a bid or a scanned row of a search is one read of LDS and a reduction or two over the
// wavefront.  All of it is exact in whole weight units, so there is no epsilon and no ladder:
//   bids      a row takes its best column and raises its price by what it prefers it to its second best (or to
//             none at all); whoever held it goes on.  A row whose best column is held and not preferred waits.
//   searches  each row that waits is placed by one shortest augmenting path (Dijkstra over columns, a label per
//             column), which may end at a free column or leave the row on it with the least to lose unmatched.
// Throughout, held pairs are tight, no pair of a placed or given-up row is worth more than its duals, and a
// column that nobody holds has price 0: in the end the duals prove the matching, with no gap.
// (The order of the two parts is that of Jonker and Volgenant 1987, "A shortest augmenting path algorithm for dense and
// sparse linear assignment problems".)
#include "scan.h"
#include "report.h"

namespace {

constexpr int SMALL_THREADS = 1024;         // one of the 16 wavefronts solves, all of them fetch the matrix
constexpr int SMALL_FETCH = 8;                  // rows a wavefront has on their way at once
constexpr int SMALL_COLS = 512;                 // eight columns a lane
constexpr int SMALL_LDS = 152 * 1024;           // (of 160 KB)
// Rows: the searches scan up to half as many rows as there are, one after the other, where the auction's bidders go on side
// by side.  Rounds of scored pairs, whose rows prefer nearly the same columns, auction / this, ms (the laws of four
// configurations, four seeds): 64 x 64 0.44..0.90 / 0.23..0.41, 80 x 80 0.56..1.1 / 0.31..0.62, 88 x 88 0.54..0.86 / 0.34..0.76,
// 104 x 104 0.58..1.1 / 0.44..1.08 (the slowest law 0.76 / 0.90 in the mean), 128 x 128 0.87 / 1.25.  With more columns than
// rows there is less to search: 64 x 150 0.51..0.88 / 0.23..0.46, 112 x 200 0.66..1.2 / 0.51..1.05, but with eight columns a lane
// 112 x 300 0.59..1.1 / 0.52..1.33.  Other matrices gain at any of these sizes (uniform weights, 100 x 100 0.36 / 0.19;
// products of a row and a column, the longest searches there are, 64 x 64 1.6 / 0.6).
// More rows than columns are left to the auction: they would have to be transposed on their way into LDS, and partners and
// duals on their way out, which is not written (it should gain as much).
constexpr int SMALL_ROWS = 88, SMALL_ROWS_WIDE = 112, SMALL_COLS_WIDE = 256;     // ... the latter with a third more columns than rows
// Bids in the first part, per row.  (More leave fewer rows waiting but prefer the same columns: 64 x 64 with 1, 2, 4 and 8 a row,
// 109 + 1018, 170 + 1035, 295 + 864 and 538 + 872 bids and scans, and a bid takes half as long again as a scan.)
constexpr int SMALL_BIDS = 1;
constexpr int SMALL_WEIGHTS = 1 << 28;          // weights below it: twice every sum below then stays within 32 bits

struct SmallShape {
    int n, m, pitch;                            // rows n <= columns m; entries from a row to the next in LDS
    long long ldw;
};

// A lane holds the columns lane * C ... lane * C + C - 1.
template <int C>
__device__ __forceinline__ void set_column(int (&x)[C], int k, int value, int lane)
{
#pragma unroll
    for (int c = 0; c < C; ++c)
        if (k == lane * C + c) x[c] = value;
}

// The largest of x over the wavefront, where it is, and what y and, with THIRD, z are there.  (One ballot and two or three moves from a lane to a
// scalar, whatever C: each lane first picks among its own.)
struct Pick { int value, column, other, third; };
template <int C, bool THIRD>
__device__ __forceinline__ Pick pick(const int (&x)[C], const int (&y)[C], const int (&z)[C], int lane)
{
    int best = x[0], which = lane * C, mine = y[0], also = z[0];
#pragma unroll
    for (int c = 1; c < C; ++c) {
        const int take = x[c] > best ? -1 : 0, there = y[c];       // (selected by bits: a choice between entries of an array ends up in memory)
        best = max(best, x[c]);
        which = ((lane * C + c) & take) | (which & ~take);
        mine = (there & take) | (mine & ~take);
        if constexpr (THIRD) { const int third = z[c]; also = (third & take) | (also & ~take); }
    }
    Pick p;
    p.value = wave_max(best);
    const int src = __builtin_ctzll(__ballot(best == p.value));
    p.column = C == 1 ? src : __builtin_amdgcn_readlane(which, src);
    p.other = __builtin_amdgcn_readlane(mine, src);
    p.third = THIRD ? __builtin_amdgcn_readlane(also, src) : 0;
    return p;
}

template <int C>
__device__ __forceinline__ int largest_of(const int (&x)[C])
{
    int b = x[0];
#pragma unroll
    for (int c = 1; c < C; ++c) b = max(b, x[c]);
    return wave_max(b);
}

// What bounds it: one chain of dependent bids and scans (0.19 us a scan with one column a lane, 0.28 with four, 0.43 with
// eight: a third of it the reduction, a quarter LDS) and 6 us for the launch and the matrix's way into one compute
// unit.  64 x 64 of scored pairs: about 110 bids and 550 to 1300 scans, 140 to 280 us, where the auction's launches took 565.
// The profit of a column's holder is kept beside the holder, so that all that a scan takes off the next row's weights is there before
// they are: read from LDS with them it came another trip to a scalar and an addition later.  Rounds of 64 x 64 186..338 / 180..324 us
// (two laws, three seeds each), 88 x 88 288..697 / 277..662, 64 x 150 212..416 / 200..382, 100 x 250 350..848 / 327..770.  With eight columns
// a lane picking one more value among them costs more than it saves (64 x 400 170..397 / 173..401): read from LDS there.
// Weights, prices, profits and labels are held doubled, and the price of a column that somebody holds is odd: of
// equally good columns the maximum then is one that nobody holds.
// Prices and profits are at most the largest weight (a price never exceeds the weight of the pair that holds it), which
// is below 2^28; a path is never longer than what its start would get; an infeasible pair's weight is taken as -2^28,
// farther than any path, and the doubled sums stay within 32 bits.
template <int C>
__global__ __launch_bounds__(SMALL_THREADS) void small_kernel(const int32_t *__restrict__ W, SmallShape s, long long K, int limit,
                                                              int32_t *__restrict__ out_row2col, int64_t *__restrict__ out_u,
                                                              int64_t *__restrict__ out_v, int *__restrict__ colmark,
                                                              mf_cert_out *__restrict__ out, unsigned long long *times)
{
    note_time(times, AT_SCORED);
    note_time(times, AT_SOLVE);
    extern __shared__ __align__(32) int lds[];
    // Rows of LDS: the weights of row r (negative: infeasible), its profit and the column it holds, from r * pitch on, which is
    // what names a row below; then zeros for the last lanes to read on into, the rows that wait, the prices.
    int *const weight = lds, *const profit = lds + s.pitch - 2, *const held = lds + s.pitch - 1;
    int *const waits = lds + s.n * s.pitch + 64 * C, *const price_out = waits + s.n;
    __shared__ int largest;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (threadIdx.x == 0) largest = 0;
    __syncthreads();
    {
        int most = 0;
        for (int j = lane; j < s.m; j += 64)
            for (int i0 = wave; i0 < s.n; i0 += SMALL_FETCH * (SMALL_THREADS / 64)) {
                int w[SMALL_FETCH];
#pragma unroll
                for (int q = 0; q < SMALL_FETCH; ++q)
                    w[q] = W[(size_t)min(i0 + q * (SMALL_THREADS / 64), s.n - 1) * s.ldw + j];
#pragma unroll
                for (int q = 0; q < SMALL_FETCH; ++q) {
                    const int i = i0 + q * (SMALL_THREADS / 64);
                    if (i >= s.n) break;
                    most = max(most, w[q]);
                    weight[i * s.pitch + j] = 2 * (w[q] < 0 || w[q] >= SMALL_WEIGHTS ? -SMALL_WEIGHTS : w[q]);
                }
            }
        most = wave_max(most);
        if (lane == 0) atomicMax(&largest, most);
        for (int j = threadIdx.x; j < s.m; j += SMALL_THREADS) colmark[j] = 0;
        for (int k = threadIdx.x; k < 64 * C; k += SMALL_THREADS) weight[s.n * s.pitch + k] = 0;
        for (int i = threadIdx.x; i < s.n; i += SMALL_THREADS) {
            for (int j = s.m; j < s.pitch - 2; ++j) weight[i * s.pitch + j] = 0;
            held[i * s.pitch] = -1;
            profit[i * s.pitch] = 0;
        }
        for (int j = threadIdx.x; j < s.m; j += SMALL_THREADS) price_out[j] = 0;
        if (threadIdx.x < MF_CERT_PARTS) mf_clear_part(out + threadIdx.x);
    }
    __syncthreads();
    const bool general = largest >= SMALL_WEIGHTS || K * (long long)largest >= MF_MAX_DUAL;
    if (wave == 0) {
        int bids = 0, scans = 0;
        bool over = false;
        if (!general) {
            // (lanes without a column read on into the next row, at a price that nobody pays)
            // (worth: the profit of a column's holder, where it is kept)
            constexpr bool KEPT = C <= 4;
            int price[C], holder[C], worth[C];
#pragma unroll
            for (int c = 0; c < C; ++c) { price[c] = lane * C + c < s.m ? 0 : 2 * SMALL_WEIGHTS; holder[c] = -1; worth[c] = 0; }
            typedef int Columns __attribute__((ext_vector_type(C)));
            auto weights_of = [&](int r) { return *(const Columns *)(weight + r + lane * C); };
            // what row r would have left of each column's weight at the prices
            int left[C];
            auto look = [&](int r) {
                const Columns w = weights_of(r);
#pragma unroll
                for (int c = 0; c < C; ++c) left[c] = w[c] - price[c];
            };
            auto even = [](int x) { return (x + 1) & ~1; };

            int waiting = 0;
            for (int row = 0; row < s.n; ++row) {
                if (bids >= limit) { over = true; break; }
                int r = row * s.pitch;
                for (;;) {
                    bids += 1;
                    look(r);
                    const Pick p = pick<C, false>(left, holder, worth, lane);
                    const int best = even(p.value), before = p.other;
                    if (best <= 0) { held[r] = -1; profit[r] = 0; break; }         // for good: prices only rise
                    set_column<C>(left, p.column, -2 * SMALL_WEIGHTS, lane);
                    const int second = even(max(largest_of<C>(left), 0));
                    if (before >= 0 && (second == best || bids >= SMALL_BIDS * s.n)) { waits[waiting++] = r; break; }
#pragma unroll
                    for (int c = 0; c < C; ++c)
                        if (p.column == lane * C + c) { price[c] = (price[c] + best - second) | 1; holder[c] = r; if constexpr (KEPT) worth[c] = second; }
                    held[r] = p.column;
                    profit[r] = second;
                    if (before < 0) break;
                    held[before] = -1;
                    r = before;
                }
            }

            for (int q = 0; q < waiting && !over; ++q) {
                const int start = __builtin_amdgcn_readfirstlane(waits[q]);
                // minus the length of the shortest path known, the row it comes from, and what it is worth to go there
                // (the lowest integer once it has been)
                int label[C], from[C], cap[C], open[C];
#pragma unroll
                for (int c = 0; c < C; ++c) { label[c] = INT32_MIN; from[c] = -1; cap[c] = lane * C + c < s.m ? INT32_MAX : INT32_MIN; }
                look(start);
                const int all = even(max(largest_of<C>(left), 0));
                int end = all, end_row = start, end_col = -1;      // the path that ends first: leave end_row unmatched
                int r = start, base = all;
                // (what a scan takes off the row's weights, and its base, are there before the weights are)
                Columns w = weights_of(start);
                int off[C];
#pragma unroll
                for (int c = 0; c < C; ++c) off[c] = price[c] + base;
                Pick p;
                for (;;) {                                         // (a column more is scanned each time)
                    scans += 1;
#pragma unroll
                    for (int c = 0; c < C; ++c) {
                        const int by_r = KEPT ? w[c] - off[c] : left[c] - base;     // (never above the label of a scanned column)
                        from[c] = by_r > label[c] ? r : from[c];
                        label[c] = max(label[c], by_r);
                        open[c] = min(label[c], cap[c]);
                    }
                    p = pick<C, KEPT>(open, holder, worth, lane);
                    if (min(p.value + (end - 1), p.other) < 0) break;       // the path known ends first, or a column that nobody holds
                    r = p.other;
                    if constexpr (KEPT) {
                        w = weights_of(r);
                        set_column<C>(cap, p.column, INT32_MIN, lane);
                        base = p.third - even(p.value);
#pragma unroll
                        for (int c = 0; c < C; ++c) off[c] = price[c] + base;
                    } else {
                        look(r);
                        const int has = __builtin_amdgcn_readfirstlane(profit[r]);
                        set_column<C>(cap, p.column, INT32_MIN, lane);
                        base = has - even(p.value);
                    }
                    end_row = base < end ? r : end_row;
                    end = min(base, end);
                }
                if (p.value > -end) { end = -p.value; end_col = p.column; }
                over = bids + scans >= limit;
                // the new duals: what was nearer than the path's end gives up the difference
#pragma unroll
                for (int c = 0; c < C; ++c)
                    if (cap[c] == INT32_MIN && lane * C + c < s.m) {
                        const int give = end + even(label[c]);
                        if (give > 0) {
                            price[c] += give;
                            if constexpr (KEPT) { worth[c] -= give; profit[holder[c]] = worth[c]; }
                            else profit[holder[c]] -= give;
                        }
                    }
                __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
                profit[start] = all - end;
                // and the path: columns change hands back to the start
                int k = end_col;
                if (k < 0) {
                    k = __builtin_amdgcn_readfirstlane(held[end_row]);
                    held[end_row] = -1;
                }
                for (int hop = 0; k >= 0 && hop < s.n; ++hop) {       // (the start holds nothing)
                    int mine = 0;
#pragma unroll
                    for (int c = 0; c < C; ++c) mine |= from[c] & (k % C == c ? -1 : 0);
                    const int to = __builtin_amdgcn_readlane(mine, k / C);
                    const int next = __builtin_amdgcn_readfirstlane(held[to]);
                    held[to] = k;
                    set_column<C>(holder, k, to, lane);
                    if constexpr (KEPT) set_column<C>(worth, k, profit[to], lane);
                    k = next;
                }
            }
#pragma unroll
            for (int c = 0; c < C; ++c)
                if (lane * C + c < s.m) price_out[lane * C + c] = price[c];
        }
        if (lane == 0) {
            out->bids = bids; out->scans = scans;
            out->status = general ? MF_SMALL_GENERAL : (over ? MF_ERR_NOT_CONVERGED : MF_OK);
        }
    }
    __syncthreads();
    for (int i = threadIdx.x; i < s.n; i += SMALL_THREADS) {
        out_u[i] = K * (long long)(profit[i * s.pitch] >> 1);
        out_row2col[i] = held[i * s.pitch];
    }
    for (int j = threadIdx.x; j < s.m; j += SMALL_THREADS) out_v[j] = K * (long long)(price_out[j] >> 1);
}

SmallShape small_shape(int n, int m, int64_t ldw, int *columns)
{
    *columns = m <= 64 ? 1 : (m <= 128 ? 2 : (m <= 256 ? 4 : 8));
    return SmallShape{n, m, (m + 2 + *columns - 1) / *columns * *columns, (long long)ldw};       // (whole loads)
}

size_t small_bytes(const SmallShape &s, int columns)
{
    return sizeof(int) * ((size_t)s.n * (size_t)s.pitch + 64 * (size_t)columns + (size_t)s.n + (size_t)s.m);
}

template <int C>
int launch_small(mf_ctx *ctx, const SmallShape &s, const int32_t *d_W, long long K, int32_t *d_row2col, int64_t *d_u, int64_t *d_v)
{
    static_assert(SMALL_COLS == 64 * 8, "the widest instance");
    const unsigned flag = 1u << (C == 1 ? 21 : (C == 2 ? 22 : (C == 4 ? 23 : 24)));
    if (!(ctx->kernels_configured & flag)) {
        MF_HIP(hipFuncSetAttribute((const void *)small_kernel<C>, hipFuncAttributeMaxDynamicSharedMemorySize, SMALL_LDS));
        ctx->kernels_configured |= flag;
    }
    hipLaunchKernelGGL((small_kernel<C>), dim3(1), dim3(SMALL_THREADS), small_bytes(s, C), ctx->stream, d_W, s, K,
                       (int)(ctx->max_rounds < INT32_MAX ? ctx->max_rounds : INT32_MAX), d_row2col, d_u, d_v, ctx->colmark, ctx->cert, ctx->times);
    MF_HIP(hipGetLastError());
    return MF_OK;
}

}  // namespace

bool mf_small_fits(const mf_ctx *ctx, int n, int m)
{
    int columns = 0;
    const SmallShape s = small_shape(n, m, 0, &columns);
    const bool few = s.n <= SMALL_ROWS || (s.n <= SMALL_ROWS_WIDE && 3 * s.m >= 4 * s.n && s.m <= SMALL_COLS_WIDE);
    return !ctx->as_told() && n <= m && few && s.m <= SMALL_COLS && small_bytes(s, columns) <= (size_t)SMALL_LDS;
}

// Leaves row2col, u, v with the caller and ctx->cert and ctx->colmark ready for the certificate.
int mf_launch_small(mf_ctx *ctx, const int32_t *d_W, int n, int m, int64_t ldw, int32_t *d_row2col, int64_t *d_u, int64_t *d_v)
{
    int columns = 0;
    const SmallShape s = small_shape(n, m, ldw, &columns);
    const long long K = (long long)n + 1;
    if (columns == 1) return launch_small<1>(ctx, s, d_W, K, d_row2col, d_u, d_v);
    if (columns == 2) return launch_small<2>(ctx, s, d_W, K, d_row2col, d_u, d_v);
    if (columns == 4) return launch_small<4>(ctx, s, d_W, K, d_row2col, d_u, d_v);
    return launch_small<8>(ctx, s, d_W, K, d_row2col, d_u, d_v);
}
