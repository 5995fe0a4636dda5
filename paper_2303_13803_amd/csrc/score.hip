// Edge weights for every online x offline pair (paper: Algorithm "Scheduling
// algorithm", the loop that calls CalcNormTput and AddEdge; Section
// "Matching-based scheduling" for the predictor's inputs and output).
//
// The predictor is an MLP 2F -> H -> H -> 1 over [online ; offline] features.
// Its first layer is linear in the concatenation, so it splits exactly into a
// per-online and a per-offline projection that are computed once per workload:
//     W1 [x_u ; x_v] + b1 = (W1[:, :F] x_u + b1) + (W1[:, F:] x_v).
// The pair kernel then only adds the two projections, applies ReLU, and runs
// the H x H hidden layer on the matrix cores with pairs along the N axis of
// the MFMA tile, so each lane ends up owning whole pairs and the output layer,
// logistic, quantisation and memory-fit mask run in registers before one
// coalesced int32 store.
#include "report.h"
#include <limits.h>
#include <math.h>
#include <type_traits>

typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef int intx4 __attribute__((ext_vector_type(4)));
typedef _Float16 half8 __attribute__((ext_vector_type(8)));
union Half8Words { half8 v; unsigned int u[4]; uint4 q; };

namespace {

// Both layer-1 projections, P_on = W1[:, :F] x + b1 and P_off = W1[:, F:] x, and the largest
// magnitude of everything the fp16 pieces are scaled by (range[0..4], as bit patterns of non-negative
// floats, which order like unsigned integers; zero on entry).
//
// A workgroup takes PROJECT_ROWS workloads of one side and 64 hidden units: lane k of every wavefront is
// hidden unit k of the slab, and a wavefront does PROJECT_ROWS / 4 rows, so that one LDS read of a weight
// (a row of 64, no conflicts) serves them all and a feature is a broadcast.  Weights and features are
// staged PROJECT_FEATURES at a time; the sum runs over the features in order, starting from the bias.  A
// thread per output, reading its weights 2F floats apart from its neighbour's, took 155 us a side for
// 20,000 workloads x 128 units where storing them takes 2, and the ranges another 40 us of reading it
// all back; both sides and the ranges now take 36 us.  The last PROJECT_EXTRA workgroups look at W2 and the SM term.
constexpr int PROJECT_ROWS = 32, PROJECT_FEATURES = 32, PROJECT_EXTRA = 4;

struct ProjectArgs {
    const float *X[2];                                     // features: online, offline
    int rows[2];
    float *P[2];
    const float *W1, *b1;
    int F, H;
    const float *range_of[3];                              // W2, W1sm, sm_off (the latter two may be null)
    int range_count[3];
    unsigned *range;                                       // null: not wanted
};

__device__ __forceinline__ void note_range(float mx, unsigned *slot, float *wave_mx)
{
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) mx = fmaxf(mx, __shfl_xor(mx, off));
    if ((threadIdx.x & 63) == 0) wave_mx[threadIdx.x >> 6] = mx;
    __syncthreads();
    if (threadIdx.x == 0) {
        mx = fmaxf(fmaxf(wave_mx[0], wave_mx[1]), fmaxf(wave_mx[2], wave_mx[3]));
        // the maximum only grows, so an outdated (smaller) cached value at worst costs a redundant atomic
        if (mx > 0.0f && __float_as_uint(mx) > *slot) atomicMax(slot, __float_as_uint(mx));
    }
    __syncthreads();
}

__global__ __launch_bounds__(256) void project_kernel(ProjectArgs a)
{
    __shared__ float w_lds[PROJECT_FEATURES][64];
    __shared__ float x_lds[PROJECT_ROWS][PROJECT_FEATURES];
    __shared__ float wave_mx[4];
    const int tiles_on = (a.rows[0] + PROJECT_ROWS - 1) / PROJECT_ROWS, tiles_off = (a.rows[1] + PROJECT_ROWS - 1) / PROJECT_ROWS;
    int tile = blockIdx.x;
    if (tile >= tiles_on + tiles_off) {
        if (!a.range || blockIdx.y > 0) return;
        tile -= tiles_on + tiles_off;
        for (int q = 0; q < 3; ++q) {
            if (!a.range_of[q]) continue;
            float mx = 0.0f;
            for (int i = tile * 256 + threadIdx.x; i < a.range_count[q]; i += PROJECT_EXTRA * 256) mx = fmaxf(mx, fabsf(a.range_of[q][i]));
            note_range(mx, &a.range[2 + q], wave_mx);
        }
        return;
    }
    const int side = tile >= tiles_on;
    if (side) tile -= tiles_on;
    const int k0 = blockIdx.y * 64, lane = threadIdx.x & 63, group = threadIdx.x >> 6;
    constexpr int MINE = PROJECT_ROWS / 4;
    const int row0 = tile * PROJECT_ROWS, rows = min(PROJECT_ROWS, a.rows[side] - row0);
    const float *X = a.X[side] + (size_t)row0 * a.F, *W = a.W1 + (size_t)k0 * 2 * a.F + (side ? a.F : 0);
    float sum[MINE];
#pragma unroll
    for (int r = 0; r < MINE; ++r) sum[r] = side == 0 ? a.b1[k0 + lane] : 0.0f;
    for (int t0 = 0; t0 < a.F; t0 += PROJECT_FEATURES) {
        const int depth = min(PROJECT_FEATURES, a.F - t0);
        __syncthreads();
        for (int e = threadIdx.x; e < 64 * PROJECT_FEATURES; e += 256) {
            const int k = e / PROJECT_FEATURES, t = e % PROJECT_FEATURES;
            if (t < depth) w_lds[t][k] = W[(size_t)k * 2 * a.F + t0 + t];
        }
        for (int e = threadIdx.x; e < PROJECT_ROWS * PROJECT_FEATURES; e += 256) {
            const int r = e / PROJECT_FEATURES, t = e % PROJECT_FEATURES;
            if (t < depth) x_lds[r][t] = r < rows ? X[(size_t)r * a.F + t0 + t] : 0.0f;
        }
        __syncthreads();
        for (int t = 0; t < depth; ++t) {
            const float w = w_lds[t][lane];
#pragma unroll
            for (int r = 0; r < MINE; ++r) sum[r] = fmaf(x_lds[group * MINE + r][t], w, sum[r]);
        }
    }
    float mx = 0.0f;
#pragma unroll
    for (int r = 0; r < MINE; ++r) {
        const int row = group * MINE + r;
        if (row < rows) {
            a.P[side][(size_t)(row0 + row) * a.H + k0 + lane] = sum[r];
            mx = fmaxf(mx, fabsf(sum[r]));
        }
    }
    if (a.range) note_range(mx, &a.range[side], wave_mx);
}

// What is prepared per workload before anything is ordered: its memory fraction and SM share, its rank
// (zero), and the words later kernels of the call count or take maxima in.
struct SetupArgs {
    const float *X[2];                                     // online, offline
    int rows[2];
    int F, mem_feature, sm_feature[2];                     // sm_feature < 0: none
    float *mem[2], *sm[2];
    int32_t *rank[2], *order[2];                           // null: this side is not ordered
    unsigned long long *keys[2];                           // [rows] where many keys are sorted
    const int32_t *group;                                  // of the online side: order by group first (optional)
    float *sorted[2];                                      // null: not wanted
    int32_t *fit_len[2];
    int32_t *staged;                                       // the matrix in memory order, 16-byte aligned,
    int64_t pitch;                                         // a multiple of four
    float mem_limit;
    int slice[2];
    unsigned long long *pairs_evaluated, *feasible_pairs;
    int *largest;
    unsigned *range;
    int *queue, launches;                                  // counters of the next task, for so many launches of the pair kernel
    unsigned long long *times;
};

__global__ __launch_bounds__(256) void setup_kernel(SetupArgs a)
{
    note_time(a.times, AT_SCORE);
    const int side = blockIdx.y, r = blockIdx.x * 256 + threadIdx.x;
    if (side == 0 && blockIdx.x == 0)
        for (int q = r; q < a.launches * MF_PAIR_QUEUES; q += 256) *(int4 *)(a.queue + q * MF_PAIR_QUEUE_STEP) = make_int4(0, 0, 0, 0);
    if (side == 0 && r < 8) {
        a.range[r] = 0u;
        if (r == 0) { *a.pairs_evaluated = 0ull; if (a.feasible_pairs) *a.feasible_pairs = 0ull; if (a.largest) *a.largest = 0; }
    }
    if (r >= a.rows[side]) return;
    const float *x = a.X[side] + (size_t)r * a.F;
    a.mem[side][r] = x[a.mem_feature];
    if (a.sm_feature[side] >= 0) a.sm[side][r] = x[a.sm_feature[side]];
    if (a.rank[side]) a.rank[side][r] = 0;
}

// order[k] = the workload with the k-th smallest key (ties by index).  Keys are
// compared through the usual order-preserving map of float bits to unsigned
// integers, so the result is a permutation whatever the keys hold.  A plain
// rank count: count^2 comparisons, staged through LDS, is microseconds at the
// sizes a weight matrix fits in memory for.
__device__ __forceinline__ unsigned ordered_bits(float x)
{
    const unsigned b = __float_as_uint(x);
    return (b & 0x80000000u) ? ~b : (b | 0x80000000u);
}

constexpr int RANK_THREADS = 256, RANK_TILE = 2048;

// rank[i] += number of keys in [first, last) that sort before key i.  The y
// extent of the grid splits the comparisons into slices so that a few thousand
// keys still fill the device; rank[] starts at zero.  With GROUPED the order is
// by group first (group[i] in [0, 2^15)) and by key within a group.
template <bool GROUPED>
__device__ __forceinline__ void count_ranks(const float *__restrict__ key, const int32_t *__restrict__ group, int count,
                                            int slice, int32_t *__restrict__ rank, unsigned *tile, int *gtile)
{
    const int i = blockIdx.x * RANK_THREADS + threadIdx.x;
    const unsigned mine = i < count ? ordered_bits(key[i]) : 0u;
    const int gmine = (GROUPED && i < count) ? group[i] : 0;
    const int first = blockIdx.y * slice, last = min(count, first + slice);
    const int ties_upto = min(i, last);                 // equal keys count when they sit earlier; padding never does
    int before = 0;
    for (int base = first; base < last; base += RANK_TILE) {
        const int lim = min(RANK_TILE, last - base);
        __syncthreads();
        for (int t = threadIdx.x; t < RANK_TILE; t += RANK_THREADS) {
            tile[t] = t < lim ? ordered_bits(key[base + t]) : 0xffffffffu;      // padding sorts after everything
            if (GROUPED) gtile[t] = t < lim ? group[base + t] : 0x7fffffff;
        }
        __syncthreads();
        const int upto = (lim + 3) & ~3;
        // a stretch of keys that all sit earlier than this workgroup's, or all later: one comparison decides
        // also between equal ones (two instructions a key, not seven)
        const int own = blockIdx.x * RANK_THREADS;
        if (!GROUPED && (base + lim <= own || base >= own + RANK_THREADS)) {
            const bool earlier = base < own;
            for (int t = 0; t < upto; t += 4) {
                const uint4 v = *(const uint4 *)(tile + t);
                if (earlier) before += (v.x <= mine) + (v.y <= mine) + (v.z <= mine) + (v.w <= mine);
                else before += (v.x < mine) + (v.y < mine) + (v.z < mine) + (v.w < mine);
            }
            continue;
        }
        for (int t = 0; t < upto; t += 4) {
            const uint4 v = *(const uint4 *)(tile + t);
            const int at = base + t;
            int c0 = (v.x < mine) + ((v.x == mine) & (at < ties_upto));
            int c1 = (v.y < mine) + ((v.y == mine) & (at + 1 < ties_upto));
            int c2 = (v.z < mine) + ((v.z == mine) & (at + 2 < ties_upto));
            int c3 = (v.w < mine) + ((v.w == mine) & (at + 3 < ties_upto));
            if (GROUPED) {
                const int4 g = *(const int4 *)(gtile + t);
                c0 = (g.x < gmine) + ((g.x == gmine) & c0);
                c1 = (g.y < gmine) + ((g.y == gmine) & c1);
                c2 = (g.z < gmine) + ((g.z == gmine) & c2);
                c3 = (g.w < gmine) + ((g.w == gmine) & c3);
            }
            before += c0 + c1 + c2 + c3;
        }
    }
    if (i < count && before) atomicAdd(&rank[i], before);
}

// The same ranks for many keys: counting compares every key with every other, 200 us for 20,000 and 40,000 of them.  Here a
// workgroup sorts SORT_TILE keys in LDS (bitonic, 66 steps with a barrier each), and every key then looks itself up in
// every sorted stretch, a thread for each SORT_STRETCHES of those.  What bounds either is latency, of the steps
// and of the twelve dependent reads of a look-up (four stretches at once).  20,000 + 40,000 keys 210 -> 31 us, 20,000 + 20,000 83 -> 31; 6001 + 9007
// and fewer take less by counting (22 us), so the line is at SORT_FROM keys on one side, where both take as long.
constexpr int SORT_TILE = 2048, SORT_THREADS = SORT_TILE / 2, SORT_STRETCHES = 4, SORT_FROM = 12288;

__global__ __launch_bounds__(SORT_THREADS) void rank_sort_kernel(SetupArgs a)
{
    __shared__ unsigned long long keys[SORT_TILE];
    const int side = blockIdx.z, count = a.rows[side], base = blockIdx.x * SORT_TILE;
    if (!a.rank[side] || base >= count) return;
    for (int t = threadIdx.x; t < SORT_TILE; t += SORT_THREADS) {
        const int i = base + t;
        // by group, key and index: no two are the same
        const unsigned long long group = side == 0 && a.group && i < count ? (unsigned long long)a.group[i] : 0ull;
        keys[t] = i < count ? group << 52 | (unsigned long long)ordered_bits(a.mem[side][i]) << 20 | (unsigned long long)i : ~0ull;
    }
    for (int k = 2; k <= SORT_TILE; k <<= 1)
        for (int j = k >> 1; j > 0; j >>= 1) {
            __syncthreads();
            const int t = threadIdx.x, i = ((t & ~(j - 1)) << 1) | (t & (j - 1));
            const unsigned long long x = keys[i], y = keys[i | j];
            if ((x > y) == ((i & k) == 0)) { keys[i] = y; keys[i | j] = x; }
        }
    __syncthreads();
    for (int t = threadIdx.x; t < SORT_TILE; t += SORT_THREADS)
        if (base + t < count) a.keys[side][base + t] = keys[t];
}

__global__ __launch_bounds__(256) void rank_merge_kernel(SetupArgs a)
{
    const int side = blockIdx.z, count = a.rows[side], e = blockIdx.x * 256 + threadIdx.x;
    const int first = blockIdx.y * SORT_STRETCHES * SORT_TILE;
    if (!a.rank[side] || e >= count || first >= count) return;
    const unsigned long long *keys = a.keys[side] + first, key = a.keys[side][e];
    int at[SORT_STRETCHES];                                // keys of the stretch that sort before this one
#pragma unroll
    for (int q = 0; q < SORT_STRETCHES; ++q) at[q] = 0;
#pragma unroll
    for (int step = SORT_TILE; step > 0; step >>= 1)
#pragma unroll
        for (int q = 0; q < SORT_STRETCHES; ++q) {
            const int to = at[q] + step;
            if (to <= SORT_TILE && first + q * SORT_TILE + to <= count && keys[q * SORT_TILE + to - 1] < key) at[q] = to;
        }
    int before = 0;
#pragma unroll
    for (int q = 0; q < SORT_STRETCHES; ++q) before += at[q];
    if (before) atomicAdd(&a.rank[side][(int)(key & 0xfffffull)], before);
}

// Both sides of the matrix (blockIdx.z).
__global__ __launch_bounds__(RANK_THREADS) void rank_count_kernel(SetupArgs a)
{
    __shared__ __align__(16) unsigned tile[RANK_TILE];
    __shared__ __align__(16) int gtile[RANK_TILE];
    const int side = blockIdx.z, count = a.rows[side];
    if (!a.rank[side] || (int)blockIdx.x * RANK_THREADS >= count || (int)blockIdx.y * a.slice[side] >= count) return;
    if (side == 0 && a.group) count_ranks<true>(a.mem[0], a.group, count, a.slice[0], a.rank[0], tile, gtile);
    else count_ranks<false>(a.mem[side], nullptr, count, a.slice[side], a.rank[side], tile, gtile);
}

__global__ __launch_bounds__(256) void order_kernel(SetupArgs a)
{
    const int side = blockIdx.y, i = blockIdx.x * 256 + threadIdx.x;
    if (!a.rank[side] || i >= a.rows[side]) return;
    const int at = a.rank[side][i];
    a.order[side][at] = i;
    if (a.sorted[side]) a.sorted[side][at] = a.mem[side][i];
}

// In memory order the pairs that can share form, in every row, a prefix of the columns (and in
// every column a prefix of the rows): len[k] = how many entries of `other` (ascending) fit next
// to mine[k].  A binary search on the same float32 rule the marks were written with.
// (columns with rows ordered by group first: count of all rows.)  Also how many pairs can share at all.
//
// The staged matrix has rows and columns in that order.  The scoring kernel writes the prefixes, and everything that
// reads a row reads its prefix only, in groups of four: so all it needs besides are infeasible marks in the group
// the prefix ends in (paper: Section "Implementation", the memory quota).  Marking the rest, as was done
// before, wrote 2.9 GB for 20,000 x 40,000 pairs of which a tenth can share, 0.8 ms.
__global__ __launch_bounds__(256) void fit_prefix_kernel(SetupArgs a)
{
    const int side = blockIdx.y, k = blockIdx.x * 256 + threadIdx.x;
    int len = 0;
    if (k < a.rows[side]) {
        if (side == 1 && a.group) len = a.rows[0];
        else {
            const float mine = a.sorted[side][k];
            const float *other = a.sorted[1 - side];
            int lo = 0, hi = a.rows[1 - side];             // first position that does not fit
            while (lo < hi) {
                const int mid = (lo + hi) >> 1;
                if (mine + other[mid] > a.mem_limit) hi = mid; else lo = mid + 1;
            }
            len = lo;
        }
        a.fit_len[side][k] = len;
        if (side == 0 && (len & 3)) {
            const int first = len & ~3, m = a.rows[1];
            int32_t w[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) w[e] = first + e >= len && first + e < m ? MF_INFEASIBLE : 0;
            *(int4 *)(a.staged + (size_t)k * a.pitch + first) = make_int4(w[0], w[1], w[2], w[3]);
        }
    }
    if (side) return;
    unsigned long long t = (unsigned)len;
    for (int off = 32; off >= 1; off >>= 1) t += __shfl_xor(t, off);
    if ((threadIdx.x & 63) == 0 && t) atomicAdd(a.feasible_pairs, t);
}

// The placement kernels see every weight once more: they note the largest on the way (the
// matching's first epsilon is set by it), at most one atomic per workgroup and only when it has
// news.  Every thread of the NT-thread workgroup calls this.
template <int NT>
__device__ inline void note_largest(int mx, int *largest)
{
    __shared__ int wave_largest[NT / 64];
    for (int off = 32; off >= 1; off >>= 1) mx = max(mx, __shfl_xor(mx, off));
    if ((threadIdx.x & 63) == 0) wave_largest[threadIdx.x >> 6] = mx;
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int wv = 1; wv < NT / 64; ++wv) mx = max(mx, wave_largest[wv]);
        // the maximum only grows, so an outdated (smaller) cached value at worst costs a redundant atomic
        if (mx > *largest) atomicMax(largest, mx);
    }
}

// Puts the staged scores in place: W[i][j] = S[rank_on[i]][rank_off[j]].  General form: a row of
// S is read back in scattered 4-byte pieces, every piece of it by the same workgroup while it
// sits in the caches.
__global__ __launch_bounds__(256) void place_kernel(const int32_t *__restrict__ S, int64_t lds,
                                                    const int32_t *__restrict__ rank_on,
                                                    const int32_t *__restrict__ rank_off,
                                                    const int32_t *__restrict__ fit_len, int n, int m,
                                                    int32_t *__restrict__ W, int64_t ldw, int wide_stores,
                                                    int *largest, unsigned long long *times)
{
    note_time(times, AT_PLACE);
    const int i = blockIdx.x, from = rank_on[i], len = fit_len[from];       // entries at or beyond len cannot share
    const int32_t *src = S + (size_t)from * lds;
    int32_t *row = W + (size_t)i * ldw;
    int mx = 0;                                             // "cannot share" is the smallest integer
    auto entry = [&](int p) { const int32_t w = p < len ? src[p] : MF_INFEASIBLE; mx = max(mx, w); return w; };
    const int whole = m & ~3;
    for (int j = (blockIdx.y * 256 + threadIdx.x) * 4; j < whole; j += gridDim.y * 1024) {
        const int4 p = *(const int4 *)(rank_off + j);
        const int4 w = make_int4(entry(p.x), entry(p.y), entry(p.z), entry(p.w));
        if (wide_stores) *(int4 *)(row + j) = w;
        else { row[j] = w.x; row[j + 1] = w.y; row[j + 2] = w.z; row[j + 3] = w.w; }
    }
    if (blockIdx.y == 0 && whole + (int)threadIdx.x < m) row[whole + threadIdx.x] = entry(rank_off[whole + threadIdx.x]);
    note_largest<256>(mx, largest);
}

// The same through LDS: a
// workgroup per row loads the staged row in whole lines - only as far as its pairs can share,
// everything beyond is a mark anyway - picks each output's entry out of LDS, and stores the row
// in whole lines: no scattered access reaches the caches.  LDS takes PLACE_LDS_ENTRIES of a row, so that a
// compute unit has two workgroups, one storing while the other loads; what a longer prefix has beyond that is
// picked out of the caches (20,000 x 40,000 with prefixes of 4000 entries on average: 1.16 ms with LDS for whole rows
// and one workgroup a compute unit, 1.06 so).  What bounds it is storing the row (3.2 GB there), if the entries' places are
// read by fours and the reads of four steps are on their way together: 1.06 -> 0.73 ms, 20,000 x 20,000 0.66 -> 0.53, when they were read
// one by one and waited for in every step.
constexpr int PLACE_THREADS = 1024, PLACE_LDS_ENTRIES = 79 * 256;

// Which of the two.  A workgroup has a whole row with LDS, and a part of one without, which is faster where long rows do not give every compute unit its
// two, and beyond 200,000 columns, most of whose prefixes do not fit in LDS.  A whole pass without / with, ms: 2000 x 45,000 3.28 / 2.37, 2000 x
// 200,000 16.0 / 13.6, with a tenth of the pairs 4.09 / 3.72, and 16,000 x 48,900 7.98 / 7.12; 64 x 100,000 0.30 / 0.33, 30 x 60,000
// 0.140 / 0.155, 192 x 200,000 with a tenth 0.69 / 0.74, 300 x 300,000 1.49 / 1.53.  Up to 40,704 columns they differ by 2 %, from 40,000 and for 30
// rows and fewer by 5 to 11 %.
constexpr int64_t PLACE_LONGEST = 200000, PLACE_SHORT = 40704;
constexpr int PLACE_MANY = 512;
bool place_by_lds(int n, int64_t columns) { return columns <= PLACE_SHORT || (n >= PLACE_MANY && columns <= PLACE_LONGEST); }

__global__ __launch_bounds__(PLACE_THREADS) void place_lds_kernel(
    const int32_t *__restrict__ S, int64_t lds, const int32_t *__restrict__ rank_on,
    const int32_t *__restrict__ rank_off, const int32_t *__restrict__ fit_len, int n, int m,
    int32_t *__restrict__ W, int64_t ldw, int wide_stores, int *largest, unsigned long long *times)
{
    note_time(times, AT_PLACE);
    __shared__ int32_t staged[PLACE_LDS_ENTRIES];
    const int i = blockIdx.x, tid = threadIdx.x;
    const int from = rank_on[i];
    const int32_t *src = S + (size_t)from * lds;
    const int len = fit_len[from];                          // staged entries at or beyond it are marks
    int32_t *row = W + (size_t)i * ldw;
    int mx = 0;                                             // "cannot share" is the smallest integer
    for (int t = tid * 4; t < len; t += PLACE_THREADS * 4) {
        const int4 v = *(const int4 *)(src + t);            // the last group may reach into the marks
        if (t < PLACE_LDS_ENTRIES) *(int4 *)(staged + t) = v;
        mx = max(max(mx, max(v.x, v.y)), max(v.z, v.w));
    }
    note_largest<PLACE_THREADS>(mx, largest);               // passes a barrier: the staged row is complete
    auto entry = [&](int p) { return p < len ? (p < PLACE_LDS_ENTRIES ? staged[p] : src[p]) : MF_INFEASIBLE; };
    const int whole = m & ~3;
#pragma unroll 4
    for (int j = tid * 4; j < whole; j += PLACE_THREADS * 4) {
        const int4 p = *(const int4 *)(rank_off + j);
        const intx4 w = {entry(p.x), entry(p.y), entry(p.z), entry(p.w)};
        if (wide_stores == 2) __builtin_nontemporal_store(w, (intx4 *)(row + j));
        else if (wide_stores) *(intx4 *)(row + j) = w;
        else { row[j] = w.x; row[j + 1] = w.y; row[j + 2] = w.z; row[j + 3] = w.w; }
    }
    if (whole + tid < m) row[whole + tid] = entry(rank_off[whole + tid]);
}

__global__ void fill_flag_kernel(int *flag) { *flag = 0; }

__global__ void range_clear_kernel(unsigned *slots)
{
    if (threadIdx.x < 8) slots[threadIdx.x] = 0u;
}

template <int H> struct PairShape {
    static constexpr int WAVES = H == 128 ? 8 : 4;         // wavefronts that share an LDS copy of W2 and its pieces,
    static constexpr int THREADS = WAVES * 64;
    static constexpr int PER_UNIT = H == 128 ? 1 : 3;      // such workgroups a compute unit: two wavefronts a SIMD, or three
    static constexpr int ROWS = 16;                        // online rows a wavefront has in LDS at a time
    static constexpr int KS = H / 2;                       // k-steps of the 32x32x2 tile
    static constexpr int MB = H / 32;                      // 32-row blocks of the hidden layer
    static constexpr int WAVE_FLOATS = ROWS * H + 2 * ROWS;
    static constexpr size_t LDS_BYTES = sizeof(float) * ((size_t)H * H + 4 * H + 4 + (size_t)WAVES * WAVE_FLOATS);
};

// One wavefront owns 32 offline columns (lane & 31) and walks down the online
// rows of a task: those columns beside task_rows rows.  n and m count the rows and columns to score; with
// row_map / col_map (either may be null) entry t of the map names the online
// row / offline column that position t stands for, so a scattered subset
// of rows or columns can be re-scored in place.
//
// Workgroups stay (but see pair_tasks.h): each makes W2's pieces once, then its wavefronts take one task after the other, each on its
// own, the rows' projections in LDS of their own, with no barrier.  What bounds the kernel is the matrix pipe at the clock that
// power allows: the matrix instructions alone, on operands as they occur here, take 17.9 ns each and 21.4 with four
// vector instructions and the reads of W2 beside them (constants, which toggle nothing: 13.5), so the 9.6e8 of
// 20,000 x 20,000 pairs take 16.8 and 20.1 ms.  A workgroup per tile of 64 x 256 pairs set itself up
// for each (7 percent of its time, and nothing else fits into the compute unit meanwhile), waited for its slowest
// wavefront, and was launched for every tile that cannot fit as well.  Before / now: 20,000 x 20,000 23.0 / 22.2 ms,
// 20,000 x 40,000 with a tenth of the pairs 6.85 / 5.9, 4096 x 8192 2.10 / 1.93, 777 x 1501 0.134 / 0.090.
//
// v_mfma_f32_32x32x2_f32 computes D[32x32] += A[32x2] B[2x32]
// with lane l supplying A[l%32][l/32] and B[l/32][l%32]; we let the two k
// slots of step s be hidden features s and H/2 + s, so each half-wave streams
// a contiguous half of the projections.  Accumulator register r of lane l is
// D[8*(r/4) + 4*(l/32) + r%4][l%32].
// PAIR_SM: the predictor has a third input, the SM share of the pair
// min(1 - sm_on[i], sm_off[j]); its layer-1 weights w_sm[H] add w_sm[k] * share to hidden unit k.
// SLOWDOWN: a second output unit on the same hidden layers (weights w3_slow[H], b3_slow) predicts
// how much the online workload of the pair slows down; a pair above slow_limit is infeasible.
// SPLIT: the hidden layer's products are formed from half-precision pieces.  Every fp32 operand is
// x = hi + lo with hi = x rounded to fp16 and lo = the fp16 of the exact remainder (together 22
// significant bits; the hardware keeps fp16 subnormals), and w * h = w_hi h_hi + w_hi h_lo + w_lo h_hi
// up to 2^-22 relative, accumulated in fp32 by v_mfma_f32_32x32x16_f16: three matrix instructions
// of 16,384 multiply-adds in 8 passes each where fp32 operands need eight of 2,048 in 16 passes
// each.  Measured against the fp64 reference the scores are as close as those of the fp32 products
// (largest relative error 3-4e-7 on every benchmark configuration).  fp16 ends at 65,504 and
// thins out below 6e-5, so both operands are first scaled by powers of two (exact) that bring the
// largest weight, and the largest value a layer-1 unit can take, to about 2^13: `range` holds the
// largest magnitudes of the projections, of W2 and of the SM term, found by project_kernel; the
// accumulators then carry the product of the two scales, which b2 is given on the way in and W3
// takes out again.  The result therefore does not depend on the size of the numbers.
// For lane l, element t of its operand of k-block kb is hidden unit (l / 32) * H/2 + 8 kb + t, for
// A (rows of W2) and B (pairs) alike.
template <int H, bool PAIR_SM, bool SLOWDOWN, bool SPLIT, bool LONG>
__global__ __launch_bounds__(PairShape<H>::THREADS, PairShape<H>::PER_UNIT * PairShape<H>::WAVES / 4) void pair_mlp_kernel(
    const float *__restrict__ P_on, const float *__restrict__ P_off,
    const float *__restrict__ W2, const float *__restrict__ b2, const float *__restrict__ W3,
    const float *__restrict__ b3, const float *__restrict__ mem_on,
    const float *__restrict__ mem_off, int n, int m, float scale, float mem_limit,
    int32_t *__restrict__ W, int64_t ldw, float *__restrict__ sigma,
    const int32_t *__restrict__ row_map, const int32_t *__restrict__ col_map, int by_memory,
    unsigned long long *__restrict__ evaluated, const int32_t *__restrict__ segment,
    const float *__restrict__ w_sm, const float *__restrict__ sm_on, const float *__restrict__ sm_off,
    const float *__restrict__ w3_slow, const float *__restrict__ b3_slow, float slow_limit,
    const unsigned *__restrict__ range, float units, const unsigned long long *__restrict__ feasible, const int32_t *__restrict__ fit_len,
    int *__restrict__ next_task, int begin, unsigned long long *times)
{
    note_time(times, AT_PAIRS);
    using S = PairShape<H>;
    constexpr int KS = S::KS, MB = S::MB, ROWS = S::ROWS, Q = KS / 4, KB = H / 16;
    extern __shared__ float4 lds4[];
    float4 *a_lds = lds4;                                  // [MB][Q][64] float4: MFMA A operand order
    uint4 *a16_lds = (uint4 *)lds4;                        // SPLIT: [2 pieces][MB][KB][64] eight fp16 each (the same bytes)
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int hh = lane >> 5, nn = lane & 31;
    float *b2_lds = (float *)(lds4) + H * H;
    float *w3_lds = b2_lds + H;
    float *wsm_lds = w3_lds + H;                           // [H] layer-1 weights of the SM share
    float *w3s_lds = wsm_lds + H;                          // [H] output weights of the slowdown unit
    unsigned long long *scored_lds = (unsigned long long *)(w3s_lds + H);  // pairs the workgroup has scored
    int *ended_lds = (int *)(scored_lds + 1);              // its wavefronts that are done
    int *leave_lds = ended_lds + 1;                        // it leaves (before its set-up: nothing is left to do)
    float *pon_lds = w3s_lds + H + 4 + wave * S::WAVE_FLOATS;  // this wavefront's own: [ROWS][H] projections,
    float *mon_lds = pon_lds + ROWS * H;                   // [ROWS] memory fractions and
    float *son_lds = mon_lds + ROWS;                       // [ROWS] 1 - SM activities of its rows

    const int blocks = (m + 31) / 32;
    // blocks of columns that a row has: in memory order as many as fit, on average, and the last one in part
    const float row_blocks = by_memory ? (float)*feasible / (32.0f * (float)n) + 0.5f : (float)blocks;
    int staged_row0 = 0;                    // where the row map's entry 0 sits in the staged matrix
    if (segment) {                          // only entries [segment[0], segment[1]) of the row map
        row_map += segment[0];
        staged_row0 = segment[0];
        n = segment[1] - segment[0];
    }
    const int task_rows = __builtin_amdgcn_readfirstlane(pair_task_rows(H, (float)n * row_blocks, units));
    const int first = LONG ? begin : (int)gridDim.x, later = (int)gridDim.x - first, queue = pair_queue(blockIdx.x, first);
    int *const next = next_task + queue * MF_PAIR_QUEUE_STEP;
    if (LONG && (int)blockIdx.x >= first) {
        if (tid == 0) *leave_lds = __hip_atomic_load(next + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __syncthreads();
        if (*leave_lds) return;
        if (tid == 0) atomicAdd(next + 2, 1);
    }
    if (LONG && tid == 0 && ((int)blockIdx.x >= first || (int)blockIdx.x < pair_queues(first)))
        __hip_atomic_store(next + 3, (int)device_time(), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    // SPLIT: the powers of two that scale layer-1 values and W2 into fp16's comfortable range
    float scale_p = 1.0f, scale_w = 1.0f;
    if (SPLIT) {
        auto toward_8192 = [](float largest) {
            if (!(largest > 0.0f) || !(largest < 3.0e38f)) return 1.0f;
            return ldexpf(1.0f, max(-60, min(60, 13 - ilogbf(largest))));
        };
        const float sm_term = PAIR_SM ? __uint_as_float(range[3]) * fmaxf(1.0f, __uint_as_float(range[4])) : 0.0f;
        scale_p = toward_8192(__uint_as_float(range[0]) + __uint_as_float(range[1]) + sm_term);
        scale_w = toward_8192(__uint_as_float(range[2]));
    }
    const float scale_acc = scale_p * scale_w, unscale_acc = 1.0f / scale_acc;
    if (SPLIT) {
        for (int idx = tid; idx < MB * KB * 64; idx += S::THREADS) {
            const int ln = idx & 63, kb = (idx >> 6) % KB, mb = idx / (64 * KB);
            const float *src = W2 + (size_t)(mb * 32 + (ln & 31)) * H + (ln >> 5) * KS + kb * 8;
            const float4 w0 = *(const float4 *)src, w1 = *(const float4 *)(src + 4);
            const float w[8] = {w0.x, w0.y, w0.z, w0.w, w1.x, w1.y, w1.z, w1.w};
            Half8Words hi, lo;
#pragma unroll
            for (int t = 0; t < 8; ++t) {
                const float ws = w[t] * scale_w;
                const _Float16 h = (_Float16)ws;
                hi.v[t] = h;
                lo.v[t] = (_Float16)(ws - (float)h);
            }
            a16_lds[(mb * KB + kb) * 64 + ln] = hi.q;
            a16_lds[((MB + mb) * KB + kb) * 64 + ln] = lo.q;
        }
    } else {
        for (int idx = tid; idx < MB * Q * 64; idx += S::THREADS) {
            int ln = idx & 63, s4 = (idx >> 6) % Q, mb = idx / (64 * Q);
            a_lds[idx] = *(const float4 *)(W2 + (size_t)(mb * 32 + (ln & 31)) * H + (ln >> 5) * KS + s4 * 4);
        }
    }
    if (tid < H) { b2_lds[tid] = b2[tid] * scale_acc; w3_lds[tid] = W3[tid] * unscale_acc; }
    if (tid == 0) { *scored_lds = 0ull; *ended_lds = 0; *leave_lds = 0; }
    if (PAIR_SM && tid < H) wsm_lds[tid] = w_sm[tid] * scale_p;
    if (SLOWDOWN && tid < H) w3s_lds[tid] = w3_slow[tid] * unscale_acc;
    __syncthreads();

    // what the wavefront's lanes keep of their column while they walk down a task's rows
    float poff[KS], moff = 0.0f, soff = 0.0f;
    int j = 0, jc = 0, row0 = 0;
    const float bias3 = b3[0];
    const float bias3_slow = SLOWDOWN ? b3_slow[0] : 0.0f;
    // NR of the wavefront's rows at once against this wavefront's 32 columns.  Two rows share every
    // W2 operand fetched from LDS and give the matrix pipe two independent accumulator sets.
    auto score_rows = [&](auto nr_tag, auto split_tag, const int r) {
        constexpr int NR = decltype(nr_tag)::value;
        constexpr bool SPLIT_HERE = decltype(split_tag)::value;
        floatx16 acc[NR][MB];
        // b2, what the accumulators start from: the addend of a block's first matrix instructions, read by every
        // row's from the same registers (copies of it were 64 instructions a row)
        auto bias_of = [&](const int mb) {
            floatx16 b;
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                const float4 bv = *(const float4 *)(b2_lds + mb * 32 + 8 * g + 4 * hh);
                b[4 * g] = bv.x; b[4 * g + 1] = bv.y; b[4 * g + 2] = bv.z; b[4 * g + 3] = bv.w;
            }
            return b;
        };
        float share[NR];
#pragma unroll
        for (int x = 0; x < NR; ++x) share[x] = PAIR_SM ? fminf(son_lds[r + x], soff) : 0.0f;
        if constexpr (SPLIT_HERE) {
            float minus_one = -1.0f;
            asm volatile("" : "+s"(minus_one));             // no instruction: only hides the constant from the optimiser
            // the two fp16 pieces of this lane's eight layer-1 values of k-block kb, for row r + x
            auto pieces = [&](const int kb, const int x, const float4 &p0, const float4 &p1, Half8Words &hi, Half8Words &lo) {
                const float pq[8] = {p0.x, p0.y, p0.z, p0.w, p1.x, p1.y, p1.z, p1.w};
                float y[8];
                if (PAIR_SM) {
                    const float4 s0 = *(const float4 *)(wsm_lds + hh * KS + 8 * kb);
                    const float4 s1 = *(const float4 *)(wsm_lds + hh * KS + 8 * kb + 4);
                    const float ws[8] = {s0.x, s0.y, s0.z, s0.w, s1.x, s1.y, s1.z, s1.w};
#pragma unroll
                    for (int t = 0; t < 8; ++t) y[t] = fmaxf(fmaf(ws[t], share[x], pq[t] + poff[8 * kb + t]), 0.0f);
                } else {
#pragma unroll
                    for (int t = 0; t < 8; ++t) y[t] = fmaxf(pq[t] + poff[8 * kb + t], 0.0f);
                }
#pragma unroll
                for (int t = 0; t < 4; ++t) {
                    // toward zero, so the remainder keeps the sign; it is exact in fp32
                    const auto h2 = __builtin_amdgcn_cvt_pkrtz(y[2 * t], y[2 * t + 1]);
                    hi.u[t] = __builtin_bit_cast(unsigned int, h2);
                    // y - hi written as a fused multiply-add by a -1 the optimiser cannot see: it is then
                    // selected as the mixed-precision instruction that reads the fp16 piece itself, one
                    // instruction per value instead of a conversion and a subtraction (same value: the
                    // remainder is exact either way)
                    const auto l2 = __builtin_amdgcn_cvt_pkrtz(__builtin_fmaf((float)h2[0], minus_one, y[2 * t]),
                                                               __builtin_fmaf((float)h2[1], minus_one, y[2 * t + 1]));
                    lo.u[t] = __builtin_bit_cast(unsigned int, l2);
                }
            };
            // W2's pieces for step (kb, mb) + 1 are requested from LDS before the matrix instructions of
            // step (kb, mb) are issued, so that their latency passes behind those instructions (the
            // scheduling fences keep the compiler from moving the requests back next to their use)
            Half8Words ahi[2], alo[2];
            ahi[0].q = a16_lds[lane];
            alo[0].q = a16_lds[(MB * KB) * 64 + lane];
            // ... and the rows' projections for k-block kb + 1 before the last step of k-block kb
            float4 pn[NR][2];
#pragma unroll
            for (int x = 0; x < NR; ++x) {
                pn[x][0] = *(const float4 *)(pon_lds + (r + x) * H + hh * KS);
                pn[x][1] = *(const float4 *)(pon_lds + (r + x) * H + hh * KS + 4);
            }
#pragma unroll
            for (int kb = 0; kb < KB; ++kb) {
                Half8Words bhi[NR], blo[NR];
#pragma unroll
                for (int x = 0; x < NR; ++x) pieces(kb, x, pn[x][0], pn[x][1], bhi[x], blo[x]);
#pragma unroll
                for (int mb = 0; mb < MB; ++mb) {
                    const int step = kb * MB + mb, cur = step & 1, nxt = cur ^ 1;
                    if (step + 1 < KB * MB) {
                        const int kb1 = (step + 1) / MB, mb1 = (step + 1) % MB;
                        ahi[nxt].q = a16_lds[(mb1 * KB + kb1) * 64 + lane];
                        alo[nxt].q = a16_lds[((MB + mb1) * KB + kb1) * 64 + lane];
                        if (mb == MB - 1) {
#pragma unroll
                            for (int x = 0; x < NR; ++x) {
                                pn[x][0] = *(const float4 *)(pon_lds + (r + x) * H + hh * KS + 8 * (kb + 1));
                                pn[x][1] = *(const float4 *)(pon_lds + (r + x) * H + hh * KS + 8 * (kb + 1) + 4);
                            }
                        }
                    }
                    __builtin_amdgcn_sched_barrier(0);
                    // hi x hi, then the two cross terms; consecutive instructions alternate between the rows' accumulators
                    floatx16 bias;
                    if (kb == 0) bias = bias_of(mb);
#pragma unroll
                    for (int x = 0; x < NR; ++x)
                        acc[x][mb] = __builtin_amdgcn_mfma_f32_32x32x16_f16(ahi[cur].v, bhi[x].v, kb == 0 ? bias : acc[x][mb], 0, 0, 0);
#pragma unroll
                    for (int x = 0; x < NR; ++x)
                        acc[x][mb] = __builtin_amdgcn_mfma_f32_32x32x16_f16(ahi[cur].v, blo[x].v, acc[x][mb], 0, 0, 0);
#pragma unroll
                    for (int x = 0; x < NR; ++x)
                        acc[x][mb] = __builtin_amdgcn_mfma_f32_32x32x16_f16(alo[cur].v, bhi[x].v, acc[x][mb], 0, 0, 0);
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
        } else {
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) {
            const floatx16 bias = bias_of(mb);
#pragma unroll
            for (int x = 0; x < NR; ++x) acc[x][mb] = bias;
        }
        // operands of step q + 1 are fetched from LDS before the matrix instructions of step q are
        // issued, so that their latency hides behind those instead of in front of the next ones
        float4 av[2][MB], pv[2][NR];
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) av[0][mb] = a_lds[(mb * Q) * 64 + lane];
#pragma unroll
        for (int x = 0; x < NR; ++x) pv[0][x] = *(const float4 *)(pon_lds + (r + x) * H + hh * KS);
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            const int cur = q & 1, nxt = cur ^ 1;
            if (q + 1 < Q) {
#pragma unroll
                for (int mb = 0; mb < MB; ++mb) av[nxt][mb] = a_lds[(mb * Q + q + 1) * 64 + lane];
#pragma unroll
                for (int x = 0; x < NR; ++x)
                    pv[nxt][x] = *(const float4 *)(pon_lds + (r + x) * H + hh * KS + 4 * (q + 1));
            }
            float h1[NR][4];
#pragma unroll
            for (int x = 0; x < NR; ++x) {
                const float4 pq = pv[cur][x];
                if (PAIR_SM) {
                    const float4 ws = *(const float4 *)(wsm_lds + hh * KS + 4 * q);
                    h1[x][0] = fmaxf(fmaf(ws.x, share[x], pq.x + poff[4 * q]), 0.0f);
                    h1[x][1] = fmaxf(fmaf(ws.y, share[x], pq.y + poff[4 * q + 1]), 0.0f);
                    h1[x][2] = fmaxf(fmaf(ws.z, share[x], pq.z + poff[4 * q + 2]), 0.0f);
                    h1[x][3] = fmaxf(fmaf(ws.w, share[x], pq.w + poff[4 * q + 3]), 0.0f);
                } else {
                    h1[x][0] = fmaxf(pq.x + poff[4 * q], 0.0f);
                    h1[x][1] = fmaxf(pq.y + poff[4 * q + 1], 0.0f);
                    h1[x][2] = fmaxf(pq.z + poff[4 * q + 2], 0.0f);
                    h1[x][3] = fmaxf(pq.w + poff[4 * q + 3], 0.0f);
                }
            }
            // consecutive matrix instructions go to different accumulators: none waits for the one before
#pragma unroll
            for (int mb = 0; mb < MB; ++mb)
#pragma unroll
                for (int x = 0; x < NR; ++x)
                    acc[x][mb] = __builtin_amdgcn_mfma_f32_32x32x2f32(av[cur][mb].x, h1[x][0], acc[x][mb], 0, 0, 0);
#pragma unroll
            for (int mb = 0; mb < MB; ++mb)
#pragma unroll
                for (int x = 0; x < NR; ++x)
                    acc[x][mb] = __builtin_amdgcn_mfma_f32_32x32x2f32(av[cur][mb].y, h1[x][1], acc[x][mb], 0, 0, 0);
#pragma unroll
            for (int mb = 0; mb < MB; ++mb)
#pragma unroll
                for (int x = 0; x < NR; ++x)
                    acc[x][mb] = __builtin_amdgcn_mfma_f32_32x32x2f32(av[cur][mb].z, h1[x][2], acc[x][mb], 0, 0, 0);
#pragma unroll
            for (int mb = 0; mb < MB; ++mb)
#pragma unroll
                for (int x = 0; x < NR; ++x)
                    acc[x][mb] = __builtin_amdgcn_mfma_f32_32x32x2f32(av[cur][mb].w, h1[x][3], acc[x][mb], 0, 0, 0);
        }
        }
        // max(v, 0) as the median of (v, 0, +inf): one instruction.  fmaxf costs two on values that
        // come out of the matrix pipe, because the compiler first has to make sure of a quiet NaN
        // (same result: the median of a NaN, 0 and +inf is 0 as well).
        // The +inf is hidden from the optimiser (an empty asm, no instruction), or it would turn the
        // median back into fmaxf.
        float plus_inf = __builtin_inff();
        asm volatile("" : "+s"(plus_inf));
        auto relu = [plus_inf](const float v) { return __builtin_amdgcn_fmed3f(v, 0.0f, plus_inf); };
        // output layer on this lane's 16*MB hidden units
        float zp[NR], sp[NR];
#pragma unroll
        for (int x = 0; x < NR; ++x) zp[x] = sp[x] = 0.0f;
#pragma unroll
        for (int mb = 0; mb < MB; ++mb)
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                const float4 wv = *(const float4 *)(w3_lds + mb * 32 + 8 * g + 4 * hh);
                const float4 sv = SLOWDOWN ? *(const float4 *)(w3s_lds + mb * 32 + 8 * g + 4 * hh) : wv;
                const float w[4] = {wv.x, wv.y, wv.z, wv.w}, ws[4] = {sv.x, sv.y, sv.z, sv.w};
#pragma unroll
                for (int e = 0; e < 4; ++e)
#pragma unroll
                    for (int x = 0; x < NR; ++x) {
                        const float h2 = relu(acc[x][mb][4 * g + e]);
                        zp[x] = fmaf(w[e], h2, zp[x]);
                        if (SLOWDOWN) sp[x] = fmaf(ws[e], h2, sp[x]);
                    }
            }
        // ... plus the other half-wave's.  Of two rows the lower half-wave takes the first one's sum and the upper
        // half-wave the second one's, and either goes on with its own row: one logistic for both rows
        auto both_halves = [](const float *p) {
            if constexpr (NR == 2) {
                const auto swapped = __builtin_amdgcn_permlane32_swap(__float_as_uint(p[0]), __float_as_uint(p[1]), false, false);
                return __uint_as_float(swapped[0]) + __uint_as_float(swapped[1]);
            } else {
                return p[0] + __shfl_xor(p[0], 32);
            }
        };
        const int mine = NR == 2 ? r + hh : r;
        const float z = both_halves(zp) + bias3;
        const float sg = 1.0f / (1.0f + expf(-z));
        bool too_slow = false;
        if (SLOWDOWN) {
            const float zs = both_halves(sp) + bias3_slow;
            too_slow = 1.0f / (1.0f + expf(-zs)) > slow_limit;
        }
        if ((NR == 2 || hh == 0) && j < m) {
            float qv = rintf(sg * scale);
            qv = fminf(fmaxf(qv, 0.0f), scale);
            int32_t w = (int32_t)qv;
            const float memsum = mon_lds[mine] + moff;
            if (memsum > mem_limit || too_slow) w = MF_INFEASIBLE;
            if (by_memory) {
                // the staged matrix: rows and columns both in memory order, a whole line per half-wave
                W[(size_t)(staged_row0 + row0 + mine) * ldw + j] = w;
            } else {
                // (looked up here, not above: a load still in flight at the end of a row makes
                // the next row wait for it and for every store issued after it)
                const int i = row_map ? row_map[row0 + mine] : row0 + mine;
                W[(size_t)i * ldw + jc] = w;
                if (sigma) sigma[(size_t)i * m + jc] = sg;
            }
        }
    };

    const int chunks = (n + task_rows - 1) / task_rows;
    const auto take = [&]() {
        int taken = 0;
        if (lane == 0) taken = atomicAdd(next, 1);
        return pair_task_taken(queue, __builtin_amdgcn_readfirstlane(taken), first, S::WAVES);
    };
    int task = !LONG || (int)blockIdx.x < first ? pair_task_by_place(blockIdx.x, wave, first) : take();
    int chunk = 0, before = 0;              // (before: tasks of earlier chunks)
    unsigned long long scored = 0;
    const bool turns = LONG && pair_takes_turns(blockIdx.x, first, later);
    int left = turns ? max(PAIR_STAY_ROWS / task_rows, 1) : INT_MAX;       // tasks until it leaves
    unsigned begun = LONG ? (unsigned)device_time() : 0u, longest = 0;     // of its tasks, in ticks
    bool none = false;
    for (;; task = take()) {
        int block;
        if (by_memory) {
            // a chunk of rows has as many tasks as blocks of columns fit its first row: a prefix of them
            int had = 0;
            unsigned long long beyond = 0;
            for (; chunk < chunks; chunk += 64, before += had) {
                const int c = chunk + lane;
                const int mine = c < chunks ? (fit_len[staged_row0 + c * task_rows] + 31) >> 5 : 0;
                int upto = mine;
#pragma unroll
                for (int off = 1; off < 64; off <<= 1) { const int o = __shfl_up(upto, off); if (lane >= off) upto += o; }
                beyond = __ballot(before + upto > task);
                if (beyond) {
                    const int at = __builtin_ctzll(beyond);
                    before += __builtin_amdgcn_readfirstlane(__shfl(upto - mine, at));
                    chunk += at;
                    break;
                }
                had = __builtin_amdgcn_readfirstlane(__shfl(upto, 63));
            }
            if (!beyond) { none = true; break; }
            block = task - before;
        } else {
            if (task >= chunks * blocks) { none = true; break; }
            chunk = task / blocks;
            block = task % blocks;
        }
        row0 = chunk * task_rows;
        const int j0 = block * 32, rows = min(task_rows, n - row0);
        j = j0 + nn;
        jc = col_map ? col_map[min(j, m - 1)] : min(j, m - 1);             // the column this lane scores
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            float4 t = *(const float4 *)(P_off + (size_t)jc * H + hh * KS + q * 4);
            poff[4 * q] = t.x * scale_p; poff[4 * q + 1] = t.y * scale_p; poff[4 * q + 2] = t.z * scale_p; poff[4 * q + 3] = t.w * scale_p;
        }
        moff = mem_off[jc];
        soff = PAIR_SM ? sm_off[jc] : 0.0f;
        // by_memory: the maps list rows and columns by ascending memory fraction, so this
        // wavefront's first column has its smallest one, and once a row does not fit next to
        // that column (float addition is monotone) no later row of the chunk fits any of its columns
        const float moff_least = by_memory ? __uint_as_float(__builtin_amdgcn_readfirstlane(__float_as_uint(moff))) : 0.0f;
        int done = 0;
        while (done < rows) {
            const int here = min(ROWS, rows - done);
            // LDS instructions of one wavefront are carried out in order; the compiler has to keep them so
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            for (int idx = lane; idx < here * (H / 4); idx += 64) {
                const int at = row0 + idx / (H / 4), gi = row_map ? row_map[at] : at;
                float4 v = ((const float4 *)(P_on + (size_t)gi * H))[idx % (H / 4)];
                if (SPLIT) { v.x *= scale_p; v.y *= scale_p; v.z *= scale_p; v.w *= scale_p; }
                ((float4 *)pon_lds)[idx] = v;
            }
            bool out = true;
            if (lane < here) {
                const int gi = row_map ? row_map[row0 + lane] : row0 + lane;
                const float mon = mem_on[gi];
                mon_lds[lane] = mon;
                if (PAIR_SM) son_lds[lane] = 1.0f - sm_on[gi];
                out = by_memory && mon + moff_least > mem_limit;
            }
            const int fit = __builtin_ctzll(__ballot(out));                // (lanes from ROWS on are out)
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            for (int r = 0; r < fit;) {
                // W2 does not fit in registers next to the accumulators: keep its loads inside the row loop
                asm volatile("" ::: "memory");
                if (r + 1 < fit) { score_rows(std::integral_constant<int, 2>{}, std::integral_constant<bool, SPLIT>{}, r); r += 2; }
                else { score_rows(std::integral_constant<int, 1>{}, std::integral_constant<bool, SPLIT>{}, r); r += 1; }
            }
            done += fit;
            row0 += fit;
            if (fit < here) break;          // (what rows left out have here lies beyond their feasible prefixes and is never read)
        }
        scored += (unsigned long long)done * (unsigned)min(32, m - j0);
        if (LONG && (--left == 0 || __builtin_amdgcn_readfirstlane(*(volatile int *)leave_lds))) break;
        if (LONG && !turns && (int)blockIdx.x < first) {
            const int later_begun = __builtin_amdgcn_readfirstlane(__hip_atomic_load(next + 2, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
            const unsigned last = (unsigned)__builtin_amdgcn_readfirstlane(__hip_atomic_load(next + 3, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
            const unsigned now = (unsigned)device_time();
            longest = max(longest, now - begun);
            begun = now;
            if (pair_may_leave(blockIdx.x, first, later, later_begun) && (int)(now - last) > 0 && now - last > PAIR_PATIENCE * longest) {
                *(volatile int *)leave_lds = 1;
                break;
            }
        }
    }
    if (lane == 0) {                        // the workgroup's last wavefront adds for all
        if (LONG && none) __hip_atomic_store(next + 1, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        atomicAdd(scored_lds, scored);
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");
        if (atomicAdd(ended_lds, 1) == S::WAVES - 1) atomicAdd(evaluated, atomicAdd(scored_lds, 0ull));
    }
}

template <int H, bool PAIR_SM, bool SLOWDOWN, bool SPLIT>
int launch_pair_variant(mf_ctx *ctx, const mf_predictor *p, int n, int m, int32_t *d_W, int64_t ldw,
                        float *d_sigma, const int32_t *row_map, const int32_t *col_map, bool by_memory,
                        const int32_t *segment, int grid_rows, int launch, unsigned long long *times)
{
    using S = PairShape<H>;
    // (the attribute belongs to the device, so what has been set is remembered per context)
    const unsigned flag = 1u << (5 + (H == 128 ? 8 : 0) + (PAIR_SM ? 4 : 0) + (SLOWDOWN ? 2 : 0) + (SPLIT ? 1 : 0));
    if (!(ctx->kernels_configured & flag)) {
        for (const auto kernel : {pair_mlp_kernel<H, PAIR_SM, SLOWDOWN, SPLIT, false>, pair_mlp_kernel<H, PAIR_SM, SLOWDOWN, SPLIT, true>})
            MF_HIP(hipFuncSetAttribute((const void *)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)S::LDS_BYTES));
        ctx->kernels_configured |= flag;
    }
    const int blocks = (m + 31) / 32, units = ctx->n_cus > 0 ? ctx->n_cus : 1;
    // No more workgroups a compute unit than its wavefronts have tasks: each sets itself up, and three in one unit at once take
    // longer (H = 64: 200 x 400 three to a unit 20 us, one 15; 500 x 1000 30 / 27 with two).
    // (In memory order the kernel finds that there is less to do than this, and takes fewer rows a task.)
    const int task_rows = pair_task_rows(H, (float)grid_rows * (float)blocks, (float)units);
    const long long tasks = (long long)((grid_rows + task_rows - 1) / task_rows) * blocks, waves = (long long)units * S::WAVES;
    const long long most = units * (tasks > waves * S::PER_UNIT ? S::PER_UNIT : (tasks + waves - 1) / waves);
    const int first = (int)(tasks < most ? tasks : most);
    // What turns cost, in code and registers, short passes do not pay: 1 us of 23 to 33 for 64 x 64 to 200 x 400 pairs with every option.
    const long long later = pair_later(tasks, waves * S::PER_UNIT, S::WAVES, grid_rows, blocks, first);
    hipLaunchKernelGGL((later ? pair_mlp_kernel<H, PAIR_SM, SLOWDOWN, SPLIT, true> : pair_mlp_kernel<H, PAIR_SM, SLOWDOWN, SPLIT, false>),
                       dim3((unsigned)(first + later)), dim3(S::THREADS), S::LDS_BYTES, ctx->stream,
                       ctx->proj_on, ctx->proj_off, p->d_W2, p->d_b2, p->d_W3, p->d_b3,
                       ctx->mem_on, ctx->mem_off, n, m, p->scale, p->mem_limit, d_W, ldw, d_sigma, row_map, col_map,
                       by_memory ? 1 : 0, ctx->pairs_evaluated, segment, p->d_W1sm, ctx->sm_on, ctx->sm_off,
                       p->d_W3_slow, p->d_b3_slow, p->slow_limit, SPLIT ? ctx->score_range : nullptr, (float)units,
                       by_memory ? ctx->feasible_pairs : nullptr, by_memory ? ctx->fit_len_on : nullptr, ctx->score_queue + launch * MF_PAIR_QUEUES * MF_PAIR_QUEUE_STEP, first, times);
    MF_HIP(hipGetLastError());
    return MF_OK;
}

template <int H>
int launch_pair(mf_ctx *ctx, const mf_predictor *p, int n, int m, int32_t *d_W, int64_t ldw,
                float *d_sigma, const int32_t *row_map, const int32_t *col_map, bool by_memory,
                unsigned long long *times, int launch, const int32_t *segment = nullptr, int segment_rows = -1)
{
    const int grid_rows = segment_rows >= 0 ? segment_rows : n;
    const int which = (p->d_W1sm ? 4 : 0) + (p->d_W3_slow ? 2 : 0) + (ctx->score_split ? 1 : 0);
#define MF_PAIR_CASE(SM, SLOW, SPL) \
    return launch_pair_variant<H, SM, SLOW, SPL>(ctx, p, n, m, d_W, ldw, d_sigma, row_map, col_map, by_memory, segment, grid_rows, launch, times)
    switch (which) {
    case 0: MF_PAIR_CASE(false, false, false);
    case 1: MF_PAIR_CASE(false, false, true);
    case 2: MF_PAIR_CASE(false, true, false);
    case 3: MF_PAIR_CASE(false, true, true);
    case 4: MF_PAIR_CASE(true, false, false);
    case 5: MF_PAIR_CASE(true, false, true);
    case 6: MF_PAIR_CASE(true, true, false);
    default: MF_PAIR_CASE(true, true, true);
    }
#undef MF_PAIR_CASE
}

// Layer 1 of everybody, and what the fp16 pieces of the hidden layer are scaled by (slots zero on entry).
void launch_projections(mf_ctx *ctx, const mf_predictor *p, const float *d_on, int n, const float *d_off, int m)
{
    ProjectArgs a{};
    a.X[0] = d_on; a.X[1] = d_off;
    a.rows[0] = n; a.rows[1] = m;
    a.P[0] = ctx->proj_on; a.P[1] = ctx->proj_off;
    a.W1 = p->d_W1; a.b1 = p->d_b1;
    a.F = p->F; a.H = p->H;
    a.range_of[0] = p->d_W2; a.range_count[0] = p->H * p->H;
    a.range_of[1] = p->d_W1sm; a.range_count[1] = p->H;
    a.range_of[2] = p->d_W1sm ? ctx->sm_off : nullptr; a.range_count[2] = m;
    a.range = ctx->score_split ? ctx->score_range : nullptr;
    const int tiles = (n + PROJECT_ROWS - 1) / PROJECT_ROWS + (m + PROJECT_ROWS - 1) / PROJECT_ROWS;
    hipLaunchKernelGGL(project_kernel, dim3(tiles + PROJECT_EXTRA, p->H / 64), dim3(256), 0, ctx->stream, a);
}

SetupArgs setup_args(mf_ctx *ctx, const mf_predictor *p, const float *d_on, int n, const float *d_off, int m, int launches)
{
    SetupArgs a{};
    a.X[0] = d_on; a.X[1] = d_off;
    a.rows[0] = n; a.rows[1] = m;
    a.F = p->F; a.mem_feature = p->mem_feature;
    a.sm_feature[0] = p->d_W1sm ? p->sm_on_feature : -1;
    a.sm_feature[1] = p->d_W1sm ? p->sm_off_feature : -1;
    a.mem[0] = ctx->mem_on; a.mem[1] = ctx->mem_off;
    a.sm[0] = ctx->sm_on; a.sm[1] = ctx->sm_off;
    a.mem_limit = p->mem_limit;
    a.pairs_evaluated = ctx->pairs_evaluated;
    a.range = ctx->score_range;
    a.queue = ctx->score_queue; a.launches = launches;
    a.times = ctx->times;
    return a;
}

// segment[t] = number of workloads whose type is below t (t = 0..n_types); *bad is raised for
// a type outside [0, n_types).  One workgroup: the type counts are a few dozen integers.
__global__ __launch_bounds__(1024) void type_segments_kernel(const int32_t *__restrict__ type, int count,
                                                             int n_types, int32_t *__restrict__ segment, int *bad)
{
    __shared__ int hist[MF_MAX_TYPES];
    for (int t = threadIdx.x; t < MF_MAX_TYPES; t += blockDim.x) hist[t] = 0;
    __syncthreads();
    for (int i = threadIdx.x; i < count; i += blockDim.x) {
        const int t = type[i];
        if (t < 0 || t >= n_types) atomicExch(bad, 1);
        else atomicAdd(&hist[t], 1);
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        int run = 0;
        for (int t = 0; t <= n_types; ++t) { segment[t] = run; if (t < n_types) run += hist[t]; }
    }
}

}  // namespace

// preds[0..n_types): with d_type == nullptr there is one predictor for everybody; otherwise
// online workload i is scored by preds[d_type[i]] (all of them agree on F, the memory feature,
// the memory limit and the scale; the hidden width may differ).  Per type: project everybody
// with that type's first layer, then run the pair kernel on that type's rows - a contiguous
// segment of the row map, which lists the online workloads by (type, memory fraction).
int mf_launch_score(mf_ctx *ctx, const mf_predictor *preds, int n_types, const int32_t *d_type,
                    const float *d_on, int n, const float *d_off, int m, int32_t *d_W, int64_t ldw,
                    float *d_sigma, bool as_it_comes)
{
    const mf_predictor *p0 = &preds[0];
    const bool typed = d_type != nullptr;
    if (typed) {
        hipLaunchKernelGGL(fill_flag_kernel, dim3(1), dim3(1), 0, ctx->stream, ctx->colmark);
        hipLaunchKernelGGL(type_segments_kernel, dim3(1), dim3(1024), 0, ctx->stream, d_type, n, n_types,
                           ctx->type_segment, ctx->colmark);
        MF_HIP(hipGetLastError());
        // the host sizes each type's launch by its number of rows
        const int rc = mf_send_and_await(ctx, mf_report{{{ctx->colmark, ctx->h_bad, 1}, {ctx->type_segment, ctx->h_type_first, n_types + 1}}});
        if (rc != MF_OK) return rc;
        if (*ctx->h_bad) return MF_ERR_ARG;
    }
    const int32_t *type_first = ctx->h_type_first;
    // Pairs whose memory fractions do not fit get no score, so unless the caller wants every
    // score, walk rows and columns in memory order: the pairs that cannot fit then form one
    // corner of the tile grid and the kernel leaves them out.  Results land at the same places.
    // (as_it_comes: a problem so small that the four launches which find the order and undo it take longer than
    // the pairs: a 64 x 64 round 241 / 218 us)
    const bool by_memory = ctx->fit_order && !d_sigma && !as_it_comes;
    const int64_t lds = ((int64_t)m + 3) & ~3ll;
    // (each of these is a few microseconds of work: as eight launches, not twenty-two, the set-up of a
    // 64 x 64 round takes 31 us, not 310)
    SetupArgs a = setup_args(ctx, p0, d_on, n, d_off, m, n_types);
    a.largest = ctx->largest_weight;
    ctx->largest_weight_known = false;
    a.group = d_type;
    if (by_memory || typed) { a.rank[0] = ctx->rank_on; a.order[0] = ctx->order_on; }
    if (by_memory) {
        a.rank[1] = ctx->rank_off; a.order[1] = ctx->order_off;
        a.sorted[0] = ctx->mem_on_sorted; a.sorted[1] = ctx->mem_off_sorted;
        a.fit_len[0] = ctx->fit_len_on; a.fit_len[1] = ctx->fit_len_off;
        a.feasible_pairs = ctx->feasible_pairs;
        a.staged = ctx->staged;
        a.pitch = lds;
    }
    const int most = n > m ? n : m, blocks = (most + 255) / 256;
    hipLaunchKernelGGL(setup_kernel, dim3(blocks, 2), dim3(256), 0, ctx->stream, a);
    if ((by_memory || typed) && most >= SORT_FROM) {
        a.keys[0] = ctx->path_label; a.keys[1] = ctx->path_expanded;       // (of the matching, which has not begun)
        const int stretches = (most + SORT_TILE - 1) / SORT_TILE;
        hipLaunchKernelGGL(rank_sort_kernel, dim3(stretches, 1, 2), dim3(SORT_THREADS), 0, ctx->stream, a);
        hipLaunchKernelGGL(rank_merge_kernel, dim3(blocks, (stretches + SORT_STRETCHES - 1) / SORT_STRETCHES, 2), dim3(256), 0, ctx->stream, a);
        hipLaunchKernelGGL(order_kernel, dim3(blocks, 2), dim3(256), 0, ctx->stream, a);
    } else if (by_memory || typed) {
        int slices = 0;
        for (int side = 0; side < 2; ++side) {
            const int count = a.rows[side];
            int split = 2048 / ((count + RANK_THREADS - 1) / RANK_THREADS);
            split = split < 1 ? 1 : (split > 64 ? 64 : split);
            a.slice[side] = ((count + split - 1) / split + 3) & ~3;
            const int mine = (count + a.slice[side] - 1) / a.slice[side];
            if (a.rank[side] && mine > slices) slices = mine;
        }
        hipLaunchKernelGGL(rank_count_kernel, dim3((most + RANK_THREADS - 1) / RANK_THREADS, slices, 2), dim3(RANK_THREADS), 0,
                           ctx->stream, a);
        hipLaunchKernelGGL(order_kernel, dim3(blocks, 2), dim3(256), 0, ctx->stream, a);
    }
    ctx->staged_n = ctx->staged_m = 0;
    if (by_memory) {
        // feasibility is a prefix of every staged row (columns are in memory order) and, when the
        // rows are in memory order too - one predictor - of every staged column; with several
        // predictors the rows are ordered by type first and columns are read whole
        hipLaunchKernelGGL(fit_prefix_kernel, dim3(blocks, 2), dim3(256), 0, ctx->stream, a);
        ctx->staged_n = n;
        ctx->staged_m = m;
    }
    MF_HIP(hipGetLastError());
    ctx->pairs_total = (double)n * (double)m;
    const int32_t *rmap = (by_memory || typed) ? ctx->order_on : nullptr, *cmap = by_memory ? ctx->order_off : nullptr;
    // in memory order the scores go to the staged matrix
    int32_t *out = by_memory ? ctx->staged : d_W;
    const int64_t ldo = by_memory ? lds : ldw;
    unsigned long long *times = ctx->times;
    for (int t = 0; t < n_types; ++t) {
        const mf_predictor *p = &preds[t];
        const int H = p->H;
        if (t > 0) hipLaunchKernelGGL(range_clear_kernel, dim3(1), dim3(64), 0, ctx->stream, ctx->score_range);
        launch_projections(ctx, p, d_on, n, d_off, m);
        MF_HIP(hipGetLastError());
        const int32_t *segment = typed ? ctx->type_segment + t : nullptr;
        const int segment_rows = typed ? type_first[t + 1] - type_first[t] : -1;
        if (segment_rows == 0) continue;                                   // no workload of this type
        int rc = (H == 64) ? launch_pair<64>(ctx, p, n, m, out, ldo, d_sigma, rmap, cmap, by_memory, times, t, segment, segment_rows)
                           : launch_pair<128>(ctx, p, n, m, out, ldo, d_sigma, rmap, cmap, by_memory, times, t, segment, segment_rows);
        times = nullptr;                                                   // (later types' projections count as scoring)
        if (rc != MF_OK) return rc;
    }
    if (by_memory) {
        const int chunks = (m + 4095) / 4096 < 16 ? (m + 4095) / 4096 : 16;
        // 0: entry by entry; 1: by fours; 2: by fours and, with LDS, past the caches, for a matrix that does not stay in the last one until
        // it is read (256 MB): 20,000 x 40,000 0.05 ms less, 20,000 x 20,000 0.02
        int wide = ((uintptr_t)d_W & 15u) == 0 && (ldw & 3) == 0;
        if (wide && (int64_t)n * ldw * 4 > (256ll << 20)) wide = 2;
        if (place_by_lds(n, lds)) {
            hipLaunchKernelGGL(place_lds_kernel, dim3(n), dim3(PLACE_THREADS), 0, ctx->stream,
                               ctx->staged, lds, ctx->rank_on, ctx->rank_off, ctx->fit_len_on, n, m, d_W, ldw, wide,
                               ctx->largest_weight, ctx->times);
        } else {
            hipLaunchKernelGGL(place_kernel, dim3(n, chunks), dim3(256), 0, ctx->stream, ctx->staged, lds,
                               ctx->rank_on, ctx->rank_off, ctx->fit_len_on, n, m, d_W, ldw, wide, ctx->largest_weight, ctx->times);
        }
        MF_HIP(hipGetLastError());
        ctx->largest_weight_known = true;
    }
    ctx->score_placed = by_memory;
    ctx->score_pending = true;
    return MF_OK;
}

namespace {

__global__ void check_indices_kernel(const int32_t *__restrict__ list, int count, int limit, int *bad)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < count && (list[i] < 0 || list[i] >= limit)) atomicExch(bad, 1);
}

}  // namespace

// Re-scores, in place, the rows of the listed online workloads and the columns
// of the listed offline workloads (device index lists).  Projections are
// recomputed for everybody (they cost 2(n+m)FH flop); the pair kernel then runs
// on `n_rows x m` and `n x n_cols` through its index maps.
int mf_launch_rescore(mf_ctx *ctx, const mf_predictor *p, const float *d_on, int n, const float *d_off,
                      int m, int32_t *d_W, int64_t ldw, const int32_t *d_rows, int n_rows,
                      const int32_t *d_cols, int n_cols)
{
    const int H = p->H;
    ctx->staged_n = ctx->staged_m = 0;       // the staged copy no longer matches the matrix
    ctx->largest_weight_known = false;
    // the lists index device arrays: refuse anything out of range before a kernel trusts it
    hipLaunchKernelGGL(fill_flag_kernel, dim3(1), dim3(1), 0, ctx->stream, ctx->colmark);
    if (n_rows > 0)
        hipLaunchKernelGGL(check_indices_kernel, dim3((n_rows + 255) / 256), dim3(256), 0, ctx->stream, d_rows,
                           n_rows, n, ctx->colmark);
    if (n_cols > 0)
        hipLaunchKernelGGL(check_indices_kernel, dim3((n_cols + 255) / 256), dim3(256), 0, ctx->stream, d_cols,
                           n_cols, m, ctx->colmark);
    MF_HIP(hipGetLastError());
    int rc = mf_send_and_await(ctx, mf_report{{{ctx->colmark, ctx->h_bad, 1}}});
    if (rc != MF_OK) return rc;
    if (*ctx->h_bad) return MF_ERR_ARG;
    const SetupArgs a = setup_args(ctx, p, d_on, n, d_off, m, 2);
    hipLaunchKernelGGL(setup_kernel, dim3(((n > m ? n : m) + 255) / 256, 2), dim3(256), 0, ctx->stream, a);
    launch_projections(ctx, p, d_on, n, d_off, m);          // of everybody, and so the range, as in a full scoring pass
    MF_HIP(hipGetLastError());
    ctx->pairs_total = (double)n_rows * (double)m + (double)n * (double)n_cols;
    if (n_rows == 0 && n_cols == 0) mf_note_time(ctx, AT_PAIRS);
    if (n_rows > 0)
        rc = (H == 64) ? launch_pair<64>(ctx, p, n_rows, m, d_W, ldw, nullptr, d_rows, nullptr, false, ctx->times, 0)
                       : launch_pair<128>(ctx, p, n_rows, m, d_W, ldw, nullptr, d_rows, nullptr, false, ctx->times, 0);
    if (rc == MF_OK && n_cols > 0)
        rc = (H == 64) ? launch_pair<64>(ctx, p, n, n_cols, d_W, ldw, nullptr, nullptr, d_cols, false, n_rows > 0 ? nullptr : ctx->times, 1)
                       : launch_pair<128>(ctx, p, n, n_cols, d_W, ldw, nullptr, nullptr, d_cols, false, n_rows > 0 ? nullptr : ctx->times, 1);
    if (rc != MF_OK) return rc;
    ctx->score_placed = false;
    ctx->score_pending = true;
    return MF_OK;
}
