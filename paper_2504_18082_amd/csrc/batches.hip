// Root node partitioning (Algorithm 1 Step-1; Section 4.1; Table 1): the epoch's permutation of the
// training set under NORAND-ROOTS, COMM-RAND-MIX and RAND-ROOTS.  Every shuffle is a sort by a Philox key,
// equal keys keep the smaller id first, so the result does not depend on scheduling.
//
// The keys are uniform random numbers, so an element's place is known to within a few positions before anything is
// sorted: with `count` elements in its super-block, which starts at `first`, it belongs near
//     p = first + (upper key word * count) >> 32,
// and p ascends with (super-block, key).  A shuffle is therefore ONE distribution pass into buckets of equal stretches
// of p and a sort of every bucket in LDS (about 512 elements into 512 bins, one each on average), instead of a
// radix pass per key byte: 1.22 M training nodes in 100 000 communities (MIX-12.5 %) 2136 -> 125 us, the same
// nodes under RAND-ROOTS 1456 -> 49 us.
#include <mutex>

#include "cr_common.h"

namespace cr {

constexpr int MAX_BUCKETS = 4096;       // LDS counters of the distribution kernels (16 KB)
constexpr int MIN_SHIFT = 9;            // a bucket spans at least 512 positions: one per LDS bin of the bucket sort
constexpr int BIN_SHIFT = 10;           // ... and is sorted 1024 positions at a time
constexpr int SORT_CAP = 2048;          // elements of such a stretch that fit LDS (mean 1024, deviation 32)
constexpr int DIST_TILE = 4096;         // elements a distribution workgroup takes at least
constexpr int DIST_BLOCKS = 256;        // ... and the most such workgroups (one per compute unit)

// one shuffle: what is sorted and how it is cut
struct ShufflePlan {
    int n;                  // elements
    int shift;              // bucket = p >> shift
    int n_buckets;          // buckets the positions 0..n-1 fall into (<= MAX_BUCKETS)
    int n_tiles, tile;      // distribution workgroups and their elements
};

__host__ static ShufflePlan shuffle_plan(int n)
{
    ShufflePlan s;
    s.n = n;
    s.shift = MIN_SHIFT;
    while (((n - 1) >> s.shift) >= MAX_BUCKETS) ++s.shift;
    s.n_buckets = n > 0 ? ((n - 1) >> s.shift) + 1 : 1;
    const int64_t want = ceil_div(n, DIST_TILE);
    s.n_tiles = (int)(want < 1 ? 1 : (want > DIST_BLOCKS ? DIST_BLOCKS : want));
    s.tile = (int)ceil_div(n > 0 ? n : 1, s.n_tiles);
    return s;
}

// What is shuffled.  Nodes: element i is train[i], and its super-block's stretch of the permutation comes from its
// community (`stretch`, NULL: one super-block, RAND-ROOTS).  Communities: element i is community i, taking part when the
// training set has a node of it; *n_present of them do.
struct ShuffleArgs {
    const int32_t *train;
    const int32_t *node_comm;       // [n] community of train[i] (with `stretch`)
    const int2 *stretch;            // [n_comm] (first position, length) of the community's super-block
    const int32_t *present;         // [n_comm] training nodes of every community
    const int32_t *n_present;
    uint64_t seed;
    uint32_t epoch;
    ShufflePlan plan;
    uint32_t *pos;                  // [n] p of every element (ABSENT: takes no part)
    int32_t *counts;                // [n_tiles][n_buckets]
    int32_t *totals;                // [n_buckets]
    uint2 *pairs;                   // [n] (p, id), bucket by bucket
    int32_t *out;                   // [n] ids in order
};
constexpr uint32_t ABSENT = 0xFFFFFFFFu;

template <bool COMMUNITIES>
__device__ __forceinline__ uint64_t element_key(const ShuffleArgs &a, uint32_t id)
{
    return shuffle_key(a.seed, a.epoch, COMMUNITIES ? DOMAIN_COMMUNITY : DOMAIN_NODE, id);
}

// positions of a tile's elements, and how many fall into every bucket
template <bool COMMUNITIES>
__global__ __launch_bounds__(1024) void shuffle_count_kernel(ShuffleArgs a)
{
    __shared__ int cnt[MAX_BUCKETS];
    const ShufflePlan &pl = a.plan;
    for (int b = threadIdx.x; b < pl.n_buckets; b += 1024) cnt[b] = 0;
    __syncthreads();
    const int64_t start = (int64_t)blockIdx.x * pl.tile, stop = min((int64_t)pl.n, start + pl.tile);
    for (int64_t i = start + threadIdx.x; i < stop; i += 1024) {
        uint32_t p;
        if constexpr (COMMUNITIES) {
            const uint32_t hi = (uint32_t)(element_key<true>(a, (uint32_t)i) >> 32);
            p = a.present[i] > 0 ? __umulhi(hi, (uint32_t)*a.n_present) : ABSENT;
        } else {
            const int v = a.train[i];
            const uint32_t hi = (uint32_t)(element_key<false>(a, (uint32_t)v) >> 32);
            const int2 st = a.stretch ? a.stretch[a.node_comm[i]] : make_int2(0, pl.n);
            p = (uint32_t)st.x + __umulhi(hi, (uint32_t)st.y);
        }
        a.pos[i] = p;
        if (p != ABSENT) atomicAdd(&cnt[p >> pl.shift], 1);
    }
    __syncthreads();
    int32_t *row = a.counts + (int64_t)blockIdx.x * pl.n_buckets;
    for (int b = threadIdx.x; b < pl.n_buckets; b += 1024) row[b] = cnt[b];
}

// counts[tile][bucket] -> elements of the bucket in the tiles in front; totals[bucket].  A workgroup takes 64 buckets, its
// sixteen waves a sixteenth of the tiles each.
__global__ __launch_bounds__(1024) void shuffle_prefix_kernel(ShufflePlan pl, int32_t *counts, int32_t *totals)
{
    __shared__ int part[16][64];
    constexpr int PER = DIST_BLOCKS / 16;
    const int lane = lane_id(), wave = threadIdx.x / WAVE;
    const int b = blockIdx.x * 64 + lane;
    const bool have = b < pl.n_buckets;
    const int t0 = wave * PER;
    int x[PER], sum = 0;
#pragma unroll
    for (int k = 0; k < PER; ++k) x[k] = (have && t0 + k < pl.n_tiles) ? counts[(int64_t)(t0 + k) * pl.n_buckets + b] : 0;
#pragma unroll
    for (int k = 0; k < PER; ++k) sum += x[k];
    part[wave][lane] = sum;
    __syncthreads();
    int run = 0;
    for (int w = 0; w < wave; ++w) run += part[w][lane];
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        if (have && t0 + k < pl.n_tiles) counts[(int64_t)(t0 + k) * pl.n_buckets + b] = run;
        run += x[k];
    }
    if (have && wave == 15) totals[b] = run;
}

// (p, id) of a tile's elements into their buckets; the order inside a bucket does not matter, the bucket is sorted
__global__ __launch_bounds__(1024) void shuffle_scatter_kernel(ShuffleArgs a, int communities)
{
    __shared__ int cursor[MAX_BUCKETS];
    __shared__ int lds[17];
    constexpr int PER = MAX_BUCKETS / 1024;
    const ShufflePlan &pl = a.plan;
    const int32_t *row = a.counts + (int64_t)blockIdx.x * pl.n_buckets;
    const int b0 = (int)threadIdx.x * PER;
    int x[PER], y[PER], sum = 0;
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        x[k] = b0 + k < pl.n_buckets ? a.totals[b0 + k] : 0;
        y[k] = b0 + k < pl.n_buckets ? row[b0 + k] : 0;
        sum += x[k];
    }
    int total;
    int run = block_exclusive_scan_1024(sum, lds, total);
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        cursor[b0 + k] = run + y[k];
        run += x[k];
    }
    __syncthreads();
    const int64_t start = (int64_t)blockIdx.x * pl.tile, stop = min((int64_t)pl.n, start + pl.tile);
    for (int64_t i = start + threadIdx.x; i < stop; i += 1024) {
        const uint32_t p = a.pos[i];
        if (p == ABSENT) continue;
        a.pairs[atomicAdd(&cursor[p >> pl.shift], 1)] = make_uint2(p, (uint32_t)(communities ? i : a.train[i]));
    }
}

// Whether element (pa, ka, ia) comes before (pb, kb, ib).  Equal p does not mean equal key, but p ascends with the
// (super-block, key) pair, so p first and the key inside p is the same order.
__device__ __forceinline__ bool comes_before(uint32_t pa, uint64_t ka, uint32_t ia, uint32_t pb, uint64_t kb, uint32_t ib)
{
    return pa != pb ? pa < pb : (ka != kb ? ka < kb : ia < ib);
}

// A bucket per workgroup.  A stretch of 1024 positions of it (the whole bucket, unless there are more than 4 M elements)
// is counted into one bin per position, laid out bin by bin in LDS with the elements' full keys, and every element finds
// its rank among the one or two of its own bin.  A stretch that does not fit LDS -- which a uniform key does not produce,
// only ids that are given more than once -- sends the bucket through a merge network in memory instead.
template <bool COMMUNITIES>
__global__ __launch_bounds__(256) void shuffle_sort_kernel(ShuffleArgs a)
{
    __shared__ uint64_t keys[SORT_CAP];
    __shared__ uint32_t ids[SORT_CAP];
    __shared__ uint16_t bin_of[SORT_CAP];
    __shared__ int bin_end[1 << BIN_SHIFT];
    __shared__ int lds[17];
    const ShufflePlan &pl = a.plan;
    const int tid = threadIdx.x, bucket = blockIdx.x;
    // first element: the buckets in front, added up by the workgroup
    int before = 0, m;
    for (int b = tid; b < bucket; b += 256) before += a.totals[b];
    block_exclusive_scan<4>(before, lds, before);
    m = a.totals[bucket];
    uint2 *pairs = a.pairs + before;
    int32_t *out = a.out + before;
    const int n_bins = 1 << min(pl.shift, BIN_SHIFT);
    const int n_stretches = 1 << max(0, pl.shift - BIN_SHIFT);
    int done = 0;
    for (int st = 0; st < n_stretches && done < m; ++st) {
        const uint32_t tag = ((uint32_t)bucket << max(0, pl.shift - BIN_SHIFT)) + (uint32_t)st;      // p / 1024 (or the bucket)
        const int tag_shift = min(pl.shift, BIN_SHIFT);
        __syncthreads();
        for (int i = tid; i < n_bins; i += 256) bin_end[i] = 0;
        __syncthreads();
        for (int i = tid; i < m; i += 256) {
            const uint32_t p = pairs[i].x;
            if ((p >> tag_shift) == tag) atomicAdd(&bin_end[p & (n_bins - 1)], 1);
        }
        __syncthreads();
        // bin starts (a thread owns consecutive bins)
        constexpr int PER = (1 << BIN_SHIFT) / 256;
        int x[PER], sum = 0, total;
#pragma unroll
        for (int k = 0; k < PER; ++k) {
            x[k] = tid * PER + k < n_bins ? bin_end[tid * PER + k] : 0;
            sum += x[k];
        }
        int run = block_exclusive_scan<4>(sum, lds, total);
        if (total > SORT_CAP) break;                                   // (uniform)
#pragma unroll
        for (int k = 0; k < PER; ++k) {
            if (tid * PER + k < n_bins) bin_end[tid * PER + k] = run;  // advanced to the bin's end below
            run += x[k];
        }
        __syncthreads();
        for (int i = tid; i < m; i += 256) {
            const uint2 e = pairs[i];
            if ((e.x >> tag_shift) != tag) continue;
            const int bin = (int)(e.x & (n_bins - 1));
            const int at = atomicAdd(&bin_end[bin], 1);
            ids[at] = e.y;
            keys[at] = element_key<COMMUNITIES>(a, e.y);
            bin_of[at] = (uint16_t)bin;
        }
        __syncthreads();
        for (int i = tid; i < total; i += 256) {
            const int bin = bin_of[i];
            const int lo = bin > 0 ? bin_end[bin - 1] : 0, hi = bin_end[bin];
            const uint64_t k = keys[i];
            const uint32_t id = ids[i];
            int rank = lo;
            for (int j = lo; j < hi; ++j) rank += (keys[j] < k || (keys[j] == k && (ids[j] < id || (ids[j] == id && j < i)))) ? 1 : 0;
            out[done + rank] = (int32_t)id;
        }
        done += total;
    }
    if (done >= m) return;
    // merge network over the bucket's pairs in memory: every exchange moves the earlier element to the lower index, so
    // the places past m act as elements behind all others and are never touched
    __syncthreads();
    auto exchange = [&](int i, int j) {
        if (j >= m) return;
        const uint2 x = pairs[i], y = pairs[j];
        if (comes_before(y.x, element_key<COMMUNITIES>(a, y.y), y.y, x.x, element_key<COMMUNITIES>(a, x.y), x.y)) { pairs[i] = y; pairs[j] = x; }
    };
    for (int64_t size = 2; size < 2 * (int64_t)m; size *= 2) {
        const int half = (int)(size / 2);
        for (int i = tid; i < m; i += 256)
            if ((i & (size - 1)) < half) exchange(i, (int)min((int64_t)m, (i & ~(size - 1)) + size - 1 - (i & (size - 1))));
        __syncthreads();
        for (int d = half / 2; d > 0; d /= 2) {
            for (int i = tid; i < m; i += 256)
                if ((i & d) == 0) exchange(i, (int)min((int64_t)m, (int64_t)i + d));
            __syncthreads();
        }
    }
    for (int i = tid; i < m; i += 256) out[i] = (int32_t)pairs[i].y;
}

__global__ __launch_bounds__(256) void zero_i32_kernel(int32_t *p, int64_t n)
{
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) p[i] = 0;
}

// Training nodes per community, and how many communities have one (both zeroed before); the communities are kept for
// the distribution of the nodes, which needs them again.  Training nodes are thinly spread (1 % of the papers-like
// graph), so every look-up is a memory line of its own: 1.22 M of them are 156 MB and most of this kernel's 28 us,
// and what a second look-up would cost (the distribution's counting pass: 22.3 us with it, 8.0 with the kept ones).
// Training ids ascend and communities are stretches of ids in the graphs this is used on, so a wave takes consecutive
// ids, all of its look-ups in flight at once, and adds to a community's counter once per run of ids: adds to one
// address are served one after another (one add per 256 ids on *n_present alone made the kernel take 64 us).
constexpr int COUNT_CHUNKS = 8;         // chunks of 64 ids a wave takes in a row
__global__ __launch_bounds__(256) void count_communities_kernel(const int32_t *__restrict__ train, int n_train, const int32_t *__restrict__ comm,
                                                                int32_t *__restrict__ count, int32_t *__restrict__ n_present,
                                                                int32_t *__restrict__ node_comm)
{
    __shared__ int found;
    if (threadIdx.x == 0) found = 0;
    __syncthreads();
    const int lane = lane_id();
    const int64_t first = ((int64_t)blockIdx.x * 4 + threadIdx.x / WAVE) * (COUNT_CHUNKS * 64) + lane;
    int c[COUNT_CHUNKS];
#pragma unroll
    for (int k = 0; k < COUNT_CHUNKS; ++k) c[k] = train[min(first + k * 64, (int64_t)n_train - 1)];
#pragma unroll
    for (int k = 0; k < COUNT_CHUNKS; ++k) c[k] = comm[c[k]];
    int mine = 0, at = -1, held = 0;                     // community of the open run (the same in all lanes) and its ids so far
    auto add = [&](int community, int len) {
        if (atomicAdd(&count[community], len) == 0) ++mine;
    };
#pragma unroll
    for (int k = 0; k < COUNT_CHUNKS; ++k) {
        if (first + k * 64 < n_train) node_comm[first + k * 64] = c[k];
        else c[k] = -1;
        const int c0 = __builtin_amdgcn_readfirstlane(c[k]);
        if (c0 != at && held > 0) {
            if (lane == 0) add(at, held);
            held = 0;
        }
        at = c0;
        if (__ballot(c[k] != c0) == 0) {                 // one community throughout
            held = c0 >= 0 ? held + 64 : 0;
            continue;
        }
        const int left = __shfl_up(c[k], 1);
        const bool head = lane == 0 || left != c[k];
        const uint64_t after = __ballot(head) & (lane < 63 ? ~0ull << (lane + 1) : 0ull);
        const int len = (after ? __ffsll((unsigned long long)after) - 1 : 64) - lane;
        if (head && c[k] >= 0) add(c[k], len + (lane == 0 ? held : 0));
        at = -1;
        held = 0;
    }
    if (held > 0 && lane == 0) add(at, held);
    if (mine) atomicAdd(&found, mine);
    __syncthreads();
    if (threadIdx.x == 0 && found) atomicAdd(n_present, found);
}

// Training nodes of the communities of a bucket (their order is known by now), added up.
__global__ __launch_bounds__(256) void bucket_nodes_kernel(ShufflePlan pl, const int32_t *__restrict__ totals, const int32_t *__restrict__ order,
                                                           const int32_t *__restrict__ count, int32_t *__restrict__ nodes_of_bucket)
{
    __shared__ int lds[17];
    int before = 0, sum = 0;
    for (int b = threadIdx.x; b < (int)blockIdx.x; b += 256) before += totals[b];
    block_exclusive_scan<4>(before, lds, before);
    const int m = totals[blockIdx.x];
    for (int i = threadIdx.x; i < m; i += 256) sum += count[order[before + i]];
    __syncthreads();
    block_exclusive_scan<4>(sum, lds, sum);
    if (threadIdx.x == 0) nodes_of_bucket[blockIdx.x] = sum;
}

// nodes_before[r] = training nodes of the communities in front of rank r (one entry more than there are communities)
__global__ __launch_bounds__(256) void nodes_before_kernel(ShufflePlan pl, const int32_t *__restrict__ totals, const int32_t *__restrict__ order,
                                                           const int32_t *__restrict__ count, const int32_t *__restrict__ nodes_of_bucket,
                                                           int n_train, const int32_t *__restrict__ n_present, int32_t *__restrict__ nodes_before)
{
    __shared__ int lds[17];
    int before = 0, carry = 0;
    for (int b = threadIdx.x; b < (int)blockIdx.x; b += 256) {
        before += totals[b];
        carry += nodes_of_bucket[b];
    }
    block_exclusive_scan<4>(before, lds, before);
    __syncthreads();
    block_exclusive_scan<4>(carry, lds, carry);
    const int m = totals[blockIdx.x];
    for (int t = 0; t < m; t += 256) {
        const int i = t + (int)threadIdx.x;
        const int x = i < m ? count[order[before + i]] : 0;
        __syncthreads();
        int total;
        const int run = carry + block_exclusive_scan<4>(x, lds, total);
        if (i < m) nodes_before[before + i] = run;
        carry += total;
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) nodes_before[*n_present] = n_train;
}

// the stretch of the permutation that a community's super-block (`mix` communities in a row) takes
__global__ __launch_bounds__(256) void stretch_kernel(const int32_t *__restrict__ order, const int32_t *__restrict__ nodes_before,
                                                      const int32_t *__restrict__ n_present, int mix, int2 *__restrict__ stretch)
{
    const int r = (int)blockIdx.x * 256 + (int)threadIdx.x, n = *n_present;
    if (r >= n) return;
    const int first = r - r % mix;
    const int lo = nodes_before[first], hi = nodes_before[(int)min((int64_t)first + mix, (int64_t)n)];
    stretch[order[r]] = make_int2(lo, hi - lo);
}

__global__ __launch_bounds__(256) void copy_i32_kernel(const int32_t *__restrict__ in, int n, int32_t *out)
{
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i < n) out[i] = in[i];
}

template <bool COMMUNITIES>
static void launch_shuffle(const ShuffleArgs &a, hipStream_t s)
{
    const ShufflePlan &pl = a.plan;
    hipLaunchKernelGGL(shuffle_count_kernel<COMMUNITIES>, dim3(pl.n_tiles), dim3(1024), 0, s, a);
    hipLaunchKernelGGL(shuffle_prefix_kernel, dim3((unsigned)ceil_div(pl.n_buckets, 64)), dim3(1024), 0, s, pl, a.counts, a.totals);
    hipLaunchKernelGGL(shuffle_scatter_kernel, dim3(pl.n_tiles), dim3(1024), 0, s, a, COMMUNITIES ? 1 : 0);
    hipLaunchKernelGGL(shuffle_sort_kernel<COMMUNITIES>, dim3(pl.n_buckets), dim3(256), 0, s, a);
}

struct BatchPlan {
    uint32_t *pos;
    uint2 *pairs;
    int32_t *node_comm;
    int32_t *counts, *totals;
    int32_t *present;           // [n_comm] training nodes per community, followed by the number of communities that have one
    int32_t *order, *nodes_of_bucket, *nodes_before;
    int2 *stretch;
    size_t bytes;
};

static void plan_batches(int64_t n_train, int32_t n_comm, void *ws, BatchPlan &p)
{
    const int n = (int)(n_train > n_comm ? n_train : n_comm);
    const ShufflePlan a = shuffle_plan((int)n_train), b = shuffle_plan(n_comm);
    const int64_t cells_a = (int64_t)a.n_tiles * a.n_buckets, cells_b = (int64_t)b.n_tiles * b.n_buckets;
    Carver c(ws);
    p.pos = c.take<uint32_t>((size_t)n);
    p.pairs = c.take<uint2>((size_t)n);
    p.node_comm = c.take<int32_t>((size_t)n_train);
    p.counts = c.take<int32_t>((size_t)(cells_a > cells_b ? cells_a : cells_b));
    p.totals = c.take<int32_t>((size_t)(a.n_buckets > b.n_buckets ? a.n_buckets : b.n_buckets));
    p.present = c.take<int32_t>((size_t)n_comm + 1);
    p.order = c.take<int32_t>((size_t)n_comm);
    p.nodes_of_bucket = c.take<int32_t>((size_t)b.n_buckets);
    p.nodes_before = c.take<int32_t>((size_t)n_comm + 1);
    p.stretch = c.take<int2>((size_t)n_comm);
    p.bytes = c.bytes();
}

}  // namespace cr

using namespace cr;

extern "C" cr_status cr_build_batches_workspace_bytes(int64_t n_train, int32_t n_comm, size_t *bytes)
{
    CR_REQUIRE(n_train >= 0 && n_train < 0x7FFFFFFF, CR_ERR_INVALID_ARG, "n_train must be in 0..2^31-2");
    CR_REQUIRE(n_comm >= 1, CR_ERR_INVALID_ARG, "n_comm must be positive");
    CR_REQUIRE(bytes != nullptr, CR_ERR_INVALID_ARG, "bytes is NULL");
    BatchPlan p;
    plan_batches(n_train, n_comm, nullptr, p);
    *bytes = p.bytes;
    return CR_OK;
}

static cr_status build_batches_impl(const cr_batch_cfg *cfg, const int32_t *train_ids, int64_t n_train,
                                    const int32_t *comm, int32_t n_comm, void *ws, size_t ws_bytes,
                                    int32_t *out_perm, int64_t *out_n_batches, void *stream)
{
    BatchPlan p;
    plan_batches(n_train, n_comm, ws, p);
    CR_REQUIRE(ws != nullptr && aligned16(ws), CR_ERR_INVALID_ARG, "workspace must be a 16-byte aligned device pointer");
    CR_REQUIRE(ws_bytes >= p.bytes, CR_ERR_CAPACITY, "workspace of %zu bytes, %zu needed", ws_bytes, p.bytes);
    if (out_n_batches) *out_n_batches = ceil_div(n_train, cfg->batch_size);
    if (dry_run() || n_train == 0) return CR_OK;

    hipStream_t s = static_cast<hipStream_t>(stream);
    const int n = (int)n_train;
    const dim3 blk(256);
    if (cfg->policy == CR_ROOTS_NORAND) {
        hipLaunchKernelGGL(copy_i32_kernel, dim3((unsigned)ceil_div(n, 256)), blk, 0, s, train_ids, n, out_perm);
        CR_LAUNCH_CHECK();
        return CR_OK;
    }
    ShuffleArgs a;
    a.train = train_ids; a.node_comm = p.node_comm; a.stretch = nullptr; a.present = p.present; a.n_present = p.present + n_comm;
    a.seed = cfg->seed; a.epoch = cfg->epoch;
    a.pos = p.pos; a.counts = p.counts; a.totals = p.totals; a.pairs = p.pairs;
    if (cfg->policy == CR_ROOTS_COMM_RAND && cfg->mix_count < n_comm) {
        // the communities present in the training set, in shuffled order; every one's super-block with its stretch
        hipLaunchKernelGGL(zero_i32_kernel, dim3((unsigned)(ceil_div(n_comm + 1ll, 256) > 1024 ? 1024 : ceil_div(n_comm + 1ll, 256))), blk, 0, s, p.present, n_comm + 1ll);
        hipLaunchKernelGGL(count_communities_kernel, dim3((unsigned)ceil_div(n, 4 * 64 * COUNT_CHUNKS)), blk, 0, s, train_ids, n, comm, p.present, p.present + n_comm, p.node_comm);
        a.plan = shuffle_plan(n_comm);
        a.out = p.order;
        launch_shuffle<true>(a, s);
        const dim3 buckets((unsigned)a.plan.n_buckets);
        hipLaunchKernelGGL(bucket_nodes_kernel, buckets, blk, 0, s, a.plan, p.totals, p.order, p.present, p.nodes_of_bucket);
        hipLaunchKernelGGL(nodes_before_kernel, buckets, blk, 0, s, a.plan, p.totals, p.order, p.present, p.nodes_of_bucket, n, p.present + n_comm, p.nodes_before);
        hipLaunchKernelGGL(stretch_kernel, dim3((unsigned)ceil_div(n_comm, 256)), blk, 0, s, p.order, p.nodes_before, p.present + n_comm, cfg->mix_count, p.stretch);
        a.stretch = p.stretch;
    }
    a.plan = shuffle_plan(n);
    a.out = out_perm;
    launch_shuffle<false>(a, s);
    CR_LAUNCH_CHECK();
    return CR_OK;
}

static cr_status check_batch_args(const cr_batch_cfg *cfg, const int32_t *train_ids, int64_t n_train, const int32_t *comm,
                                  int32_t n_comm, const int32_t *out_perm)
{
    CR_REQUIRE(cfg != nullptr, CR_ERR_INVALID_ARG, "cfg is NULL");
    CR_REQUIRE(cfg->policy >= CR_ROOTS_NORAND && cfg->policy <= CR_ROOTS_RAND, CR_ERR_INVALID_ARG, "unknown root policy %d", cfg->policy);
    CR_REQUIRE(cfg->policy != CR_ROOTS_COMM_RAND || cfg->mix_count >= 1, CR_ERR_INVALID_ARG, "mix_count must be >= 1");
    CR_REQUIRE(cfg->batch_size >= 1, CR_ERR_INVALID_ARG, "batch_size must be positive");
    CR_REQUIRE(cfg->epoch < (1u << 24), CR_ERR_INVALID_ARG, "epoch must be below 2^24");
    CR_REQUIRE(n_train >= 0 && n_train < 0x7FFFFFFF, CR_ERR_INVALID_ARG, "n_train must be in 0..2^31-2");
    CR_REQUIRE(n_comm >= 1, CR_ERR_INVALID_ARG, "n_comm must be positive");
    CR_REQUIRE(n_train == 0 || (train_ids && out_perm), CR_ERR_INVALID_ARG, "train_ids / out_perm must not be NULL");
    CR_REQUIRE(comm != nullptr, CR_ERR_INVALID_ARG, "comm is NULL");
    return CR_OK;
}

extern "C" cr_status cr_build_batches(const cr_batch_cfg *cfg, const int32_t *train_ids, int64_t n_train,
                                      const int32_t *comm, int32_t n_comm, void *ws, size_t ws_bytes,
                                      int32_t *out_perm, int64_t *out_n_batches, void *stream)
{
    cr_status st = check_batch_args(cfg, train_ids, n_train, comm, n_comm, out_perm);
    if (st != CR_OK) return st;
    return build_batches_impl(cfg, train_ids, n_train, comm, n_comm, ws, ws_bytes, out_perm, out_n_batches, stream);
}

// ---------------------------------------------------------------------------------------------
// The same without a caller workspace: sort buffers, histograms and community tables live in a fixed device array of
// this library.  Host code never uses the array's name as an address: the array's device address is looked up once
// per device and kept.
// ---------------------------------------------------------------------------------------------
constexpr size_t STATIC_SCRATCH_BYTES = 8u << 20;
static __device__ __align__(256) unsigned char scratch[STATIC_SCRATCH_BYTES];

namespace {
constexpr int MAX_DEVICES = 64;
std::mutex scratch_mutex;
void *scratch_ptr[MAX_DEVICES] = {};
}  // namespace

extern "C" cr_status cr_build_batches_static(const cr_batch_cfg *cfg, const int32_t *train_ids, int64_t n_train,
                                             const int32_t *comm, int32_t n_comm, int32_t *out_perm,
                                             int64_t *out_n_batches, void *stream)
{
    cr_status st = check_batch_args(cfg, train_ids, n_train, comm, n_comm, out_perm);
    if (st != CR_OK) return st;
    CR_REQUIRE(n_train <= CR_STATIC_MAX_TRAIN, CR_ERR_CAPACITY,
               "n_train = %lld exceeds what the library's fixed scratch array holds (%d training nodes); use cr_build_batches with a workspace",
               (long long)n_train, CR_STATIC_MAX_TRAIN);
    CR_REQUIRE(n_comm <= CR_STATIC_MAX_COMM, CR_ERR_CAPACITY,
               "n_comm = %d exceeds what the library's fixed scratch array holds (%d communities); use cr_build_batches with a workspace",
               n_comm, CR_STATIC_MAX_COMM);
    BatchPlan p;
    plan_batches(n_train, n_comm, nullptr, p);
    CR_REQUIRE(p.bytes <= STATIC_SCRATCH_BYTES, CR_ERR_CAPACITY, "scratch of %zu bytes, %zu needed", STATIC_SCRATCH_BYTES, p.bytes);
    if (dry_run()) {
        if (out_n_batches) *out_n_batches = ceil_div(n_train, cfg->batch_size);
        return CR_OK;
    }
    int dev = 0;
    CR_HIP_CHECK(hipGetDevice(&dev));
    CR_REQUIRE(dev >= 0 && dev < MAX_DEVICES, CR_ERR_UNSUPPORTED, "device index %d outside 0..%d", dev, MAX_DEVICES - 1);
    void *ws = nullptr;
    {
        std::lock_guard<std::mutex> lock(scratch_mutex);
        if (!scratch_ptr[dev]) {
            void *ptr = nullptr;
            CR_HIP_CHECK(hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)));
            CR_REQUIRE(ptr != nullptr, CR_ERR_HIP, "the scratch array has no device address");
            scratch_ptr[dev] = ptr;
        }
        ws = scratch_ptr[dev];
    }
    return build_batches_impl(cfg, train_ids, n_train, comm, n_comm, ws, STATIC_SCRATCH_BYTES, out_perm, out_n_batches, stream);
}
