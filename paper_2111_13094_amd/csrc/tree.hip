// tree.hip -- the spatial kD-tree on gfx950: pre-subdivision, refinement of leaves with
// many samples, copies of the parent mixture into new leaves, leaf initialisation, and
// the reordering of the samples by leaf that the batched fit consumes (Dodik et al.,
// arXiv 2111.13094, Sec. 4.2 "Refinement of the spatial kD-tree", Sec. 4.3
// "Initialization").
//
// Refinement: every sample is located in the tree once; a stable counting sort by leaf
// moves the samples into leaf order as 16-byte records (position and index, direction and
// weight); then rounds of splits work on the leaves' contiguous segments. Each round, for
// every leaf of the round with more than c samples: the split from its FP64 position
// statistics (fixed reduction order), the decisions in leaf order by one work group (block
// prefix sums number the new nodes and leaves), and a stable partition of its segment,
// which also forms the two children's statistics. Leaves that do not split are not
// touched. No round waits for the host: the rounds' lists of leaves and work items live on
// the device, the host queues a group of rounds ahead and reads back whether any leaf is
// left. At the end the records are written out in the order of the leaf indices, and new
// leaves get copies of their parent's mixture and Robbins-Monro state.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <vector>

#include "common.hpp"
#include "launch_rules.hpp"
#include "timing.hpp"

namespace sdmm {

constexpr int kSortThreads = 1024;
constexpr int kSortWaves = kSortThreads / 64;
constexpr int kSortItems = 4;                         // samples per thread per tile
constexpr int kSortTile = kSortThreads * kSortItems;  // samples per tile
constexpr int kDigitBits = 12, kMaxBins = 1 << kDigitBits;  // bins of one sorting pass
constexpr int kScanRows = 32;                         // tiles per group of the tables' prefix sum
constexpr int kChunkThreads = 512;
constexpr int kChunkItems = 8;                              // records per thread per chunk
constexpr int kChunk = kChunkThreads * kChunkItems;         // most records per chunk of a leaf
constexpr int kMaxRounds = 64;

struct TreePtrs {
    int32_t max_nodes, max_leaves;
    int32_t *counts, *axis, *left, *leaf;
    double* split;
    int32_t* leaf_node;
    double *lo, *hi;
    int32_t* init;
};

// ---------------------------------------------------------------------------------
// pre-subdivision: node n of the complete tree (children 2n + 1, 2n + 2); its path from
// the root is the binary expansion of n + 1 after the leading one (0 = left)
// ---------------------------------------------------------------------------------
__global__ void tree_init_kernel(TreePtrs t, int levels, double lo0, double lo1, double lo2, double hi0, double hi1,
                                 double hi2)
{
    const int64_t n_leaves = int64_t(1) << levels, n_nodes = 2 * n_leaves - 1;
    const int64_t n = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (n >= n_nodes) return;
    int level = 0;
    while ((int64_t(1) << (level + 1)) - 1 <= n) ++level;
    double blo[3] = {lo0, lo1, lo2}, bhi[3] = {hi0, hi1, hi2};
    const uint64_t path = (uint64_t)(n + 1);
    for (int l = 0; l < level; ++l) {  // walk down from the root
        const int ax = l % 3;
        const double mid = 0.5 * (blo[ax] + bhi[ax]);
        const int right = (int)((path >> (level - 1 - l)) & 1);
        if (right) blo[ax] = mid;
        else bhi[ax] = mid;
    }
    if (level < levels) {
        const int ax = level % 3;
        t.axis[n] = ax;
        t.split[n] = 0.5 * (blo[ax] + bhi[ax]);
        t.left[n] = (int32_t)(2 * n + 1);
        t.leaf[n] = -1;
    } else {
        const int64_t l = n - (n_leaves - 1);
        t.axis[n] = -1;
        t.split[n] = 0.0;
        t.left[n] = -1;
        t.leaf[n] = (int32_t)l;
        t.leaf_node[l] = (int32_t)n;
        for (int d = 0; d < 3; ++d) {
            t.lo[3 * l + d] = blo[d];
            t.hi[3 * l + d] = bhi[d];
        }
        t.init[l] = 0;
    }
    if (n == 0) {
        t.counts[0] = (int32_t)n_nodes;
        t.counts[1] = (int32_t)n_leaves;
    }
}

// Work groups go to the eight XCDs in turn (group b to XCD b % 8), each XCD with its own
// L2. The groups of one XCD take consecutive ranges of the output, so that a line
// that two groups share is read or written in one L2, not in two.
__device__ __forceinline__ int64_t xcd_block_order(int64_t b, int64_t nb)
{
    const int64_t x = b % 8, q = b / 8, per = nb / 8, extra = nb % 8;
    return x * per + (x < extra ? x : extra) + q;
}

// ---------------------------------------------------------------------------------
// point location: left where p[axis] < split, else right; child indices exceed their
// parent's, so a walk ends within max_nodes steps. The oldest nodes, the top of the tree,
// are staged in LDS by every work group (one 8-byte entry per node, indices below
// kLocStaged: the whole tree while it has no more nodes than that), so a walk costs one
// LDS read per level there; below them a node's axis, split, left child and leaf index
// are loaded from global memory together (one memory round trip per level). Each thread
// walks kLocPer samples side by side, so their reads overlap, and issues the next step's
// positions before it walks the current ones. The work group also counts its tile's
// samples per bin of the first sorting pass (the low kDigitBits bits of the leaf) in LDS
// and writes the counts as one row of the sort's table.
//
// A staged entry holds the split rounded up to FP32: for an FP32 coordinate p and an FP64
// split s, p < s exactly when p < f, f the least FP32 value not below s (every FP32 value
// below s is at most the greatest one below f), so the walk takes the FP64 comparison's
// branch with an FP32 comparison.
// ---------------------------------------------------------------------------------
constexpr int kLocThreads = 512;
constexpr int kLocPer = 4;                       // samples per thread per step
constexpr int kLocTile = kLocThreads * kLocPer;  // samples per work group per step
static_assert(kSortTile % kLocTile == 0, "a sorting tile is a whole number of steps");
constexpr int kLocStaged = 4096;                 // nodes staged in LDS (32 KB)
constexpr int kLocMaxGroups = 256 * 4;           // 4 work groups per CU
constexpr int32_t kUnstaged = INT32_MIN;         // an inner node whose child index does not fit the code

struct alignas(8) StagedNode {
    float split;   // the split rounded up to FP32
    int32_t code;  // inner node: 4 left + axis; leaf: -(leaf index) - 1; or kUnstaged
};

__device__ __forceinline__ float round_up_f32(double s)
{
    float f = (float)s;
    if ((double)f < s) f = __int_as_float(__float_as_int(f) + (f >= 0.0f ? 1 : -1));
    return f;
}

__device__ __forceinline__ void loc_loads(const float* __restrict__ smp, int64_t N, int64_t b, float (&p0)[kLocPer],
                                          float (&p1)[kLocPer], float (&p2)[kLocPer])
{
#pragma unroll
    for (int r = 0; r < kLocPer; ++r) {  // a lane past the end loads the last sample's
        const int64_t ic = min(b + r * kLocThreads, N - 1);
        p0[r] = smp[3 * N + ic];
        p1[r] = smp[4 * N + ic];
        p2[r] = smp[5 * N + ic];
    }
}

// adds one to h[bin] for every valid lane; a wave whose valid lanes share the bin (samples
// that arrive grouped by leaf) adds their number once, where the atomics would serialise
__device__ __forceinline__ void count_bins(int32_t* h, int bin, bool valid)
{
    const uint64_t vm = __ballot(valid);
    const int b0 = __builtin_amdgcn_readlane(bin, vm ? __builtin_ctzll(vm) : 0);
    if (__all(!valid || bin == b0)) {
        if (vm && (threadIdx.x & 63) == 0) atomicAdd(&h[b0], __popcll(vm));
    } else if (valid) {
        atomicAdd(&h[bin], 1);
    }
}

__global__ __launch_bounds__(kLocThreads) void locate_kernel(TreePtrs t, const float* __restrict__ smp, int64_t N,
                                                             int32_t* __restrict__ leaf_of, int32_t* __restrict__ hist,
                                                             int n_tiles)
{
    __shared__ StagedNode top[kLocStaged];
    __shared__ int32_t h[kMaxBins];
    const int32_t ns = max(1, min(min(t.counts[0], t.max_nodes), kLocStaged));
    // bins of the first sorting pass; a leaf index of a tree that the host will reject for
    // its counts is kept inside them
    const int32_t bins = max(1, min(min(t.counts[1], t.max_leaves), kMaxBins));
    {
        constexpr int kPer = kLocStaged / kLocThreads;
        const int jn = (ns + kLocThreads - 1) / kLocThreads;  // the same in every lane
        int32_t ax[kPer], lf[kPer], lv[kPer];
        double sp[kPer];
#pragma unroll
        for (int j = 0; j < kPer; ++j) {  // all loads first, then the LDS writes
            if (j >= jn) break;
            const int k = min(j * kLocThreads + (int)threadIdx.x, ns - 1);
            ax[j] = t.axis[k];
            lf[j] = t.left[k];
            lv[j] = t.leaf[k];
            sp[j] = t.split[k];
        }
#pragma unroll
        for (int j = 0; j < kPer; ++j) {
            if (j >= jn) break;
            const int k = j * kLocThreads + (int)threadIdx.x;
            const int32_t code = ax[j] < 0 ? -lv[j] - 1 : (lf[j] < (1 << 29) ? 4 * lf[j] + ax[j] : kUnstaged);
            if (k < ns) top[k] = StagedNode{round_up_f32(sp[j]), code};
        }
    }
    for (int b = threadIdx.x; b < bins; b += kLocThreads) h[b] = 0;
    __syncthreads();
    // a lane past the end walks the last sample's path again and stores nothing
    constexpr int kSteps = kSortTile / kLocTile;
    float p0[kLocPer], p1[kLocPer], p2[kLocPer];  // positions of the next step
    if ((int)blockIdx.x < n_tiles)
        loc_loads(smp, N, (int64_t)blockIdx.x * kSortTile + threadIdx.x, p0, p1, p2);
    for (int tile = blockIdx.x; tile < n_tiles; tile += gridDim.x) {
        for (int step = 0; step < kSteps; ++step) {
            const int64_t base = (int64_t)tile * kSortTile + step * kLocTile + threadIdx.x;
            int32_t n[kLocPer];
            float q0[kLocPer], q1[kLocPer], q2[kLocPer];
#pragma unroll
            for (int r = 0; r < kLocPer; ++r) {
                n[r] = 0;
                q0[r] = p0[r];
                q1[r] = p1[r];
                q2[r] = p2[r];
            }
            const int64_t next = step + 1 < kSteps ? base + kLocTile
                                                   : (int64_t)(tile + (int)gridDim.x) * kSortTile + threadIdx.x;
            if (step + 1 < kSteps || tile + (int)gridDim.x < n_tiles) loc_loads(smp, N, next, p0, p1, p2);
            // the staged levels: a step per LDS read
            for (int32_t s = 0; s <= ns; ++s) {
                bool more = false;
                StagedNode e[kLocPer];
#pragma unroll
                for (int r = 0; r < kLocPer; ++r) e[r] = top[min(n[r], ns - 1)];
#pragma unroll
                for (int r = 0; r < kLocPer; ++r) {
                    const bool go = n[r] < ns && e[r].code >= 0;
                    const float t01 = (e[r].code & 1) ? q1[r] : q0[r];
                    const float pa = (e[r].code & 2) ? q2[r] : t01;
                    const int32_t to = (e[r].code >> 2) + (pa < e[r].split ? 0 : 1);
                    n[r] = go ? to : n[r];
                    more |= go;
                }
                if (!more) break;
            }
            // the levels below: a step per global round trip (only where a walk left the
            // staged nodes, so that the other waves never wait for the next tile's loads)
            int32_t lv[kLocPer];
            bool staged[kLocPer], below = false;
#pragma unroll
            for (int r = 0; r < kLocPer; ++r) {
                const int32_t c = top[min(n[r], ns - 1)].code;
                staged[r] = n[r] < ns && c != kUnstaged;  // then a leaf
                lv[r] = -c - 1;
                below |= !staged[r];
            }
            if (below) {
                int32_t ax[kLocPer], lf[kLocPer];
                double sp[kLocPer];
#pragma unroll
                for (int r = 0; r < kLocPer; ++r) {
                    ax[r] = -1;
                    lf[r] = -1;
                    sp[r] = 0.0;
                    if (!staged[r]) {
                        ax[r] = t.axis[n[r]];
                        lf[r] = t.left[n[r]];
                        sp[r] = t.split[n[r]];
                        lv[r] = t.leaf[n[r]];
                    }
                }
                for (int32_t s = 0; s < t.max_nodes; ++s) {
                    // the loads above and below complete together at these empty statements
                    // (the compiler would otherwise issue the later ones only after the axis
                    // came back)
#pragma unroll
                    for (int r = 0; r < kLocPer; ++r)
                        asm volatile("" ::"v"(ax[r]), "v"(lf[r]), "v"(sp[r]), "v"(lv[r]));
                    bool more = false;
#pragma unroll
                    for (int r = 0; r < kLocPer; ++r) {
                        if (ax[r] >= 0) {
                            const float pa = ax[r] == 0 ? q0[r] : (ax[r] == 1 ? q1[r] : q2[r]);
                            n[r] = (double)pa < sp[r] ? lf[r] : lf[r] + 1;
                            ax[r] = t.axis[n[r]];
                            lf[r] = t.left[n[r]];
                            sp[r] = t.split[n[r]];
                            lv[r] = t.leaf[n[r]];
                            more = true;
                        }
                    }
                    if (!more) break;
                }
            }

#pragma unroll
            for (int r = 0; r < kLocPer; ++r) {
                const int64_t i = base + r * kLocThreads;
                const int32_t leaf = max(lv[r], 0);
                if (i < N) leaf_of[i] = leaf;
                count_bins(h, min(leaf & (kMaxBins - 1), bins - 1), i < N);
            }
        }
        __syncthreads();
        for (int b = threadIdx.x; b < bins; b += kLocThreads) {
            hist[(int64_t)tile * bins + b] = h[b];
            h[b] = 0;
        }
        __syncthreads();
    }
}

// ---------------------------------------------------------------------------------
// Stable counting sort by leaf, kDigitBits bits of the leaf index per pass (one pass up to
// 4096 leaves): a table of counts with one row per tile (written by the location for the
// first pass), its prefix sums down the tiles and across the bins, and the move. The
// samples are moved whole, as two 16-byte records: position and index, direction and
// weight. A sample's record then lands in a full sector, and runs of one tile's samples of
// a leaf are contiguous; moving indices only left a gather of 28 bytes in 4-byte pieces
// from 7 random lines each to the end (2.04 ms of the 12.5 ms of a 16.6M-sample refinement
// in path order), and every round's partition and statistics read through the
// permutation as well.
// ---------------------------------------------------------------------------------

// counts per tile and bin of the keys' digit (passes after the first)
__global__ __launch_bounds__(kSortThreads) void tile_hist_kernel(const int32_t* __restrict__ keys, int64_t N, int shift,
                                                                 int bins, int32_t* __restrict__ hist)
{
    __shared__ int32_t h[kMaxBins];
    for (int b = threadIdx.x; b < bins; b += kSortThreads) h[b] = 0;
    __syncthreads();
    const int64_t base = (int64_t)blockIdx.x * kSortTile + threadIdx.x;
    int32_t kv[kSortItems];  // the thread's keys, loaded together
#pragma unroll
    for (int it = 0; it < kSortItems; ++it) kv[it] = keys[min(base + it * kSortThreads, N - 1)];
#pragma unroll
    for (int it = 0; it < kSortItems; ++it)
        count_bins(h, min((kv[it] >> shift) & (kMaxBins - 1), bins - 1), base + it * kSortThreads < N);
    __syncthreads();
    for (int b = threadIdx.x; b < bins; b += kSortThreads) hist[(int64_t)blockIdx.x * bins + b] = h[b];
}

// exclusive prefix sum of each bin down the kScanRows tiles of a group (in place), and the
// group's total; consecutive threads take consecutive bins, so every row is read whole
__global__ __launch_bounds__(256) void scan_group_kernel(int32_t* __restrict__ hist, int n_tiles, int bins,
                                                         int32_t* __restrict__ gsum)
{
    const int b = blockIdx.x * 256 + threadIdx.x, g = blockIdx.y;
    if (b >= bins) return;
    const int t0 = g * kScanRows;
    int32_t v[kScanRows];
#pragma unroll
    for (int i = 0; i < kScanRows; ++i) v[i] = t0 + i < n_tiles ? hist[(int64_t)(t0 + i) * bins + b] : 0;
    int32_t run = 0;
#pragma unroll
    for (int i = 0; i < kScanRows; ++i) {
        if (t0 + i < n_tiles) hist[(int64_t)(t0 + i) * bins + b] = run;
        run += v[i];
    }
    gsum[(int64_t)g * bins + b] = run;
}

// exclusive prefix sum of each bin over the groups (in place), and the bin's total
__global__ __launch_bounds__(64) void scan_bins_kernel(int32_t* __restrict__ gsum, int n_groups, int bins,
                                                       int32_t* __restrict__ total)
{
    const int b = blockIdx.x * 64 + threadIdx.x;
    if (b >= bins) return;
    constexpr int U = 16;
    int32_t run = 0;
    for (int g0 = 0; g0 < n_groups; g0 += U) {
        int32_t v[U];
#pragma unroll
        for (int i = 0; i < U; ++i) v[i] = g0 + i < n_groups ? gsum[(int64_t)(g0 + i) * bins + b] : 0;
#pragma unroll
        for (int i = 0; i < U; ++i) {
            if (g0 + i < n_groups) gsum[(int64_t)(g0 + i) * bins + b] = run;
            run += v[i];
        }
    }
    total[b] = run;
}

// exclusive prefix sum over a work group of 1024 threads
template <typename T>
__device__ __forceinline__ T block_scan_1024(T v, T* wsum, T& total)
{
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    T x = v;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const T y = __shfl_up(x, o);
        if (lane >= o) x += y;
    }
    if (lane == 63) wsum[w] = x;
    __syncthreads();
    T before = 0, all = 0;
#pragma unroll
    for (int q = 0; q < 16; ++q) {
        const T s = wsum[q];
        before += q < w ? s : T(0);
        all += s;
    }
    total = all;
    __syncthreads();
    return before + x - v;
}

// A leaf of a round: its segment of the records (in buffer src), its chunks (work items
// item0 .. item0 + nch - 1) and the partial statistics to sum for it (pn of them from
// pfirst, on one side of their records' split).
struct Entry {
    int32_t leaf, start, count, src, item0, nch, pfirst, pn2;  // pn2 = 2 pn + side
};

// statistics of a chunk's samples, or of those on one side of its split
struct Part {
    double s1[3], sq[3];
    float mn[3], mx[3];
};

// the device's control words: entries and work items of the lists of even and odd rounds,
// the status bits, the number of leaves
constexpr int kCtlEntries = 0, kCtlItems = 2, kCtlStatus = 4, kCtlLeaves = 5, kCtlWords = 8;

// whether no leaf is left to split: the list that the last of the queued rounds wrote is
// empty (done < 2: its parity), or the limit of the rounds is reached (done = 2)
__device__ __forceinline__ bool finished(const int32_t* __restrict__ ctl, int done)
{
    return done == 2 || ctl[kCtlEntries + done] == 0;
}

struct LeafTabs {
    int32_t *start, *count, *par, *next;  // segment and its buffer; the leaf whose segment follows
    int32_t* origin;                      // the leaf whose mixture a new leaf copies
    int32_t* cover;                       // leaf of the records at multiples of kCover
};
constexpr int kCover = 256;

struct RoundBufs {
    Entry* entries[2];
    int32_t *items[2], *rtot[2];  // entry of each work item; samples on the right per entry
    Part* parts[2];               // per side: parts[.][side * max_items + item]
    int32_t *item_right, *flags, *ax;
    double* split;
    int32_t max_items;
};

// One work group: a pass's bins get their bases (exclusive prefix sum of the totals); with
// leaves, every bin is a leaf and the leaf tables are set from them (else from the starts
// that starts_kernel wrote), and the first round's list takes every leaf with more than c
// samples, in leaf order.
__global__ __launch_bounds__(1024) void base_kernel(int32_t* __restrict__ total, int bins, int leaves, int32_t L, int32_t c,
                                                    LeafTabs lt, RoundBufs rb, int32_t* __restrict__ ctl)
{
    __shared__ int64_t ws[16];
    __shared__ int32_t ws32[16];
    const int tid = threadIdx.x;
    if (bins > 0) {
        int32_t run = 0;
        for (int b0 = 0; b0 < bins; b0 += 1024) {
            const int b = b0 + tid;
            const int32_t v = b < bins ? total[b] : 0;
            int32_t all;
            const int32_t x = run + block_scan_1024(v, ws32, all);
            if (b < bins) total[b] = x;
            if (leaves && b < L) {
                lt.start[b] = x;
                lt.count[b] = v;
            }
            run += all;
        }
    }
    if (!leaves) return;
    if (bins == 0) {
        for (int32_t l = tid; l < L; l += 1024) lt.count[l] = lt.start[l + 1] - lt.start[l];
    }
    __syncthreads();
    int32_t e0 = 0, i0 = 0;
    for (int32_t l0 = 0; l0 < L; l0 += 1024) {
        const int32_t l = l0 + tid;
        const int32_t n = l < L ? lt.count[l] : 0;
        if (l < L) {
            lt.par[l] = 0;
            lt.next[l] = l + 1;
            lt.origin[l] = l;
        }
        const bool in = n > c;
        const int32_t nch = in ? chunks_of(n, kChunk) : 0;
        int64_t all;
        const int64_t x = block_scan_1024(((int64_t)(in ? 1 : 0) << 32) | nch, ws, all);
        if (in) {
            const int32_t e = e0 + (int32_t)(x >> 32), it = i0 + (int32_t)x;
            rb.entries[0][e] = Entry{l, lt.start[l], n, 0, it, nch, it, 2 * nch};
            rb.rtot[0][e] = 0;
            for (int32_t q = 0; q < nch; ++q) rb.items[0][it + q] = e;
        }
        e0 += (int32_t)(all >> 32);
        i0 += (int32_t)all;
    }
    if (tid == 0) {
        ctl[kCtlEntries] = e0;
        ctl[kCtlItems] = i0;
        ctl[kCtlEntries + 1] = ctl[kCtlItems + 1] = 0;
        ctl[kCtlStatus] = 0;
        ctl[kCtlLeaves] = L;
    }
}

// start[l] = first sorted position of leaf l (start[L] = N), from the sorted keys (more
// leaves than one pass has bins)
__global__ void starts_kernel(const int32_t* __restrict__ keys, int64_t N, int32_t L, int32_t* __restrict__ start)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= N) return;
    const int32_t k = keys[i], kp = i > 0 ? keys[i - 1] : -1;
    for (int32_t l = kp + 1; l <= k; ++l) start[l] = (int32_t)i;
    if (i == N - 1)
        for (int32_t l = k + 1; l <= L; ++l) start[l] = (int32_t)N;
}

// the valid lanes of the wave whose digit equals this lane's (meaningful for valid lanes):
// one comparison when every valid lane holds the same digit, as in runs of samples of one
// leaf, else one ballot per digit bit
__device__ __forceinline__ uint64_t digit_peers(int digit, bool valid, int bits)
{
    const uint64_t vm = __ballot(valid);
    const int d0 = __builtin_amdgcn_readfirstlane(digit);
    if (__all(!valid || digit == d0)) return vm;
    uint64_t peers = vm;
    for (int b = 0; b < bits; ++b) {
        const bool on = (digit >> b) & 1;
        const uint64_t m = __ballot(on);
        peers &= on ? m : ~m;
    }
    return peers;
}

// Each work group moves its tile, wave w the w-th 64 kSortItems samples of it in order:
// first every sample's rank among the wave's samples of its digit (ballots within 64
// samples, a running count per digit in the wave's own row of LDS across them), then the
// rows' prefix over the waves, then the moves. Work groups of one XCD take consecutive
// tiles, so that a line that two tiles' runs share is written in one L2.
//
// With up to kStageBins bins the records go to LDS in their sorted order first (positions,
// then directions and weights, through the same 64 KB), and consecutive lanes then write
// the runs of a digit whole. The traffic is what it has to be (by counters 540 MB read and
// 532 MB written for 16.6M samples over 512 leaves, 32 bytes each way and the keys), so latency
// sets the time: 16 waves per tile take 243 us, 4 waves with four times the samples each took
// 428 us (4.4 against 2.5 TB/s). Stored as they come, 16 bytes a request, the records take 378 us. With more bins
// a tile's runs are only a record or two long and the rows no longer fit: the records are
// stored as they come.
constexpr int kStageBins = 2048;

template <bool FromSamples, bool Staged>
__global__ __launch_bounds__(kSortThreads) void scatter_kernel(
    const float* __restrict__ smp, const float4* __restrict__ pin, const float4* __restrict__ qin,
    const int32_t* __restrict__ kin, int64_t N, int shift, int bins, int bits, const int32_t* __restrict__ hist,
    const int32_t* __restrict__ gsum, const int32_t* __restrict__ base, float4* __restrict__ pout,
    float4* __restrict__ qout, int32_t* __restrict__ kout)
{
    extern __shared__ int32_t lds[];
    // staged: the counts share the records' LDS (every place is in registers before the
    // first record is stored)
    __shared__ float4 stage[Staged ? kSortTile : 1];
    __shared__ int32_t gbase_s[Staged ? kStageBins : 1], lbase[Staged ? kStageBins : 1];
    __shared__ int32_t wsum[kSortWaves];
    static_assert(kSortWaves * kStageBins * sizeof(uint16_t) <= kSortTile * sizeof(float4), "the counts fit");
    int32_t* gbase = Staged ? gbase_s : lds;                                                    // [bins]
    uint16_t* wc = reinterpret_cast<uint16_t*>(Staged ? (void*)stage : (void*)(lds + bins));    // [kSortWaves][bins]
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int tile = (int)xcd_block_order(blockIdx.x, gridDim.x);
    const uint64_t lt = lane ? (~0ull >> (64 - lane)) : 0ull;
    const int64_t tile0 = (int64_t)tile * kSortTile;
    const int64_t first = tile0 + w * (64 * kSortItems) + lane;
    int32_t kv[kSortItems], rank[kSortItems];
#pragma unroll
    for (int it = 0; it < kSortItems; ++it) kv[it] = kin[min(first + it * 64, N - 1)];
    for (int b = tid; b < bins; b += kSortThreads) {
        gbase[b] = base[b] + gsum[(int64_t)(tile / kScanRows) * bins + b] + hist[(int64_t)tile * bins + b];
#pragma unroll
        for (int q = 0; q < kSortWaves; ++q) wc[q * bins + b] = 0;
    }
    __syncthreads();
    volatile uint16_t* row = wc + w * bins;
#pragma unroll
    for (int it = 0; it < kSortItems; ++it) {
        const bool valid = first + it * 64 < N;
        const int digit = min((kv[it] >> shift) & (kMaxBins - 1), bins - 1);
        const uint64_t peers = digit_peers(digit, valid, bits);
        const int before = row[digit];
        rank[it] = before + __popcll(peers & lt);
        __builtin_amdgcn_wave_barrier();
        if (valid && (peers & lt) == 0) row[digit] = (uint16_t)(before + __popcll(peers));
        __builtin_amdgcn_wave_barrier();
    }
    __syncthreads();
    // rows to their prefix over the waves; staged: a digit's first place in the tile's order
    int32_t run0 = 0;
    for (int b0 = 0; b0 < bins; b0 += kSortThreads) {  // the same trips in every thread
        const int b = b0 + tid;
        int run = 0;
        if (b < bins) {
#pragma unroll
            for (int q = 0; q < kSortWaves; ++q) {
                const int v = wc[q * bins + b];
                wc[q * bins + b] = (uint16_t)run;
                run += v;
            }
        }
        if constexpr (Staged) {
            int32_t x = run;
#pragma unroll
            for (int o = 1; o < 64; o <<= 1) {
                const int32_t y = __shfl_up(x, o);
                if (lane >= o) x += y;
            }
            if (lane == 63) wsum[w] = x;
            __syncthreads();
            int32_t before = run0;
#pragma unroll
            for (int q = 0; q < kSortWaves; ++q) {
                before += q < w ? wsum[q] : 0;
                run0 += wsum[q];
            }
            if (b < bins) lbase[b] = before + x - run;
            __syncthreads();
        }
    }
    __syncthreads();
    auto digit_of = [&](int it) { return min((kv[it] >> shift) & (kMaxBins - 1), bins - 1); };
    auto load_p = [&](int64_t i) {
        if constexpr (FromSamples) return make_float4(smp[3 * N + i], smp[4 * N + i], smp[5 * N + i], 0.0f);
        else return pin[i];
    };
    auto load_q = [&](int64_t i) {
        if constexpr (FromSamples) return make_float4(smp[i], smp[N + i], smp[2 * N + i], smp[6 * N + i]);
        else return qin[i];
    };
    if constexpr (Staged) {
        const int n = (int)min((int64_t)kSortTile, N - tile0);
        float4 p[kSortItems], q[kSortItems];
#pragma unroll
        for (int it = 0; it < kSortItems; ++it) p[it] = load_p(min(first + it * 64, N - 1));
#pragma unroll
        for (int it = 0; it < kSortItems; ++it) q[it] = load_q(min(first + it * 64, N - 1));
        int32_t at[kSortItems];  // place of the thread's samples in the tile's order
#pragma unroll
        for (int it = 0; it < kSortItems; ++it) {
            const int d = digit_of(it);
            at[it] = wc[w * bins + d] + rank[it];
            rank[it] = gbase[d] + at[it];  // where it goes
            at[it] += lbase[d];
            p[it].w = __int_as_float(rank[it]);
        }
        __syncthreads();
#pragma unroll
        for (int it = 0; it < kSortItems; ++it)
            if (first + it * 64 < N) stage[at[it]] = p[it];
        __syncthreads();
        int32_t dst[kSortItems];
#pragma unroll
        for (int j = 0; j < kSortItems; ++j) {
            const int k = j * kSortThreads + tid;
            const float4 p = stage[min(k, n - 1)];
            dst[j] = __float_as_int(p.w);
            if (k < n) pout[dst[j]] = p;
        }
        __syncthreads();
#pragma unroll
        for (int it = 0; it < kSortItems; ++it)
            if (first + it * 64 < N) stage[at[it]] = q[it];
        __syncthreads();
#pragma unroll
        for (int j = 0; j < kSortItems; ++j) {
            const int k = j * kSortThreads + tid;
            if (k < n) qout[dst[j]] = stage[k];
        }
        if (kout) {
#pragma unroll
            for (int it = 0; it < kSortItems; ++it)
                if (first + it * 64 < N) kout[rank[it]] = kv[it];
        }
    } else {
        constexpr int U = 4;  // samples in flight per thread
#pragma unroll
        for (int i0 = 0; i0 < kSortItems; i0 += U) {
            float4 p[U], q[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int64_t i = min(first + (i0 + u) * 64, N - 1);
                p[u] = load_p(i);
                q[u] = load_q(i);
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int it = i0 + u;
                if (first + it * 64 >= N) continue;
                const int d = digit_of(it);
                const int32_t dst = gbase[d] + wc[w * bins + d] + rank[it];
                p[u].w = __int_as_float(dst);
                pout[dst] = p[u];
                qout[dst] = q[u];
                if (kout) kout[dst] = kv[it];
            }
        }
    }
}

// ---------------------------------------------------------------------------------
// A round's chunks: the leaves of a round are cut into chunks of at most kChunk records,
// one work group each, so a few huge leaves fill the chip as well as many small ones (one
// group per leaf took 640 us per round on 512 leaves of 1e4 to 2e5 samples). A leaf's
// chunks are of one size (a multiple of 64), the last of what is left.
// ---------------------------------------------------------------------------------
__device__ __forceinline__ void chunk_range(const Entry& e, int32_t q, int32_t& lo, int32_t& hi)
{
    lo = chunk_begin(e.count, e.nch, q);
    hi = chunk_end(e.count, e.nch, q);
}

// a thread's running statistics
struct Stat {
    double s1[3] = {0, 0, 0}, sq[3] = {0, 0, 0};
    float mn[3] = {INFINITY, INFINITY, INFINITY}, mx[3] = {-INFINITY, -INFINITY, -INFINITY};
    __device__ __forceinline__ void add(const float4& p)
    {
        const float v[3] = {p.x, p.y, p.z};
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            const double x = (double)v[d];
            s1[d] += x;
            sq[d] += x * x;
            mn[d] = fminf(mn[d], v[d]);
            mx[d] = fmaxf(mx[d], v[d]);
        }
    }
    __device__ __forceinline__ void merge(const Part& o)
    {
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            s1[d] += o.s1[d];
            sq[d] += o.sq[d];
            mn[d] = fminf(mn[d], o.mn[d]);
            mx[d] = fmaxf(mx[d], o.mx[d]);
        }
    }
    // over the wave, in a fixed order (every lane gets the result)
    __device__ __forceinline__ void wave_reduce()
    {
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            s1[d] = wave_sum_f64(s1[d]);
            sq[d] = wave_sum_f64(sq[d]);
        }
#pragma unroll
        for (int o = 1; o < 64; o <<= 1)
#pragma unroll
            for (int d = 0; d < 3; ++d) {
                mn[d] = fminf(mn[d], __shfl_xor(mn[d], o));
                mx[d] = fmaxf(mx[d], __shfl_xor(mx[d], o));
            }
    }
    __device__ __forceinline__ Part part() const
    {
        Part o;
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            o.s1[d] = s1[d];
            o.sq[d] = sq[d];
            o.mn[d] = mn[d];
            o.mx[d] = mx[d];
        }
        return o;
    }
};

// the work group's statistics from its threads': waves by butterfly, then the waves in order
__device__ __forceinline__ void block_part(Stat& s, Part* shared, Part* out)
{
    constexpr int W = kChunkThreads / 64;
    s.wave_reduce();
    __syncthreads();
    if ((threadIdx.x & 63) == 0) shared[threadIdx.x >> 6] = s.part();
    __syncthreads();
    if (threadIdx.x == 0) {
        Stat t;
        for (int q = 0; q < W; ++q) t.merge(shared[q]);
        *out = t.part();
    }
}

// the records of a thread in a chunk: wave w holds the chunk's records [512 w, 512 (w + 1)),
// lane l of step it record 512 w + 64 it + l (a record past the end is the last one again)
__device__ __forceinline__ void load_chunk(const float4* __restrict__ p, int32_t n, float4 (&r)[kChunkItems])
{
    const int first = (threadIdx.x >> 6) * (64 * kChunkItems) + (threadIdx.x & 63);
#pragma unroll
    for (int it = 0; it < kChunkItems; ++it)
        if (first - (int)(threadIdx.x & 63) + it * 64 < n) r[it] = p[min(first + it * 64, n - 1)];
}

__global__ __launch_bounds__(kChunkThreads) void chunk_stats_kernel(const float4* __restrict__ P, RoundBufs rb,
                                                                    const int32_t* __restrict__ ctl)
{
    __shared__ Part sh[kChunkThreads / 64];
    const int32_t n_items = ctl[kCtlItems];
    const int first = (threadIdx.x >> 6) * (64 * kChunkItems) + (threadIdx.x & 63);
    for (int32_t k = blockIdx.x; k < n_items; k += gridDim.x) {
        const Entry e = rb.entries[0][rb.items[0][k]];
        int32_t lo, hi;
        chunk_range(e, k - e.item0, lo, hi);
        float4 r[kChunkItems];
        load_chunk(P + e.start + lo, hi - lo, r);
        Stat s;
#pragma unroll
        for (int it = 0; it < kChunkItems; ++it)
            if (first + it * 64 < hi - lo) s.add(r[it]);
        block_part(s, sh, &rb.parts[0][k]);
    }
}

// goes right: the split of the tree's walk (FP32 coordinate against FP64 split)
__device__ __forceinline__ bool goes_right(const float4& p, int ax, double split)
{
    const float v = ax == 0 ? p.x : (ax == 1 ? p.y : p.z);
    return !((double)v < split);
}

// A round's first launch: every chunk's group sums its leaf's partial statistics (fixed
// order: a wave's partials by butterfly, then the waves in order; the records are on their
// way meanwhile), which gives the split at the
// mean of the axis of largest variance (lowest axis on ties), wanted only if samples fall
// on both sides; and counts its records on the right.
__global__ __launch_bounds__(kChunkThreads) void count_kernel(const float4* __restrict__ P0, const float4* __restrict__ P1,
                                                              RoundBufs rb, int par, const int32_t* __restrict__ ctl)
{
    constexpr int W = kChunkThreads / 64;
    __shared__ Part sh[W];
    __shared__ int ax_s, want_s, right_s;
    __shared__ double split_s;
    const int32_t n_items = ctl[kCtlItems + par];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int first = w * (64 * kChunkItems) + lane;
    for (int32_t k = blockIdx.x; k < n_items; k += gridDim.x) {
        const int32_t ei = rb.items[par][k];
        const Entry e = rb.entries[par][ei];
        int32_t lo, hi;
        chunk_range(e, k - e.item0, lo, hi);
        const int32_t n = hi - lo;
        float4 r[kChunkItems];
        load_chunk((e.src ? P1 : P0) + e.start + lo, n, r);
        const int32_t pn = e.pn2 >> 1;
        const Part* parts = rb.parts[par] + (int64_t)(e.pn2 & 1) * rb.max_items + e.pfirst;
        Stat s;
        if (w * 64 < pn) {  // the same in every lane of the wave
            for (int32_t j = threadIdx.x; j < pn; j += kChunkThreads) s.merge(parts[j]);
            s.wave_reduce();
        }
        __syncthreads();  // the previous item's shared words have been read
        if (w > 0 && w * 64 < pn && lane == 0) sh[w] = s.part();
        if (pn > 64) __syncthreads();  // the same in every thread
        if (w == 0) {
            if (lane == 0) {
                for (int q = 1; q < W && q * 64 < pn; ++q) s.merge(sh[q]);
                const double M = (double)e.count;
                int ax = 0;
                double best = -1.0;
#pragma unroll
                for (int d = 0; d < 3; ++d) {
                    const double mean = s.s1[d] / M;
                    const double var = s.sq[d] / M - mean * mean;
                    if (var > best) {
                        best = var;
                        ax = d;
                    }
                }
                const double split = (ax == 0 ? s.s1[0] : (ax == 1 ? s.s1[1] : s.s1[2])) / M;
                const float mn = ax == 0 ? s.mn[0] : (ax == 1 ? s.mn[1] : s.mn[2]);
                const float mx = ax == 0 ? s.mx[0] : (ax == 1 ? s.mx[1] : s.mx[2]);
                const int want = ((double)mn < split && split <= (double)mx) ? 1 : 0;
                ax_s = ax;
                split_s = split;
                want_s = want;
                right_s = 0;
                if (k == e.item0) {
                    rb.ax[ei] = ax;
                    rb.split[ei] = split;
                    rb.flags[ei] = want;
                }
            }
        }
        __syncthreads();
        const int ax = ax_s;
        const double split = split_s;
        int c = 0;
#pragma unroll
        for (int it = 0; it < kChunkItems; ++it)
            c += __popcll(__ballot(first + it * 64 < n && goes_right(r[it], ax, split)));
        if (lane == 0 && c) atomicAdd(&right_s, c);
        __syncthreads();
        if (threadIdx.x == 0 && want_s) {
            rb.item_right[k] = right_s;
            if (right_s) atomicAdd(&rb.rtot[par][ei], right_s);
        }
    }
}

// A round's last launch: the chunks of the leaves that split are partitioned, stably, from
// one record buffer into the other (left samples from the segment's start, right ones
// after all left ones); a child that may split in its turn gets its partial statistics
// here, while the records are in registers.
__global__ __launch_bounds__(kChunkThreads) void partition_kernel(float4* __restrict__ P0, float4* __restrict__ P1,
                                                                  RoundBufs rb, int par,
                                                                  const int32_t* __restrict__ ctl)
{
    __shared__ Part sh[kChunkThreads / 64];
    __shared__ int32_t before_s, wr[kChunkThreads / 64];
    const int32_t n_items = ctl[kCtlItems + par];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const uint64_t lt = lane ? (~0ull >> (64 - lane)) : 0ull;
    const int first = w * (64 * kChunkItems) + lane;
    for (int32_t k = blockIdx.x; k < n_items; k += gridDim.x) {
        const int32_t ei = rb.items[par][k];
        const int fl = rb.flags[ei];
        if (!(fl & 1)) continue;  // the same in every thread
        const Entry e = rb.entries[par][ei];
        const int ax = rb.ax[ei];
        const double split = rb.split[ei];
        const int32_t n_left = e.count - rb.rtot[par][ei];
        int32_t lo, hi;
        chunk_range(e, k - e.item0, lo, hi);
        const int32_t n = hi - lo;
        float4 r[kChunkItems];
        load_chunk((e.src ? P1 : P0) + e.start + lo, n, r);
        __syncthreads();  // the previous item's shared words have been read
        if (w == 0) {  // the leaf's right samples in earlier chunks
            int32_t b = 0;
            for (int32_t j = e.item0 + lane; j < k; j += 64) b += rb.item_right[j];
#pragma unroll
            for (int o = 1; o < 64; o <<= 1) b += __shfl_xor(b, o);
            if (lane == 0) before_s = b;
        }
        uint64_t m[kChunkItems];
        int c = 0;
#pragma unroll
        for (int it = 0; it < kChunkItems; ++it) {
            m[it] = __ballot(first + it * 64 < n && goes_right(r[it], ax, split));
            c += __popcll(m[it]);
        }
        if (lane == 0) wr[w] = c;
        __syncthreads();
        int32_t rights = before_s;
        for (int q = 0; q < w; ++q) rights += wr[q];
        float4* out = (e.src ? P0 : P1) + e.start;
#pragma unroll
        for (int it = 0; it < kChunkItems; ++it) {
            const int32_t at = first + it * 64;  // index in the chunk
            const int32_t rb4 = rights + __popcll(m[it] & lt);
            if (at < n) {
                const bool right = (m[it] >> lane) & 1;
                out[right ? n_left + rb4 : lo + at - rb4] = r[it];
            }
            rights += __popcll(m[it]);
        }
#pragma unroll
        for (int side = 0; side < 2; ++side) {
            if (!(fl & (2 << side))) continue;
            Stat s;
#pragma unroll
            for (int it = 0; it < kChunkItems; ++it)
                if (first + it * 64 < n && (int)((m[it] >> lane) & 1) == side) s.add(r[it]);
            block_part(s, sh, &rb.parts[par ^ 1][(int64_t)side * rb.max_items + k]);
        }
    }
}

// ---------------------------------------------------------------------------------
// A round's decisions, by one work group, over the round's list (its leaves in increasing
// order): the wanted splits are numbered by a block prefix sum, those beyond the node or
// leaf capacity are skipped (status bit 1); the tree, the boxes and the leaf tables are
// updated, and the next round's list takes the children with more than c samples, the left
// ones (which keep their parents' indices) before the right ones, which is their order.
// The launch is one chain of memory round trips, so everything that only needs an entry is
// loaded before the block scan, and one scan (of two packed words) numbers the splits and
// both children's entries and work items, unless the capacity cuts the splits off: then the
// children are scanned again. A round's decision takes 4.6 us for 60 leaves and 5.4 for 600
// (12 and 16 with each value loaded where it is used and three scans).
// Up to 1024 entries (one per thread) take one pass; a longer list takes a first pass over
// its tiles for the number of left children, whose entries come before the right ones'.
// ---------------------------------------------------------------------------------
__global__ __launch_bounds__(1024) void split_decide_kernel(TreePtrs t, RoundBufs rb, int par, int32_t c, LeafTabs lt,
                                                            int32_t* __restrict__ ctl)
{
    __shared__ int64_t ws[2][2][16];
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int32_t n = ctl[kCtlEntries + par];
    const int32_t nodes = t.counts[0], leaves = t.counts[1];
    if (n == 0) {  // the same in every thread
        if (tid == 0) ctl[kCtlEntries + (par ^ 1)] = ctl[kCtlItems + (par ^ 1)] = 0;
        return;
    }
    const int32_t cap = max(0, min((t.max_nodes - nodes) / 2, t.max_leaves - leaves));
    int parity = 0;  // of the scans: consecutive ones use different shared words
    // exclusive prefix sums of a and b over the work group, and their totals; one barrier
    auto scan2 = [&](int64_t& a, int64_t& b, int64_t& a_all, int64_t& b_all) {
        int64_t x = a, y = b;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const int64_t xo = __shfl_up(x, o), yo = __shfl_up(y, o);
            if (lane >= o) {
                x += xo;
                y += yo;
            }
        }
        if (lane == 63) {
            ws[parity][0][w] = x;
            ws[parity][1][w] = y;
        }
        __syncthreads();
        int64_t xb = 0, yb = 0;
        a_all = b_all = 0;
#pragma unroll
        for (int q = 0; q < 16; ++q) {
            const int64_t sx = ws[parity][0][q], sy = ws[parity][1][q];
            xb += q < w ? sx : 0;
            yb += q < w ? sy : 0;
            a_all += sx;
            b_all += sy;
        }
        parity ^= 1;
        a = xb + x - a;
        b = yb + y - b;
    };
    // a packed word: (entries << 32) + work items of the children of one side; the wanted
    // splits ride above the left children's entries (at most 1024 of each per tile)
    constexpr int kWantShift = 48;
    constexpr int64_t kLeftMask = (int64_t(1) << kWantShift) - 1;
    int32_t total = 0;
    int64_t lefts = 0, rights = 0;
    const int passes = n <= 1024 ? 1 : 2;
    for (int pass = 0; pass < passes; ++pass) {
        const bool write = pass == passes - 1;
        int64_t lrun = 0, rrun = lefts;
        total = 0;
        for (int32_t e0 = 0; e0 < n; e0 += 1024) {
            const int32_t ei = e0 + tid;
            const bool in = ei < n;
            Entry e{};
            int32_t want = 0, nr = 0, ax = 0, nd = 0, init = 0, origin = 0, next = 0;
            double sp = 0.0, lo[3] = {0, 0, 0}, hi[3] = {0, 0, 0};
            if (in) {
                e = rb.entries[par][ei];
                want = rb.flags[ei] & 1;
                nr = rb.rtot[par][ei];
                ax = rb.ax[ei];
                sp = rb.split[ei];
                nd = t.leaf_node[e.leaf];
                init = t.init[e.leaf];
                origin = lt.origin[e.leaf];
                next = lt.next[e.leaf];
#pragma unroll
                for (int d = 0; d < 3; ++d) {
                    lo[d] = t.lo[3 * e.leaf + d];
                    hi[d] = t.hi[3 * e.leaf + d];
                }
            }
            const int32_t nl = e.count - nr;
            auto left = [&](bool go) { return go && nl > c ? (int64_t(1) << 32) | chunks_of(nl, kChunk) : int64_t(0); };
            auto right = [&](bool go) { return go && nr > c ? (int64_t(1) << 32) | chunks_of(nr, kChunk) : int64_t(0); };
            int64_t a = left(want) | ((int64_t)want << kWantShift), b = right(want), a_all, b_all;
            scan2(a, b, a_all, b_all);
            const int32_t rk = total + (int32_t)(a >> kWantShift), wants = (int32_t)(a_all >> kWantShift);
            const bool go = want && rk < cap;
            if (total + wants > cap) {  // the same in every thread
                a = left(go);
                b = right(go);
                scan2(a, b, a_all, b_all);
            }
            total += wants;
            a_all &= kLeftMask;
            a = (a & kLeftMask) + lrun;
            lrun += a_all;
            if (passes == 1) rrun = a_all;
            b += rrun;
            rrun += b_all;
            if (!write || !in) continue;
            const bool lgo = go && nl > c, rgo = go && nr > c;
            rb.flags[ei] = go ? 1 | (lgo ? 2 : 0) | (rgo ? 4 : 0) : 0;
            if (!go) continue;
            const int32_t l = e.leaf, r = leaves + rk, Ln = nodes + 2 * rk;
            t.axis[nd] = ax;
            t.split[nd] = sp;
            t.left[nd] = Ln;
            t.leaf[nd] = -1;
            for (int q = 0; q < 2; ++q) {
                t.axis[Ln + q] = -1;
                t.left[Ln + q] = -1;
                t.split[Ln + q] = 0.0;
            }
            t.leaf[Ln] = l;
            t.leaf[Ln + 1] = r;
            t.leaf_node[l] = Ln;
            t.leaf_node[r] = Ln + 1;
#pragma unroll
            for (int d = 0; d < 3; ++d) {
                t.lo[3 * r + d] = d == ax ? sp : lo[d];
                t.hi[3 * r + d] = hi[d];
            }
            t.hi[3 * l + ax] = sp;
            t.init[r] = init;
            lt.origin[r] = origin;
            lt.next[r] = next;
            lt.next[l] = r;
            lt.count[l] = nl;
            lt.start[r] = e.start + nl;
            lt.count[r] = nr;
            lt.par[l] = lt.par[r] = e.src ^ 1;
#pragma unroll
            for (int side = 0; side < 2; ++side) {
                if (!(side ? rgo : lgo)) continue;
                const int64_t at = side ? b : a;
                const int32_t en = (int32_t)(at >> 32), it = (int32_t)at, cnt = side ? nr : nl, nch = chunks_of(cnt, kChunk);
                rb.entries[par ^ 1][en] = Entry{side ? r : l, side ? e.start + nl : e.start, cnt, e.src ^ 1, it, nch,
                                                e.item0, 2 * e.nch + side};
                rb.rtot[par ^ 1][en] = 0;
                for (int32_t q = 0; q < nch; ++q) rb.items[par ^ 1][it + q] = en;
            }
        }
        lefts = lrun;
        rights = rrun;
    }
    __syncthreads();  // every thread has read the counts
    if (tid == 0) {
        const int32_t n_split = min(total, cap);
        t.counts[0] = nodes + 2 * n_split;
        t.counts[1] = leaves + n_split;
        ctl[kCtlEntries + (par ^ 1)] = (int32_t)(rights >> 32);
        ctl[kCtlItems + (par ^ 1)] = (int32_t)rights;
        ctl[kCtlStatus] |= total > n_split ? 1 : 0;
        ctl[kCtlLeaves] = leaves + n_split;
    }
}

// After the last round (each kernel below leaves at once while a leaf is left to split):
// off[l] = first output position of leaf l, off[L] = N, by one work group.
__global__ __launch_bounds__(1024) void offsets_kernel(const int32_t* __restrict__ ctl, int done, LeafTabs lt,
                                                       int64_t* __restrict__ off)
{
    __shared__ int64_t ws[16];
    if (!finished(ctl, done)) return;
    const int32_t L = ctl[kCtlLeaves];
    int64_t run = 0;
    for (int32_t l0 = 0; l0 < L; l0 += 1024) {
        const int32_t l = l0 + (int32_t)threadIdx.x;
        int64_t all;
        const int64_t x = run + block_scan_1024<int64_t>(l < L ? lt.count[l] : 0, ws, all);
        if (l < L) off[l] = x;
        run += all;
    }
    if (threadIdx.x == 0) off[L] = run;
}

// every leaf marks the multiples of kCover in its segment as its own, and a new leaf copies
// the mixture and state of the leaf it was split from
__global__ void copy_leaves_kernel(int32_t L0, const int32_t* __restrict__ ctl, int done, LeafTabs lt, int K,
                                   MixPtrs mix, StatePtrs st)
{
    if (!finished(ctl, done)) return;
    const int32_t L = ctl[kCtlLeaves];
    for (int64_t r = blockIdx.x; r < L; r += gridDim.x) {
        const int64_t a = lt.start[r], b = a + lt.count[r];
        for (int64_t t = (a + kCover - 1) / kCover + threadIdx.x; t * kCover < b; t += blockDim.x)
            lt.cover[t] = (int32_t)r;
        if (r < L0) continue;
        const int64_t l = lt.origin[r];
        for (int q = threadIdx.x; q < 38 * K + 2; q += blockDim.x) {
            if (q < K) mix.pi[r * K + q] = mix.pi[l * K + q];
            else if (q < 4 * K) mix.mud[r * 3 * K + q - K] = mix.mud[l * 3 * K + q - K];
            else if (q < 7 * K) mix.mux[r * 3 * K + q - 4 * K] = mix.mux[l * 3 * K + q - 4 * K];
            else if (q < 22 * K) mix.cov[r * 15 * K + q - 7 * K] = mix.cov[l * 15 * K + q - 7 * K];
            else if (q < 23 * K) st.s0[r * K + q - 22 * K] = st.s0[l * K + q - 22 * K];
            else if (q < 38 * K) st.s2[r * 15 * K + q - 23 * K] = st.s2[l * 15 * K + q - 23 * K];
            else if (q == 38 * K) st.sw[r] = st.sw[l];
            else st.step[r] = st.step[l];
        }
    }
}

// The samples in the order of the leaf indices: positions from the leaves' segments,
// directions and weights by the index that travelled with them, which lies in the segment
// of the leaf they started in. The waves follow the records, not the output, so that the
// leaves split from one leaf are written at about the same time and their directions and
// weights are read from a window that stays in cache (16.6M samples: 270-300 us, 361 us in output
// order). A wave's kCover records start in a marked leaf; the next ones follow it, kFollow
// leaves at most: the leaves of a fine tree are small or empty, and each one is two memory
// round trips. Then a lane searches for its record's leaf of before the refinement, whose
// starts are in order and stay as they were through the splits, and follows from there.
// 1000 samples in a tree of 262,144 leaves took 47.7 ms leaf by leaf.
constexpr int kFollow = 8;

__global__ __launch_bounds__(256) void gather_kernel(const int32_t* __restrict__ ctl, int done, int64_t N, int32_t L0, LeafTabs lt,
                                                     const int64_t* __restrict__ off, const float4* __restrict__ P0,
                                                     const float4* __restrict__ P1, const float4* __restrict__ Q,
                                                     float* __restrict__ out)
{
    if (!finished(ctl, done)) return;
    constexpr int U = kCover / 64;
    const int64_t wave = xcd_block_order(blockIdx.x, gridDim.x) * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t i0 = wave * kCover;
    if (i0 >= N) return;
    int32_t l = lt.cover[wave];
    int32_t a = lt.start[l], b = a + lt.count[l];
    float4 p[U], q[U];
    int64_t j[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int64_t i = min(i0 + u * 64 + (threadIdx.x & 63), N - 1);
        for (int step = 1; i >= b; ++step) {  // the segments cover [0, N), so some leaf holds record i
            l = lt.next[l];
            if (step == kFollow) {
                int32_t lo = 0, hi = L0;  // start[lo] <= i < start[hi]
                while (hi - lo > 1) {
                    const int32_t mid = lo + (hi - lo) / 2;
                    if (lt.start[mid] <= i) lo = mid;
                    else hi = mid;
                }
                if (lt.start[lo] >= b) l = lo;  // else the record's leaf was split and l follows it
            }
            a = lt.start[l];
            b = a + lt.count[l];
        }
        p[u] = (lt.par[l] ? P1 : P0)[i];
        j[u] = off[l] + (i - a);
    }
#pragma unroll
    for (int u = 0; u < U; ++u) q[u] = Q[__float_as_int(p[u].w)];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        if (i0 + u * 64 + (threadIdx.x & 63) >= N) continue;
        out[j[u]] = q[u].x;
        out[N + j[u]] = q[u].y;
        out[2 * N + j[u]] = q[u].z;
        out[3 * N + j[u]] = p[u].x;
        out[4 * N + j[u]] = p[u].y;
        out[5 * N + j[u]] = p[u].z;
        out[6 * N + j[u]] = q[u].w;
    }
}

// Initial mixture of an uninitialised leaf with at least min_init samples, one thread
// per component: n_dir = min(8, K) directions at the cube vertices (signs of x, y, z,
// positive first), n_pos = ceil(K / n_dir) positions along the longest sides (two:
// centre -+ d/4; four: a 2x2 pattern; more: evenly), directional variance 2 pi / 8,
// positional variance r^2 / chi2_3^-1(0.9) with r = 2 d / n_pos, weights 1/K; the
// Robbins-Monro state starts at zero.
__device__ __forceinline__ void init_leaf(const TreePtrs& t, int32_t l, int K, const MixPtrs& mix, const StatePtrs& st)
{
    const double chi2_3_inv_090 = 6.251388631170325;
    const int n_dir = K < 8 ? K : 8;
    const int n_pos = (K + n_dir - 1) / n_dir;
    double size[3], centre[3], d = 0.0;
    for (int a = 0; a < 3; ++a) {
        size[a] = t.hi[3 * l + a] - t.lo[3 * l + a];
        centre[a] = t.lo[3 * l + a] + 0.5 * size[a];
        d = fmax(d, size[a]);
    }
    int order[3] = {0, 1, 2};
    for (int i = 1; i < 3; ++i)
        for (int j = i; j > 0 && size[order[j]] > size[order[j - 1]]; --j) {
            const int tmp = order[j];
            order[j] = order[j - 1];
            order[j - 1] = tmp;
        }
    const double r = 2.0 * d / n_pos;
    const double inv_sqrt3 = 1.0 / sqrt(3.0);
    for (int k = threadIdx.x; k < K; k += blockDim.x) {
        const int s = k / n_dir, v = k % n_dir;
        double o[3] = {0.0, 0.0, 0.0};
        if (n_pos == 2) {
            o[order[0]] = (s == 0 ? -1.0 : 1.0) * d / 4.0;
        } else if (n_pos == 4) {
            o[order[0]] = (s % 2 == 0 ? -1.0 : 1.0) * d / 4.0;
            o[order[1]] = (s / 2 == 0 ? -1.0 : 1.0) * d / 4.0;
        } else if (n_pos > 1) {
            o[order[0]] = ((s + 0.5) / n_pos - 0.5) * d;
        }
        const int64_t g = (int64_t)l * K + k;
        for (int a = 0; a < 3; ++a) mix.mux[3 * g + a] = centre[a] + o[a];
        mix.mud[3 * g + 0] = ((v >> 2) & 1 ? -1.0 : 1.0) * inv_sqrt3;
        mix.mud[3 * g + 1] = ((v >> 1) & 1 ? -1.0 : 1.0) * inv_sqrt3;
        mix.mud[3 * g + 2] = (v & 1 ? -1.0 : 1.0) * inv_sqrt3;
        for (int q = 0; q < 15; ++q) mix.cov[15 * g + q] = 0.0;
        mix.cov[15 * g + tri(0, 0)] = mix.cov[15 * g + tri(1, 1)] = 2.0 * kPi / 8.0;
        for (int a = 0; a < 3; ++a) mix.cov[15 * g + tri(2 + a, 2 + a)] = r * r / chi2_3_inv_090;
        mix.pi[g] = 1.0 / K;
        st.s0[g] = 0.0;
        for (int q = 0; q < 15; ++q) st.s2[15 * g + q] = 0.0;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        st.sw[l] = 0.0;
        st.step[l] = 0;
        t.init[l] = 1;
    }
}

__global__ void init_leaves_kernel(TreePtrs t, const int32_t* __restrict__ ctl, int done, const int64_t* __restrict__ off,
                                   int32_t min_init, int K, MixPtrs mix, StatePtrs st)
{
    if (!finished(ctl, done)) return;
    const int32_t L = ctl[kCtlLeaves];
    for (int32_t l = blockIdx.x; l < L; l += gridDim.x)
        if (!t.init[l] && off[l + 1] - off[l] >= min_init) init_leaf(t, l, K, mix, st);
}

// workspace of a refinement
struct TreeLayout {
    size_t keys[2], p[2], q[2], hist, gsum, total_bins, start, count, par, next, origin, cover, entries[2], items[2], rtot[2],
        parts[2], item_right, flags, ax, split, ctl, total;
    int tiles, groups;
    int32_t max_items;
};

inline TreeLayout tree_layout(int64_t N, int32_t max_leaves)
{
    TreeLayout L{};
    const int64_t n = N > 0 ? N : 1;
    const int64_t bins = std::min<int64_t>(max_leaves, kMaxBins);
    const bool passes = max_leaves > kMaxBins;  // more than one sorting pass may run
    L.tiles = (int)((n + kSortTile - 1) / kSortTile);
    L.groups = (L.tiles + kScanRows - 1) / kScanRows;
    // a round's leaves are disjoint and not empty; each has one partly filled chunk at most
    const int64_t leaves = std::min<int64_t>(max_leaves, n);
    L.max_items = (int32_t)(n / kChunk + leaves);
    size_t p = 0;
    auto take = [&](size_t bytes) {
        const size_t at = p;
        p = align256(p + bytes);
        return at;
    };
    L.keys[0] = take(n * 4);
    L.keys[1] = passes ? take(n * 4) : L.keys[0];
    for (int b = 0; b < 2; ++b) L.p[b] = take(n * 16);
    L.q[0] = take(n * 16);
    L.q[1] = passes ? take(n * 16) : L.q[0];
    L.hist = take((size_t)bins * L.tiles * 4);
    L.gsum = take((size_t)bins * L.groups * 4);
    L.total_bins = take((size_t)bins * 4);
    L.start = take(((size_t)max_leaves + 1) * 4);
    L.count = take((size_t)max_leaves * 4);
    L.par = take((size_t)max_leaves * 4);
    L.next = take((size_t)max_leaves * 4);
    L.origin = take((size_t)max_leaves * 4);
    L.cover = take((size_t)((n + kCover - 1) / kCover) * 4);
    for (int b = 0; b < 2; ++b) {
        L.entries[b] = take((size_t)leaves * sizeof(Entry));
        L.items[b] = take((size_t)L.max_items * 4);
        L.rtot[b] = take((size_t)leaves * 4);
        L.parts[b] = take((size_t)L.max_items * 2 * sizeof(Part));
    }
    L.item_right = take((size_t)L.max_items * 4);
    L.flags = take((size_t)leaves * 4);
    L.ax = take((size_t)leaves * 4);
    L.split = take((size_t)leaves * 8);
    L.ctl = take(kCtlWords * 4);
    L.total = p;
    return L;
}

static TreePtrs tree_ptrs(const sdmm_tree* t)
{
    return TreePtrs{t->max_nodes, t->max_leaves, t->counts, t->axis, t->left, t->leaf, t->split,
                    t->leaf_node, t->lo, t->hi, t->init};
}

static bool tree_ok(const sdmm_tree* t)
{
    return t && t->max_leaves >= 1 && t->max_nodes >= 2 * t->max_leaves - 1 && t->counts && t->axis && t->left &&
           t->leaf && t->split && t->leaf_node && t->lo && t->hi && t->init;
}

static inline unsigned blocks_for(int64_t n, int per) { return (unsigned)std::max<int64_t>(1, (n + per - 1) / per); }

}  // namespace sdmm

using namespace sdmm;

extern "C" int sdmm_tree_init(const sdmm_tree* tree, int32_t depth, const double* lo, const double* hi, void* stream)
{
    if (!tree_ok(tree) || !lo || !hi || depth < 0 || depth > 6) return SDMM_EINVAL;
    const int levels = 3 * depth;
    const int64_t n_leaves = int64_t(1) << levels, n_nodes = 2 * n_leaves - 1;
    if (n_leaves > tree->max_leaves || n_nodes > tree->max_nodes) return SDMM_EINVAL;
    for (int d = 0; d < 3; ++d)
        if (!(lo[d] < hi[d])) return SDMM_EINVAL;
    hipStream_t s = reinterpret_cast<hipStream_t>(stream);
    tree_init_kernel<<<blocks_for(n_nodes, 256), 256, 0, s>>>(tree_ptrs(tree), levels, lo[0], lo[1], lo[2], hi[0],
                                                             hi[1], hi[2]);
    return check(hipGetLastError());
}

extern "C" size_t sdmm_tree_workspace_size(int64_t n_samples, int32_t max_leaves)
{
    if (n_samples < 0 || max_leaves < 1) return 0;
    return tree_layout(n_samples, max_leaves).total;
}

extern "C" int sdmm_tree_refine(const sdmm_tree* tree, const float* samples, int64_t n_samples,
                                int32_t split_threshold, int32_t min_init, const sdmm_mixtures* mix,
                                const sdmm_em_state* state, float* sorted_out, int64_t* cell_offsets_out,
                                int32_t* n_leaves_out, int32_t* status_out, void* workspace,
                                size_t workspace_bytes, void* stream)
{
    if (!tree_ok(tree) || n_samples < 0 || (n_samples > 0 && (!samples || !sorted_out)) || split_threshold < 1 ||
        min_init < 0 || !mix || !state || !cell_offsets_out || !n_leaves_out || !workspace)
        return SDMM_EINVAL;
    if (n_samples > INT32_MAX) return SDMM_EINVAL;  // sample indices are int32
    if (mix->n_cells != tree->max_leaves || mix->K < 1 || mix->K > kMaxK || !mix->weights || !mix->mean_dir ||
        !mix->mean_pos || !mix->cov || !state->s0 || !state->s2 || !state->sw || !state->step)
        return SDMM_EINVAL;
    const int64_t N = n_samples;
    const TreeLayout TL = tree_layout(N, tree->max_leaves);
    if (workspace_bytes < TL.total) return SDMM_ENOWORKSPACE;
    hipStream_t s = reinterpret_cast<hipStream_t>(stream);
    char* ws = reinterpret_cast<char*>(workspace);
    auto i32 = [&](size_t at) { return reinterpret_cast<int32_t*>(ws + at); };
    auto f4 = [&](size_t at) { return reinterpret_cast<float4*>(ws + at); };
    int32_t *hist = i32(TL.hist), *gsum = i32(TL.gsum), *bin_total = i32(TL.total_bins), *ctl = i32(TL.ctl);
    float4 *P0 = f4(TL.p[0]), *P1 = f4(TL.p[1]);
    const LeafTabs lt{i32(TL.start), i32(TL.count), i32(TL.par), i32(TL.next), i32(TL.origin), i32(TL.cover)};
    RoundBufs rb;
    for (int b = 0; b < 2; ++b) {
        rb.entries[b] = reinterpret_cast<Entry*>(ws + TL.entries[b]);
        rb.items[b] = i32(TL.items[b]);
        rb.rtot[b] = i32(TL.rtot[b]);
        rb.parts[b] = reinterpret_cast<Part*>(ws + TL.parts[b]);
    }
    rb.item_right = i32(TL.item_right);
    rb.flags = i32(TL.flags);
    rb.ax = i32(TL.ax);
    rb.split = reinterpret_cast<double*>(ws + TL.split);
    rb.max_items = TL.max_items;
    const TreePtrs tp = tree_ptrs(tree);
    const MixPtrs mp{mix->weights, mix->mean_dir, mix->mean_pos, mix->cov};
    const StatePtrs sp{state->s0, state->s2, state->sw, state->step};
    const int K = mix->K;
    int rc;

    // the words read back land in pinned memory (a pageable destination would be staged by
    // the runtime), one buffer per host thread, kept for its lifetime
    thread_local int32_t* pinned = nullptr;
    if (!pinned && (rc = check(hipHostMalloc((void**)&pinned, kCtlWords * sizeof(int32_t), hipHostMallocPortable)))) {
        pinned = nullptr;
        return rc;
    }
    auto read_back = [&](const int32_t* from, int n) {
        const int e = check(hipMemcpyAsync(pinned, from, n * sizeof(int32_t), hipMemcpyDeviceToHost, s));
        return e ? e : check(hipStreamSynchronize(s));
    };

    // the location needs no leaf count on the host, so the GPU works on it while the host
    // waits for the tree's counts. Only the workspace is written before they are checked.
    {  // timed
        ScopedTimer tm(SDMM_TIMER_TREE, s);
        if (N > 0)
            locate_kernel<<<std::min<unsigned>((unsigned)TL.tiles, kLocMaxGroups), kLocThreads, 0, s>>>(
                tp, samples, N, i32(TL.keys[0]), hist, TL.tiles);
    }
    if ((rc = read_back(tree->counts, 2))) return rc;
    const int32_t L0 = pinned[1];
    if (L0 < 1 || L0 > tree->max_leaves || pinned[0] < 1 || pinned[0] > tree->max_nodes) return SDMM_EINVAL;

    // one leaf that will not split keeps its samples as they are, and their order: the output
    // is a copy (8M samples: 310 us through the records and the gather)
    const bool as_is = L0 == 1 && N <= split_threshold;
    // the stable sort by leaf: one pass up to kMaxBins leaves, which leaves the leaf tables
    // and the first round's list behind; more leaves take more passes
    int passes = 1;
    while (passes < 3 && (int64_t(1) << (passes * kDigitBits)) < L0) ++passes;
    for (int p = 0; p < passes && N > 0; ++p) {
        const int shift = p * kDigitBits;
        const int bins = (int)std::min<int64_t>(kMaxBins, ((int64_t)L0 + (int64_t(1) << shift) - 1) >> shift);
        int bits = 1;
        while ((1 << bits) < bins) ++bits;
        const int32_t* kin = i32(TL.keys[p & 1]);
        int32_t* kout = passes > 1 ? i32(TL.keys[(p & 1) ^ 1]) : nullptr;
        const int to = (passes - 1 - p) & 1;  // the last pass ends in buffer 0
        if (p > 0) tile_hist_kernel<<<TL.tiles, kSortThreads, 0, s>>>(kin, N, shift, bins, hist);
        scan_group_kernel<<<dim3((bins + 255) / 256, TL.groups), 256, 0, s>>>(hist, TL.tiles, bins, gsum);
        scan_bins_kernel<<<(bins + 63) / 64, 64, 0, s>>>(gsum, TL.groups, bins, bin_total);
        base_kernel<<<1, 1024, 0, s>>>(bin_total, bins, passes == 1 ? 1 : 0, L0, split_threshold, lt, rb, ctl);
        const bool staged = bins <= kStageBins;
        const size_t lds = staged ? 0 : (size_t)bins * (4 + 2 * kSortWaves);
        const auto move = p == 0 ? (staged ? scatter_kernel<true, true> : scatter_kernel<true, false>)
                                 : (staged ? scatter_kernel<false, true> : scatter_kernel<false, false>);
        if (!as_is)
            move<<<TL.tiles, kSortThreads, lds, s>>>(samples, f4(TL.p[to ^ 1]), f4(TL.q[to ^ 1]), kin, N, shift, bins, bits,
                                                     hist, gsum, bin_total, f4(TL.p[to]), f4(TL.q[to]), kout);
    }
    if (passes > 1 || N == 0) {
        if (N > 0)
            starts_kernel<<<blocks_for(N, 256), 256, 0, s>>>(i32(TL.keys[passes & 1]), N, L0, lt.start);
        else if ((rc = check(hipMemsetAsync(lt.start, 0, ((size_t)L0 + 1) * 4, s))))
            return rc;
        base_kernel<<<1, 1024, 0, s>>>(bin_total, 0, 1, L0, split_threshold, lt, rb, ctl);
    }

    // rounds, queued in groups: as many as the mean leaf would take to come down to the
    // threshold and three more for the uneven ones (a round with an empty list costs three
    // small launches, a wait for the host about 20 us), then what is left in groups of four.
    // The launches that end the refinement follow each group and leave at once while a leaf
    // is left to split.
    const int64_t bound = N / kChunk + std::min<int64_t>(tree->max_leaves, N / ((int64_t)split_threshold + 1));
    const unsigned groups = (unsigned)std::min<int64_t>(std::max<int64_t>(bound, 1), 4096);
    if (N > split_threshold) chunk_stats_kernel<<<groups, kChunkThreads, 0, s>>>(P0, rb, ctl);
    int ahead = 3;
    while (ahead < 12 && ((int64_t)split_threshold * L0 << (ahead - 3)) < N) ++ahead;
    if (N <= split_threshold) ahead = 0;
    for (int round = 0;;) {
        for (const int end = std::min(kMaxRounds, round + ahead); round < end; ++round) {
            const int par = round & 1;
            count_kernel<<<groups, kChunkThreads, 0, s>>>(P0, P1, rb, par, ctl);
            split_decide_kernel<<<1, 1024, 0, s>>>(tp, rb, par, split_threshold, lt, ctl);
            partition_kernel<<<groups, kChunkThreads, 0, s>>>(P0, P1, rb, par, ctl);
        }
        const int done = round >= kMaxRounds ? 2 : round & 1;
        offsets_kernel<<<1, 1024, 0, s>>>(ctl, done, lt, cell_offsets_out);
        copy_leaves_kernel<<<std::min(tree->max_leaves, 2048), 64, 0, s>>>(L0, ctl, done, lt, K, mp, sp);
        if (as_is) {
            if (N > 0 && (rc = check(hipMemcpyAsync(sorted_out, samples, (size_t)N * 7 * sizeof(float),
                                                    hipMemcpyDeviceToDevice, s))))
                return rc;
        } else if (N > 0) {
            gather_kernel<<<blocks_for(N, 4 * kCover), 256, 0, s>>>(ctl, done, N, L0, lt, cell_offsets_out, P0, P1,
                                                                    f4(TL.q[0]), sorted_out);
        }
        init_leaves_kernel<<<std::min(tree->max_leaves, 4096), 64, 0, s>>>(tp, ctl, done, cell_offsets_out, min_init, K,
                                                                           mp, sp);
        if ((rc = read_back(ctl, kCtlWords))) return rc;
        if (done == 2 || pinned[kCtlEntries + done] == 0) break;
        ahead = 4;
    }
    *n_leaves_out = pinned[kCtlLeaves];
    if (status_out) *status_out = pinned[kCtlStatus];
    return check(hipGetLastError());
}
