// Connectivity clean-up (Section 2, final step), under a canonical rule that
// a sequential implementation reproduces exactly:
//  1. 4-connected components of equal label, each named by its smallest
//     raster index (its root pixel);
//  2. component sizes;
//  3. a component below the size threshold, other than the one holding
//     pixel 0, joins the component of the pixel left of its root (above it
//     when the root starts a row); joins point to earlier roots, so they form
//     a forest;
//  4. each component takes its tree root's segment, and segments are
//     numbered 0.. in raster order of their roots.
//
// GPU structure: concurrent union-find whose links always point from a
// larger to a smaller index (so a tree's root is its minimum), first inside
// 32 x 32 tiles in LDS, then across tile borders in global memory; the joins
// of step 3 recorded per small root as links in the rank array and followed
// (with path splitting) by the relabel pass; ballot counts and prefix sums
// over the surviving roots for the numbering.  All integer, so the result
// is exact.
#include "ccl_tile.h"
#include "slic_internal.h"

namespace slic {
namespace {

constexpr int kBlock = 256;

__device__ __forceinline__ int load_relaxed(gmem<int>* p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ int atomic_min(gmem<int>* p, int v) {
    return __hip_atomic_fetch_min(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// The roots of a and b, the two walks advanced together so that their
// loads overlap.
__device__ __forceinline__ void find_roots(gmem<int>* P, int& a, int& b) {
    int pa = load_relaxed(P + a), pb = load_relaxed(P + b);
    while (pa != a || pb != b) {
        a = pa;
        b = pb;
        pa = load_relaxed(P + a);
        pb = load_relaxed(P + b);
    }
}

// Merge the trees of a and b, linking the larger root under the smaller.
// If another thread re-linked the root meanwhile, atomicMin returns that new
// parent and the merge continues from it.
__device__ void unite(gmem<int>* P, int a, int b) {
    bool done;
    do {
        find_roots(P, a, b);
        if (a < b) {
            const int old = atomic_min(P + b, a);
            done = old == b;
            b = old;
        } else if (b < a) {
            const int old = atomic_min(P + a, b);
            done = old == a;
            a = old;
        } else {
            done = true;
        }
    } while (!done);
}

// ---- components in three steps: union-find inside 32 x 32 tiles in LDS,
// unions across tile borders in global memory, then every pixel resolves its
// root and the tile adds its pixel counts per root.
constexpr int kTile = tile_ccl::kTile;
constexpr int kTilePx = tile_ccl::kTilePx;
constexpr int kPxPerThread = tile_ccl::kPxPerThread;
static_assert(kBlock == tile_ccl::kBlock, "the tile passes use the shared tile shape");

// The image of tile number idx of a launch and the tile's (x, y) among the
// image's 32 x 32 tiles: from the kernel argument (one image) or, for a
// batch, from the image table through the tile-to-image map.
__device__ __forceinline__ void resolve_tile(const CclImage& single, const CclMap& map, int idx,
                                             CclImage* g, int* bx, int* by) {
    int local = idx;
    if (map.images) {
        const int img = map.tile_image[idx];
        *g = map.images[img];
        local -= map.tile_first[img];
    } else {
        *g = single;
    }
    *bx = local % g->tiles_x;
    *by = local / g->tiles_x;
}

// The tile passes: one image on a two-dimensional grid of tiles (kBatch
// false: no table lookups and no division on the way in), or a batch on a
// one-dimensional grid through the map.
template <bool kBatch>
__device__ __forceinline__ void tile_of_launch(const CclImage& single, const CclMap& map,
                                               CclImage* g, int* bx, int* by) {
    if constexpr (kBatch) {
        resolve_tile(single, map, blockIdx.x, g, bx, by);
    } else {
        *g = single;
        *bx = blockIdx.x;
        *by = blockIdx.y;
    }
}

// Likewise for the passes over runs of kMergeBlock consecutive pixels.
template <bool kBatch>
__device__ __forceinline__ void resolve_block(const CclImage& single, const CclMap& map,
                                              CclImage* g, int* blk) {
    if constexpr (kBatch) {
        const int img = map.blk_image[blockIdx.x];
        *g = map.images[img];
        *blk = static_cast<int>(blockIdx.x) - map.blk_first[img];
    } else {
        *g = single;
        *blk = blockIdx.x;
    }
}

// Tile-local components of the association labels: the tile's labels into
// LDS, then tile_ccl::tile_components (P, lroot and the local roots' sizes).
// The association launch that ends a segmentation can do this itself for
// 32 x 32 tiles; the pass is then skipped.
template <bool kBatch>
__global__ __launch_bounds__(kBlock) void ccl_local_kernel(CclImage single, CclMap map) {
    __shared__ int lab[kTilePx];
    __shared__ int par[kTilePx];
    __shared__ int cnt[kTilePx];
    CclImage g;
    int bx, by;
    tile_of_launch<kBatch>(single, map, &g, &bx, &by);
    gmem<const int32_t>* __restrict__ labels = as_global(g.labels);
    gmem<int>* __restrict__ P = as_global(g.comp);
    gmem<int>* __restrict__ lroot = as_global(g.lroot);
    gmem<int>* __restrict__ size = as_global(g.size);
    const int w = g.w, h = g.h;
    const int x0 = bx * kTile, y0 = by * kTile;
    const int col = threadIdx.x % kTile;
    int v[kPxPerThread];
#pragma unroll
    for (int j = 0; j < kPxPerThread; ++j) {  // clamped: the loads are issued together
        const int li = threadIdx.x + j * kBlock;
        const int x = x0 + col, y = y0 + li / kTile;
        v[j] = labels[static_cast<size_t>(min(y, h - 1)) * w + min(x, w - 1)];
    }
#pragma unroll
    for (int j = 0; j < kPxPerThread; ++j) {
        const int li = threadIdx.x + j * kBlock;
        const int x = x0 + col, y = y0 + li / kTile;
        lab[li] = (x < w && y < h) ? v[j] : -1;
        cnt[li] = 0;
    }
    __syncthreads();
    tile_ccl::tile_components(lab, par, cnt, x0, y0, w, h, P, lroot, size);
}

// Unions across the left and top borders of every tile, one lane per border
// pixel, and only where an overlap of two segments along the border begins: a
// lane whose pair has the labels of the pair before it is connected to that
// pair on both sides already.  (A union is a chain of dependent loads and
// atomics; with one per equal pair the pass took 97 us on a 3631 x 3859 frame.)
template <bool kBatch>
__global__ __launch_bounds__(2 * kTile) void ccl_border_kernel(CclImage single, CclMap map) {
    CclImage g;
    int bx, by;
    tile_of_launch<kBatch>(single, map, &g, &bx, &by);
    gmem<const int32_t>* __restrict__ labels = as_global(g.labels);
    gmem<int>* P = as_global(g.comp);
    const int w = g.w, h = g.h;
    const int x0 = bx * kTile, y0 = by * kTile;
    const int t = threadIdx.x & (kTile - 1);
    const bool left = threadIdx.x < kTile;
    const int x = left ? x0 : x0 + t, y = left ? y0 + t : y0;
    const bool border = left ? x0 > 0 && y < h : y0 > 0 && x < w;
    // clamped, so that both loads are issued together
    const int i = min(y, h - 1) * w + min(x, w - 1);
    const int o = border ? i - (left ? 1 : w) : i;
    const int mine = labels[i], other = labels[o];
    const bool equal = border && mine == other;
    const int before = __shfl_up(mine, 1);
    const bool equal_before = __shfl_up(equal ? 1 : 0, 1) != 0;
    if (equal && !(t > 0 && equal_before && before == mine)) unite(P, i, o);
}

// comp[i] = P[i] = root of i (the component's smallest index).  Only the
// tile's local roots walk the forest (the thread's walks advanced together,
// with unconditional loads, so that they overlap); every pixel then takes
// its local root's result from LDS.  A local root that is not its
// component's root adds its part's pixel count (its size entry, from the
// tile-local pass) to the root's entry, which holds the root's own part.
template <bool kBatch>
__global__ __launch_bounds__(kBlock) void ccl_flatten_kernel(CclImage single, CclMap map) {
    __shared__ int root[kTilePx];
    CclImage g;
    int bx, by;
    tile_of_launch<kBatch>(single, map, &g, &bx, &by);
    gmem<int>* P = as_global(g.comp);
    gmem<const int>* __restrict__ lroot = as_global(g.lroot);
    gmem<int>* size = as_global(g.size);
    const int w = g.w, h = g.h;
    const int x0 = bx * kTile, y0 = by * kTile;
    int lr[kPxPerThread], x[kPxPerThread], self[kPxPerThread];
    bool in[kPxPerThread];
#pragma unroll
    for (int j = 0; j < kPxPerThread; ++j) {
        const int li = threadIdx.x + j * kBlock;
        const int px = x0 + li % kTile, py = y0 + li / kTile;
        in[j] = px < w && py < h;
        lr[j] = lroot[static_cast<size_t>(min(py, h - 1)) * w + min(px, w - 1)];
        // a local root starts a walk from its own pixel; others stand on
        // pixel 0, which is always a root
        self[j] = in[j] && lr[j] == li ? py * w + px : 0;
        x[j] = self[j];
    }
    unsigned live = 0u;
#pragma unroll
    for (int j = 0; j < kPxPerThread; ++j)
        if (x[j] != 0) live |= 1u << j;
    while (live) {
        int p[kPxPerThread];
#pragma unroll
        for (int j = 0; j < kPxPerThread; ++j) p[j] = load_relaxed(P + x[j]);
#pragma unroll
        for (int j = 0; j < kPxPerThread; ++j) {
            if (!(live & (1u << j))) continue;
            if (p[j] == x[j]) live &= ~(1u << j);
            x[j] = p[j];
        }
    }
#pragma unroll
    for (int j = 0; j < kPxPerThread; ++j) {
        const int li = threadIdx.x + j * kBlock;
        if (!(in[j] && lr[j] == li)) continue;
        root[li] = x[j];
        if (x[j] != self[j])  // pixel 0 is always its own root, so self 0 never adds
            __hip_atomic_fetch_add(size + x[j], size[self[j]], __ATOMIC_RELAXED,
                                   __HIP_MEMORY_SCOPE_AGENT);
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < kPxPerThread; ++j) {
        if (!in[j]) continue;
        const int li = threadIdx.x + j * kBlock;
        const size_t gi = static_cast<size_t>(y0 + li / kTile) * w + x0 + li % kTile;
        __hip_atomic_store(P + gi, root[lr[j]], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
}

// Joins.  A small component (other than the one holding pixel 0) joins the
// component of the pixel left of its root r, or above r at a row start;
// both have smaller roots, so the joins form a forest whose tree roots are
// the smallest indices of their trees and are exactly the components that
// are not small (or hold pixel 0).  After the flatten pass every entry of
// comp holds its pixel's component root and nothing writes comp any more.
//
// The merge launch has two kinds of workgroups.  The first n_number number
// the surviving roots: each covers kMergeBlock consecutive pixels (thread t
// handles pixels t, t + kBlock, ...), gives its survivors their rank in
// raster order among the workgroup's survivors (ballot prefix counts) and
// stores their count.  The others each take a 32 x 32 tile and record the
// join of every small root in it as rank[r] = -2 - target, where target is
// the first root along the chain of joins that is not a small root of the
// same tile: the joins inside a tile are followed in LDS, so the relabel
// pass only walks the joins that cross tiles (on noisy label maps a chain of
// small components, each joining its left neighbour, can be dozens long).
// Loads are unconditional (positions past the image are clamped) so that a
// thread's loads are issued together rather than one branch at a time.
constexpr int kMergePx = 4;
constexpr int kMergeBlock = kBlock * kMergePx;

__device__ __forceinline__ bool is_small(const CclImage& g, int sz) {
    return g.min_segment > 0 ? sz < g.min_segment : 4ll * sz < g.S2;
}

template <bool kBatch>
__global__ __launch_bounds__(kBlock) void ccl_merge_kernel(CclImage single, CclMap map,
                                                           int n_number) {
    __shared__ int part[kMergePx * (kBlock / 64)];
    __shared__ int link[kTilePx];
    CclImage g;
    if (static_cast<int>(blockIdx.x) >= n_number) {
        // ---- joins of the small roots of one tile
        int bx, by;
        const int idx = static_cast<int>(blockIdx.x) - n_number;
        if constexpr (kBatch) {
            resolve_tile(single, map, idx, &g, &bx, &by);
        } else {
            g = single;
            bx = idx % g.tiles_x;
            by = idx / g.tiles_x;
        }
        const int w = g.w, h = g.h;
        const int x0 = bx * kTile, y0 = by * kTile;
        gmem<const int>* __restrict__ comp = as_global(g.comp);
        gmem<const int>* __restrict__ size = as_global(g.size);
        gmem<int>* __restrict__ rank = as_global(g.rank);
        int gi[kPxPerThread], t[kPxPerThread], sz[kPxPerThread];
        bool small[kPxPerThread], root[kPxPerThread];
        // the roots first (all loads issued together), then the size and the
        // join target, which other pixels (most are not roots) read from
        // pixel 0 instead: the loads stay unconditional, so they are issued
        // together, and non-roots fetch one shared line
#pragma unroll
        for (int j = 0; j < kPxPerThread; ++j) {
            const int li = threadIdx.x + j * kBlock;
            const int px = x0 + li % kTile, py = y0 + li / kTile;
            gi[j] = min(py, h - 1) * w + min(px, w - 1);
            const int c = comp[gi[j]];
            root[j] = px < w && py < h && c == gi[j];
        }
#pragma unroll
        for (int j = 0; j < kPxPerThread; ++j) {
            const int q = gi[j] % w > 0 ? gi[j] - 1 : max(gi[j] - w, 0);  // left, or above
            sz[j] = size[root[j] ? gi[j] : 0];
            t[j] = comp[root[j] ? q : 0];
        }
#pragma unroll
        for (int j = 0; j < kPxPerThread; ++j) {
            const int li = threadIdx.x + j * kBlock;
            small[j] = root[j] && gi[j] != 0 && is_small(g, sz[j]);
            // link: a tile slot for a target inside the tile, -4 - target for
            // one outside, -1 for a surviving root, -2 for a pixel that is
            // not a root (never reached: targets are roots)
            int l = root[j] ? -1 : -2;
            if (small[j]) {
                const int ty = t[j] / w, tx = t[j] - ty * w;
                const bool inside = tx >= x0 && tx < x0 + kTile && ty >= y0 && ty < y0 + kTile;
                l = inside ? (ty - y0) * kTile + (tx - x0) : -4 - t[j];
            }
            link[li] = l;
        }
        __syncthreads();
#pragma unroll
        for (int j = 0; j < kPxPerThread; ++j) {
            if (!small[j]) continue;
            int l = link[threadIdx.x + j * kBlock], slot = -1;
            while (l >= 0) {  // links point to smaller slots: the walk ends
                slot = l;
                l = link[slot];
            }
            const int target = l <= -4 ? -4 - l : (y0 + slot / kTile) * w + x0 + slot % kTile;
            rank[gi[j]] = -2 - target;
        }
        return;
    }
    // ---- numbering of the surviving roots of kMergeBlock consecutive pixels
    int blk;
    resolve_block<kBatch>(single, map, &g, &blk);
    const int n = g.w * g.h;
    gmem<const int>* __restrict__ comp = as_global(g.comp);
    gmem<const int>* __restrict__ size = as_global(g.size);
    gmem<int>* __restrict__ rank = as_global(g.rank);
    const int base = blk * kMergeBlock + threadIdx.x;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    bool survives[kMergePx], root[kMergePx];
#pragma unroll
    for (int j = 0; j < kMergePx; ++j) {
        const int r = base + j * kBlock;
        root[j] = r < n && comp[min(r, n - 1)] == r;
    }
#pragma unroll
    for (int j = 0; j < kMergePx; ++j) {
        const int r = base + j * kBlock;
        const int sz = size[root[j] ? r : 0];  // non-roots share one line
        survives[j] = root[j] && (r == 0 || !is_small(g, sz));
    }
    unsigned long long ballot[kMergePx];
#pragma unroll
    for (int j = 0; j < kMergePx; ++j) {
        ballot[j] = __ballot(survives[j]);
        if (lane == 0) part[j * (kBlock / 64) + wave] = __popcll(ballot[j]);
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < kMergePx; ++j) {
        if (!survives[j]) continue;
        int offset = 0;  // survivors in the (pass, wave) groups before this one
        for (int q = 0; q < j * (kBlock / 64) + wave; ++q) offset += part[q];
        rank[base + j * kBlock] = offset + __popcll(ballot[j] & ((1ull << lane) - 1ull));
    }
    if (threadIdx.x == 0) {
        int total = 0;
        for (int q = 0; q < kMergePx * (kBlock / 64); ++q) total += part[q];
        as_global(g.block_count)[blk] = total;
    }
}

// One workgroup: exclusive scan of the per-block counts in place; the total
// is the number of segments.  Each thread takes kScanPer consecutive counts of
// a chunk (one trip through memory), wavefronts scan the threads' sums by
// shuffles.  (With a run of counts per thread read one by one, twice, it took
// 25 us on a 3631 x 3859 frame's 13,684 counts.)
constexpr int kScanThreads = 1024, kScanPer = 16;

__global__ __launch_bounds__(kScanThreads) void ccl_scan_kernel(int nblocks, int* __restrict__ count,
                                                                int* __restrict__ n_segments) {
    __shared__ int part[kScanThreads / 64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    int carry = 0;
    for (int base = 0; base < nblocks; base += kScanThreads * kScanPer) {
        const int lo = base + threadIdx.x * kScanPer;
        int c[kScanPer], sum = 0;
#pragma unroll
        for (int j = 0; j < kScanPer; ++j) c[j] = count[min(lo + j, nblocks - 1)];
#pragma unroll
        for (int j = 0; j < kScanPer; ++j) {
            c[j] = lo + j < nblocks ? c[j] : 0;
            sum += c[j];
        }
        int inc = sum;
        for (int d = 1; d < 64; d <<= 1) {
            const int v = __shfl_up(inc, d);
            if (lane >= d) inc += v;
        }
        if (lane == 63) part[wave] = inc;
        __syncthreads();  // (also: every count of the chunk is read)
        int run = carry + inc - sum;
        for (int q = 0; q < kScanThreads / 64; ++q) {
            if (q < wave) run += part[q];
            carry += part[q];
        }
#pragma unroll
        for (int j = 0; j < kScanPer; ++j) {
            if (lo + j < nblocks) count[lo + j] = run;
            run += c[j];
        }
        __syncthreads();  // part is read
    }
    if (threadIdx.x == 0 && n_segments) *n_segments = carry;
}

// Up to this many runs of kMergeBlock pixels every relabel workgroup scans
// the runs' survivor counts itself, in LDS, and the one-workgroup scan launch
// is skipped; beyond it the scan kernel runs first.
constexpr int kFusedScanMax = 4096;
constexpr int kFusedScanSmall = 1024;  // a variant with fewer count loads per thread

// Final labels: rank of the pixel's surviving root plus the number of
// survivors in earlier runs.  comp[i] is the pixel's component
// root; a surviving root carries its rank, a joined one -2 - (the root it
// joins), and the joins are followed to the tree root.  Same pixel-to-thread
// map as the merge pass.  With SQ > 0 (up to SQ * kBlock runs), block_count
// holds the merge pass's counts and every workgroup derives the offsets
// itself (workgroup 0 also stores the total); with SQ = 0 it holds the
// offsets already.
template <int SQ, bool kBatch>
__global__ __launch_bounds__(kBlock) void ccl_relabel_kernel(CclImage single, CclMap map) {
    extern __shared__ int s_off[];  // SQ > 0: nblocks offsets
    __shared__ int wave_part[kBlock / 64];
    CclImage g;
    int blk;
    resolve_block<kBatch>(single, map, &g, &blk);
    const int n = g.w * g.h, nblocks = g.nmerge;
    gmem<const int>* __restrict__ comp = as_global(g.comp);
    gmem<int>* rank = as_global(g.rank);
    gmem<const int>* __restrict__ block_count = as_global(g.block_count);
    gmem<int32_t>* __restrict__ out = as_global(g.out);
    const int base = blk * kMergeBlock + threadIdx.x;
    int r[kMergePx], k[kMergePx];
#pragma unroll
    for (int j = 0; j < kMergePx; ++j)  // clamped: loads issued together
        r[j] = comp[min(base + j * kBlock, n - 1)];
#pragma unroll
    for (int j = 0; j < kMergePx; ++j) k[j] = rank[r[j]];
    if constexpr (SQ > 0) {
        // exclusive prefix sums of the counts into s_off: coalesced loads
        // into LDS, each thread sums a run of consecutive counts, the runs'
        // sums are scanned with shuffles in each wavefront and then across
        // the wavefronts, and each thread writes its run's offsets back
        constexpr int kQ = SQ;
        int cnt[kQ];
#pragma unroll
        for (int q = 0; q < kQ; ++q)  // clamped, so every load is issued at once
            cnt[q] = block_count[min(static_cast<int>(threadIdx.x) + q * kBlock, nblocks - 1)];
#pragma unroll
        for (int q = 0; q < kQ; ++q) {
            const int j = threadIdx.x + q * kBlock;
            if (j < nblocks) s_off[j] = cnt[q];
        }
        __syncthreads();
        const int per = (nblocks + kBlock - 1) / kBlock;
        const int lo = min(static_cast<int>(threadIdx.x) * per, nblocks);
        const int hi = min(lo + per, nblocks);
        int sum = 0;
        for (int j = lo; j < hi; ++j) sum += s_off[j];
        const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
        int inc = sum;
        for (int d = 1; d < 64; d <<= 1) {
            const int v = __shfl_up(inc, d);
            if (lane >= d) inc += v;
        }
        if (lane == 63) wave_part[wave] = inc;
        __syncthreads();
        int run = inc - sum, total = 0;
        for (int q = 0; q < kBlock / 64; ++q) {
            if (q < wave) run += wave_part[q];
            total += wave_part[q];
        }
        for (int j = lo; j < hi; ++j) {
            const int c = s_off[j];
            s_off[j] = run;
            run += c;
        }
        __syncthreads();
        if (blk == 0 && threadIdx.x == 0 && g.n_segments) *as_global(g.n_segments) = total;
    }
    // Follow the joins to a surviving root, one rank load per step, the
    // thread's walks advanced together (finished ones reload their root,
    // harmlessly) so that their loads overlap.  Each step also re-links the
    // root visited before to the current root's target (path splitting: the
    // target is an ancestor, so concurrent walks stay correct), so walks
    // that pass the same chain of joins later find it shorter.
    int prev[kMergePx];
#pragma unroll
    for (int j = 0; j < kMergePx; ++j) prev[j] = -1;
    unsigned live = 0u;
#pragma unroll
    for (int j = 0; j < kMergePx; ++j)
        if (k[j] < 0) live |= 1u << j;
    while (live) {
        int nx[kMergePx], kn[kMergePx];
#pragma unroll
        for (int j = 0; j < kMergePx; ++j) nx[j] = k[j] < 0 ? -2 - k[j] : r[j];
#pragma unroll
        for (int j = 0; j < kMergePx; ++j) kn[j] = rank[nx[j]];
#pragma unroll
        for (int j = 0; j < kMergePx; ++j) {
            if (!(live & (1u << j))) continue;
            if (prev[j] >= 0) rank[prev[j]] = k[j];
            prev[j] = r[j];
            r[j] = nx[j];
            k[j] = kn[j];
            if (k[j] >= 0) live &= ~(1u << j);
        }
    }
    auto offset_of = [&](int root) {
        if constexpr (SQ > 0) {
            return s_off[root / kMergeBlock];
        } else {
            return block_count[root / kMergeBlock];
        }
    };
#pragma unroll
    for (int j = 0; j < kMergePx; ++j) {
        const int i = base + j * kBlock;
        if (i < n) out[i] = k[j] + offset_of(r[j]);
    }
}

// All four passes of a small frame in one workgroup, its links and sizes in
// LDS: the unions across tile borders, the flattening, the joins with the
// numbering, and the relabelling, with a barrier for a launch between them.
// Bound by those chains of LDS round trips and, in a one-call segmentation
// of a thumbnail, by the host's launches (2.5 us each), of which it saves
// three.  One workgroup has one compute unit's LDS pipe, so its time grows
// with the frame.  A whole frame, in us, with it and with the four launches:
// 48 x 40 29.1 and 35.3; 96 x 72 34.0 and 40.2, on noise 35.4 and 48.1;
// 128 x 128 (which would also need more than 64 KB of LDS) 49.2 and 45.9, on
// noise 52.2 and 53.8.
constexpr int kSmallThreads = 1024, kSmallPx = 8;
constexpr int kSmallMax = 8000;  // 64 KB of LDS with the counts

__device__ __forceinline__ int lds_load(const int* p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}
__device__ __forceinline__ void lds_store(int* p, int v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}
__device__ __forceinline__ int lds_root(const int* P, int i) {
    for (int p = lds_load(P + i); p != i; p = lds_load(P + i)) i = p;
    return i;
}

__global__ __launch_bounds__(kSmallThreads) void ccl_small_kernel(CclImage g, Divisor by_w,
                                                                  Divisor by_h) {
    extern __shared__ int s_small[];  // n links, then n sizes (later ranks and joins)
    __shared__ int part[kSmallPx * (kSmallThreads / 64)];
    __shared__ int wave_part[kSmallPx * (kSmallThreads / 64) / 64];
    const int w = g.w, h = g.h, n = w * h;
    int* const P = s_small;
    int* const C = s_small + n;
    gmem<const int32_t>* labels = as_global(g.labels);  // may be the output
    gmem<const int>* __restrict__ lroot = as_global(g.lroot);
    gmem<const int>* __restrict__ size = as_global(g.size);
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    // links to the tile-local roots; their sizes (0: not a local root)
    int lr[kSmallPx], sz[kSmallPx];
#pragma unroll
    for (int j = 0; j < kSmallPx; ++j) {
        const int i = min(static_cast<int>(threadIdx.x) + j * kSmallThreads, n - 1);
        lr[j] = lroot[i];
        sz[j] = size[i];  // (read where only a local root's is set, used for those alone)
    }
#pragma unroll
    for (int j = 0; j < kSmallPx; ++j) {
        const int i = threadIdx.x + j * kSmallThreads;
        if (i >= n) continue;
        const int y = by_w.quotient(i), x = i - y * w;
        const int r = ((y & ~(kTile - 1)) + lr[j] / kTile) * w + (x & ~(kTile - 1)) + lr[j] % kTile;
        P[i] = r;
        C[i] = r == i ? sz[j] : 0;
    }
    __syncthreads();
    // unions across the tiles' left and top borders, as in the border pass
    const int upright = ((w - 1) / kTile) * h, level = ((h - 1) / kTile) * w;
    for (int q = threadIdx.x; q < upright + level; q += kSmallThreads) {
        int i, o, along, t;
        if (q < upright) {
            const int b = by_h.quotient(q), y = q - b * h;
            i = y * w + (b + 1) * kTile;
            o = i - 1;
            along = w;
            t = y;
        } else {
            const int b = by_w.quotient(q - upright), x = q - upright - b * w;
            i = (b + 1) * kTile * w + x;
            o = i - w;
            along = 1;
            t = x;
        }
        const bool first = (t & (kTile - 1)) == 0;
        const int back = first ? 0 : along;
        const int mine = labels[i], other = labels[o];
        const int before = labels[i - back], other_before = labels[o - back];
        if (mine != other || (!first && before == mine && other_before == mine)) continue;
        int a = i, c = o;
        for (;;) {
            a = lds_root(P, a);
            c = lds_root(P, c);
            if (a == c) break;
            const int hi = max(a, c), lo = min(a, c);
            const int old = atomicMin(P + hi, lo);
            if (old == hi) break;
            a = old;
            c = lo;
        }
    }
    __syncthreads();
    // component roots; a local root that is none adds its part's size
    for (int i = threadIdx.x; i < n; i += kSmallThreads) {
        const int r = lds_root(P, i);
        lds_store(P + i, r);
        if (r != i && C[i] > 0) atomicAdd(C + r, C[i]);
    }
    __syncthreads();
    // the survivors' ranks in raster order, the others' joins
    int rank[kSmallPx];
    bool survives[kSmallPx];
#pragma unroll
    for (int j = 0; j < kSmallPx; ++j) {
        const int i = threadIdx.x + j * kSmallThreads;
        const bool root = i < n && P[min(i, n - 1)] == i;
        survives[j] = root && (i == 0 || !is_small(g, C[i]));
        const unsigned long long b = __ballot(survives[j]);
        if (lane == 0) part[j * (kSmallThreads / 64) + wave] = __popcll(b);
        rank[j] = __popcll(b & ((1ull << lane) - 1ull));
        if (root && !survives[j]) C[i] = -2 - P[i - by_w.quotient(i) * w > 0 ? i - 1 : i - w];
    }
    __syncthreads();
    constexpr int kParts = kSmallPx * (kSmallThreads / 64);  // a thread each
    static_assert(kParts == 128 && kSmallMax <= kSmallThreads * kSmallPx,
                  "two wavefronts scan the counts");
    int own = 0, inc = 0;
    if (threadIdx.x < kParts) {
        own = inc = part[threadIdx.x];
        for (int d = 1; d < 64; d <<= 1) {
            const int v = __shfl_up(inc, d);
            if (lane >= d) inc += v;
        }
        if (lane == 63) wave_part[wave] = inc;
    }
    __syncthreads();
    if (threadIdx.x < kParts) {
        int base = 0;
        for (int q = 0; q < wave; ++q) base += wave_part[q];
        part[threadIdx.x] = base + inc - own;
        if (threadIdx.x == kParts - 1 && g.n_segments) *as_global(g.n_segments) = base + inc;
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < kSmallPx; ++j)
        if (survives[j])
            C[threadIdx.x + j * kSmallThreads] = part[j * (kSmallThreads / 64) + wave] + rank[j];
    __syncthreads();
    // final labels: the joins followed to a survivor; each step gives the root
    // before it the value (a rank, or a later join) that it read, so that the
    // walks through the same chain find it shorter
    gmem<int32_t>* out = as_global(g.out);
    for (int i = threadIdx.x; i < n; i += kSmallThreads) {
        int at = P[i], k = lds_load(C + at);
        while (k < 0) {
            const int next = -2 - k;
            k = lds_load(C + next);
            lds_store(C + at, k);
            at = next;
        }
        out[i] = k;
    }
}

}  // namespace

int scan_tiles_for(int n) { return (n + kMergeBlock - 1) / kMergeBlock; }

CclImage ccl_image(const Workspace& ws, int32_t w, int32_t h, const Grid& g, int32_t min_segment,
                   int32_t* labels_out, int32_t* n_segments) {
    CclImage c;
    c.labels = ws.labels;
    c.out = labels_out;
    c.comp = ws.ccl0;   // local roots, then component roots
    c.size = ws.ccl1;   // component sizes
    c.rank = ws.ccl2;   // ranks of the surviving roots, join links of the others
    c.lroot = ws.ccl3;  // local roots (index inside the tile)
    c.block_count = ws.scan;  // per-block surviving roots (then their offsets)
    c.n_segments = n_segments;
    c.w = w;
    c.h = h;
    c.S2 = static_cast<long long>(g.S) * g.S;
    c.min_segment = min_segment;
    c.tiles_x = (w + kTile - 1) / kTile;
    c.nmerge = scan_tiles_for(w * h);
    return c;
}

int ccl_tiles_for(int32_t w, int32_t h) {
    return ((w + kTile - 1) / kTile) * ((h + kTile - 1) / kTile);
}

bool ccl_batch_supported(int32_t w, int32_t h) { return scan_tiles_for(w * h) <= kFusedScanMax; }

#define SLIC_STEP(name, ...)                                 \
    do {                                                     \
        KernelTimer t_(name, s);                             \
        __VA_ARGS__;                                         \
        if ((e = hipGetLastError()) != hipSuccess) return e; \
    } while (0)

hipError_t launch_connectivity(const Workspace& ws, int32_t w, int32_t h, const Grid& g,
                               int32_t min_segment, int32_t* labels_out, int32_t* n_segments,
                               hipStream_t s, bool local_done) {
    const CclImage c = ccl_image(ws, w, h, g, min_segment, labels_out, n_segments);
    const CclMap none{};
    hipError_t e;
    const int tiles = ccl_tiles_for(w, h);
    const dim3 grid((w + kTile - 1) / kTile, (h + kTile - 1) / kTile);
    if (!local_done)
        SLIC_STEP("ccl_local", ccl_local_kernel<false><<<grid, kBlock, 0, s>>>(c, none));
    if (w * h <= kSmallMax) {  // the times on both sides stand at the kernel
        SLIC_STEP("ccl_small", ccl_small_kernel<<<1, kSmallThreads, 2 * sizeof(int) * w * h, s>>>(
                                   c, make_divisor(w), make_divisor(h)));
        return hipSuccess;
    }
    SLIC_STEP("ccl_border", ccl_border_kernel<false><<<grid, 2 * kTile, 0, s>>>(c, none));
    SLIC_STEP("ccl_flatten", ccl_flatten_kernel<false><<<grid, kBlock, 0, s>>>(c, none));
    SLIC_STEP("ccl_merge",
              ccl_merge_kernel<false><<<c.nmerge + tiles, kBlock, 0, s>>>(c, none, c.nmerge));
    const size_t lds = c.nmerge * sizeof(int);
    if (c.nmerge <= kFusedScanSmall) {
        SLIC_STEP("ccl_relabel",
                  ccl_relabel_kernel<kFusedScanSmall / kBlock, false><<<c.nmerge, kBlock, lds, s>>>(
                      c, none));
    } else if (c.nmerge <= kFusedScanMax) {
        SLIC_STEP("ccl_relabel",
                  ccl_relabel_kernel<kFusedScanMax / kBlock, false><<<c.nmerge, kBlock, lds, s>>>(
                      c, none));
    } else {
        SLIC_STEP("ccl_scan", ccl_scan_kernel<<<1, kScanThreads, 0, s>>>(c.nmerge, c.block_count,
                                                                   c.n_segments));
        SLIC_STEP("ccl_relabel", ccl_relabel_kernel<0, false><<<c.nmerge, kBlock, 0, s>>>(c, none));
    }
    return hipSuccess;
}

hipError_t launch_connectivity_batch(const CclMap& map, int total_tiles, int total_blocks,
                                     int max_nmerge, hipStream_t s) {
    if (!map.images || max_nmerge > kFusedScanMax) return hipErrorInvalidValue;
    const CclImage unused{};
    hipError_t e;
    SLIC_STEP("ccl_local", ccl_local_kernel<true><<<total_tiles, kBlock, 0, s>>>(unused, map));
    SLIC_STEP("ccl_border",
              ccl_border_kernel<true><<<total_tiles, 2 * kTile, 0, s>>>(unused, map));
    SLIC_STEP("ccl_flatten",
              ccl_flatten_kernel<true><<<total_tiles, kBlock, 0, s>>>(unused, map));
    SLIC_STEP("ccl_merge", ccl_merge_kernel<true><<<total_blocks + total_tiles, kBlock, 0, s>>>(
                               unused, map, total_blocks));
    const size_t lds = max_nmerge * sizeof(int);
    if (max_nmerge <= kFusedScanSmall) {
        SLIC_STEP("ccl_relabel",
                  ccl_relabel_kernel<kFusedScanSmall / kBlock, true><<<total_blocks, kBlock, lds, s>>>(
                      unused, map));
    } else {
        SLIC_STEP("ccl_relabel",
                  ccl_relabel_kernel<kFusedScanMax / kBlock, true><<<total_blocks, kBlock, lds, s>>>(
                      unused, map));
    }
    return hipSuccess;
}

#undef SLIC_STEP

// Stray-pixel filter (Section 3's clean-up: two one-thread-per-pixel passes
// of one kernel).  A pixel none of whose 4-neighbours inside the image shares
// its label takes the label that occurs most often among them, ties going to
// the first in the order up, left, right, down.  Each pass reads one map and
// writes the other.
namespace {

// kStrayPer rows of one column per thread: the pixels above and below are
// mostly the thread's own, every load is issued at once (from clamped
// positions), and no position needs a division (10 us per pass at 1024 x 1024
// with one pixel per thread and a branch around each neighbour's load).
constexpr int kStrayPer = 4, kStrayW = 64, kStrayH = kBlock / kStrayW;

__global__ __launch_bounds__(kBlock) void stray_kernel(const int32_t* __restrict__ in, int w, int h,
                                                       Divisor by_tiles, int tiles_x,
                                                       int32_t* __restrict__ out) {
    const int by = by_tiles.quotient(blockIdx.x), bx = blockIdx.x - by * tiles_x;
    const int x = bx * kStrayW + threadIdx.x % kStrayW;
    const int y0 = (by * kStrayH + threadIdx.x / kStrayW) * kStrayPer;
    const int xc = min(x, w - 1), xl = max(xc - 1, 0), xr = min(xc + 1, w - 1);
    int32_t c[kStrayPer + 2], l[kStrayPer], r[kStrayPer];
#pragma unroll
    for (int j = 0; j < kStrayPer + 2; ++j)
        c[j] = in[static_cast<size_t>(min(max(y0 + j - 1, 0), h - 1)) * w + xc];
#pragma unroll
    for (int j = 0; j < kStrayPer; ++j) {
        const size_t row = static_cast<size_t>(min(y0 + j, h - 1)) * w;
        l[j] = in[row + xl];
        r[j] = in[row + xr];
    }
    if (x >= w) return;
#pragma unroll
    for (int j = 0; j < kStrayPer; ++j) {
        const int y = y0 + j;
        if (y >= h) break;
        const int32_t own = c[j + 1];
        // up, left, right, down; outside the image: the pixel's own label,
        // not counted
        const bool ok[4] = {y > 0, x > 0, x + 1 < w, y + 1 < h};
        const int32_t nb[4] = {c[j], l[j], r[j], c[j + 2]};
        bool stray = ok[0] || ok[1] || ok[2] || ok[3];
#pragma unroll
        for (int q = 0; q < 4; ++q) stray = stray && !(ok[q] && nb[q] == own);
        int32_t v = own;
        int best_count = 0;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            int count = 0;
#pragma unroll
            for (int k = 0; k < 4; ++k) count += ok[k] && nb[k] == nb[q] ? 1 : 0;
            if (stray && ok[q] && count > best_count) {
                best_count = count;
                v = nb[q];
            }
        }
        out[static_cast<size_t>(y) * w + x] = v;
    }
}

__global__ __launch_bounds__(kBlock) void copy_labels_kernel(const int32_t* __restrict__ in, int n,
                                                             int32_t* __restrict__ out) {
    const int i = blockIdx.x * kBlock + threadIdx.x;
    if (i < n) out[i] = in[i];
}

}  // namespace

hipError_t launch_stray_filter(const Workspace& ws, int32_t w, int32_t h, int32_t* labels,
                               int32_t passes, hipStream_t s) {
    const int n = w * h;
    const int nb = (n + kBlock - 1) / kBlock;
    int32_t* buf[2] = {labels, ws.ccl0};
    for (int p = 0; p < passes; ++p) {
        KernelTimer t("stray", s);
        const int tiles_x = (w + kStrayW - 1) / kStrayW;
        const int tiles_y = (h + kStrayH * kStrayPer - 1) / (kStrayH * kStrayPer);
        stray_kernel<<<tiles_x * tiles_y, kBlock, 0, s>>>(buf[p & 1], w, h, make_divisor(tiles_x),
                                                          tiles_x, buf[(p + 1) & 1]);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    if (passes & 1) {
        KernelTimer t("stray_copy", s);
        copy_labels_kernel<<<nb, kBlock, 0, s>>>(ws.ccl0, n, labels);
        return hipGetLastError();
    }
    return hipSuccess;
}

}  // namespace slic
