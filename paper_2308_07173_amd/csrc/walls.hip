// walls.hip -- z-vote vertical-feature filter and Euclidean clustering on
// gfx950 (the wall-detection front end, paper Sec. III-D).
//
// z-vote (Sec. III-D.1, Eq. eq_hash_table, Fig. z_vote): every point votes
// for its 2-D cell (floor(x / g), floor(y / g)) in float32; a point is a
// vertical feature when its cell holds at least tau points.  As in the
// paper, the counts live in a hash table: open addressing over 2^b >= 2n
// slots keyed by the two float32 cell coordinates' bits (exact for any
// finite coordinate, -0 folded into +0), so no pass over the points has to
// size a table first and nothing waits for the host.  The vote is one
// compare-and-swap probe sequence and one atomic add per point, the
// read-back one probe sequence.
//
// Clustering (Sec. III-D.2): connected components of the graph joining
// points closer than eps (d2 <= eps^2, float32, the search's fma order).
// The points are bucketed in a grid of 1.25 eps cells (built with the target
// build, so every pair within eps lies in adjacent cells even after float32
// rounding of the cell coordinates).  Passes over the points and, of the 27
// surrounding cells, those with a smaller original index: the first makes the
// smallest of them a point's parent, the last joins the two trees of every pair
// in a lock-free union-find (the larger root is hooked under the smaller with a
// compare-and-swap, parent reads bypass the per-CU cache).
// Roots are therefore the smallest index of their component; a final pass
// writes every point's root as its label.
#include <algorithm>
#include <cmath>
#include <new>

#include "lkc_internal.h"

namespace lkc {

namespace {

constexpr int WT = 256;
constexpr int UNION_SPIN_LIMIT = 1 << 20;

inline unsigned grid_of(int64_t n, int bt) { return (unsigned)((n + bt - 1) / bt); }
inline size_t align256(size_t b) { return (b + 255) & ~size_t(255); }

struct UvMeta {      // 64 bytes, at offset 192 of the context's metadata words
    int umin, umax, vmin, vmax;
    uint32_t bad;
    uint32_t spins;  // union-find retries that hit the limit
    uint32_t n_clusters;
    uint32_t kept;   // points selected by the clustering mask
    int32_t passes;  // sort passes of the grid, laid out afresh
    uint32_t pad[7];
};
static_assert(sizeof(UvMeta) == 64, "UvMeta layout");

__global__ void k_uv_init(UvMeta* m) {
    if (threadIdx.x == 0) {
        m->umin = m->vmin = INT32_MAX;
        m->umax = m->vmax = INT32_MIN;
        m->bad = 0;
        m->spins = 0;
        m->n_clusters = 0;
    }
}

// The hash key of a point's 2-D cell: the bits of floor(x / g) and
// floor(y / g) (float32, correctly rounded division; + 0.0f folds -0 into
// +0, so equal cells have equal keys).  Never EMPTY_KEY (a NaN pattern).
__device__ __forceinline__ bool uv_key(const float* p, float g, unsigned long long& key) {
    if (!finite3(p[0], p[1], p[2])) return false;
    const float fu = floorf(p[0] / g) + 0.0f, fv = floorf(p[1] / g) + 0.0f;
    key = ((unsigned long long)__float_as_uint(fu) << 32) | __float_as_uint(fv);
    return true;
}

__device__ __forceinline__ uint32_t uv_slot(unsigned long long key, int bits) {
    return (uint32_t)((key * 0x9E3779B97F4A7C15ull) >> (64 - bits));
}

struct VoteArgs {
    const float* pts;
    int64_t n;
    float g;
    HashSlot* table;   // 2^bits slots: key, -, count
    int bits;
    int32_t tau;
    uint8_t* keep;
    int32_t* votes;
};

__global__ void __launch_bounds__(WT) k_vote_clear(HashSlot* __restrict__ t, int64_t cap) {
    const int64_t i = (int64_t)blockIdx.x * WT + threadIdx.x;
    if (i < cap) t[i] = HashSlot{EMPTY_KEY, 0u, 0u};
}

__global__ void __launch_bounds__(WT) k_vote(VoteArgs a) {
    const int64_t i = (int64_t)blockIdx.x * WT + threadIdx.x;
    if (i >= a.n) return;
    unsigned long long key;
    if (!uv_key(a.pts + 3 * i, a.g, key)) return;
    const uint32_t mask = (1u << a.bits) - 1u;
    // the table holds at most n < half its slots: an empty slot is reached
    for (uint32_t s = uv_slot(key, a.bits);; s = (s + 1) & mask) {
        const unsigned long long old = atomicCAS(&a.table[s].key, EMPTY_KEY, key);
        if (old == EMPTY_KEY || old == key) {
            atomicAdd(&a.table[s].count, 1u);
            return;
        }
    }
}

__global__ void __launch_bounds__(WT) k_vote_read(VoteArgs a) {
    const int64_t i = (int64_t)blockIdx.x * WT + threadIdx.x;
    if (i >= a.n) return;
    unsigned long long key;
    int32_t c = 0;
    if (uv_key(a.pts + 3 * i, a.g, key)) {
        const uint32_t mask = (1u << a.bits) - 1u;
        // the point's own vote put its key in the table
        for (uint32_t s = uv_slot(key, a.bits);; s = (s + 1) & mask) {
            const unsigned long long k = a.table[s].key;
            if (k == key) {
                c = (int32_t)a.table[s].count;
                break;
            }
            if (k == EMPTY_KEY) break;
        }
    }
    if (a.votes) a.votes[i] = c;
    a.keep[i] = (c > 0 && c >= a.tau) ? 1 : 0;
}

// ---------------------------------------------------------- clustering --

__device__ __forceinline__ int32_t parent_load(const int32_t* par, int32_t x) {
    return __hip_atomic_load(par + x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Root of x, reading the parents coherently (the union phase runs
// concurrently with other hooks).  Parents only ever point to smaller
// indices, so the walk ends.  Every node passed is pointed at its grandparent:
// only roots are ever hooked, so a node that has a parent may be given any
// ancestor at any time.
__device__ __forceinline__ int32_t uf_root(int32_t* par, int32_t x) {
    int32_t p = parent_load(par, x);
    while (p != x) {
        const int32_t g = parent_load(par, p);
        if (g == p) return p;
        __hip_atomic_store(par + x, g, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        x = p;
        p = g;
    }
    return x;
}

// Join the components of a and b: hook the larger root under the smaller.
// A failed compare-and-swap means another thread hooked that root first (so
// the structure progressed); the loop retries with fresh roots.  Bounded: a
// retry count past the limit is reported and the join abandoned.
__device__ __forceinline__ void uf_union(int32_t* par, int32_t a, int32_t b, UvMeta* m) {
    for (int it = 0; it < UNION_SPIN_LIMIT; ++it) {
        a = uf_root(par, a);
        b = uf_root(par, b);
        if (a == b) return;
        const int32_t hi = max(a, b), lo = min(a, b);
        if (atomicCAS(par + hi, hi, lo) == hi) return;
        a = hi;
        b = lo;
    }
    atomicAdd(&m->spins, 1u);
}

// The passes over the pairs test every point against the points of its 27
// surrounding cells with a smaller original index.  With `mask` (the grid then
// holds every point, indexed by original index) only kept points join.
struct ClusterArgs {
    const TargetView* views;
    float e2;
    const uint8_t* mask;
    int32_t* par;
    UvMeta* m;
    int64_t n;
    int chunk;   // reordered points of a wavefront, 2 to 64
};

// From CLUSTER_MANY points on the chip is full without two points a wavefront,
// and the steps count.  Wavefronts that are at least half active, with fewer
// than CLUSTER_SPARSE points a cell, then give each lane a point, whose cells
// in the box it goes through by itself (unmasked, 1 M points of a map, eps 0.5:
// 1.48 -> 1.10 ms; a fifth of them kept: 0.61 -> 0.78, so not there).
constexpr int64_t CLUSTER_MANY = 1 << 19;
constexpr int CLUSTER_SPARSE = 4;

// A volume filled evenly with hardly more points than cells has few pairs and
// short trees: one pass of joins by itself (1 M points, 0.8 a cell: 0.74 ms,
// seeded first 0.88).  (A line or a sheet of as many has long ones.)
__device__ __forceinline__ bool cluster_one_pass(const ClusterArgs& a, const TargetView& T) {
    if (a.n <= CLUSTER_MANY || a.mask || 4 * T.n >= 7 * (int64_t)T.n_cells) return false;
    int64_t box = 1;
    for (int d = 0; d < 3; ++d) {
        const int ext = T.cmax[d] - T.cmin[d] + 1;
        if (ext < 3 || box > 4 * (int64_t)T.n_cells) return false;
        box *= ext;
    }
    return box <= 4 * (int64_t)T.n_cells;
}

// Calls f(half, i, j) for the pairs (j < i) within eps of the wavefront's
// points, done(i, have) after every two of them (own(i) where a lane took its
// own).  A wavefront looks at its `chunk` points a lane each and takes those
// that have anything to do two at a time, one to each half of it; a lane probes
// one of the 27 cells.  Then every lane walks its own cell, or, where that is
// fewer steps (long cells, a few beside empty ones), all lanes walk one cell
// after another (118,000 points of a sweep, eps 1: a lane a cell 11.8 ms, so
// 1.8; a thread a point, in one pass of joins, 8.3).  SEEDED: past the
// first pass, points that are their own parent have no such pair (only a point
// without one ever was), and nothing to do.
template <bool SEEDED, typename F, typename Done, typename Own>
__device__ __forceinline__ void cluster_pairs(const ClusterArgs& a, F f, Done done, Own own) {
    const TargetView T = load_uniform(a.views);
    const int lane = lane_id(), half = lane / 32, c = lane % 32;
    const int64_t wave = ((int64_t)xcd_tile(blockIdx.x, gridDim.x) * WT + threadIdx.x) / WAVE;
    const bool two = a.chunk == 2;   // every lane loads its half's point at once
    const int64_t s = wave * a.chunk + (two ? half : lane);
    float4 p = make_float4(0.f, 0.f, 0.f, 0.f);
    bool active = false;
    if ((two || lane < a.chunk) && s < T.n) {
        p = gload(T.pts + s);
        const int32_t i = __float_as_int(p.w);
        active = SEEDED && !cluster_one_pass(a, T) ? a.par[i] != i : !a.mask || a.mask[i];
        if (!SEEDED && !active) a.par[i] = i;
    }
    unsigned long long todo = ballot(active);
    if (a.chunk == WAVE && T.n < CLUSTER_SPARSE * (int64_t)T.n_cells && __popcll(todo) >= WAVE / 2) {
        if (active) {
            const int32_t i = __float_as_int(p.w);
            const int cx = cell_coord(p.x, T.inv_cell), cy = cell_coord(p.y, T.inv_cell),
                      cz = cell_coord(p.z, T.inv_cell);
            for (int z = max(cz - 1, T.cmin[2]); z <= min(cz + 1, T.cmax[2]); ++z)
                for (int y = max(cy - 1, T.cmin[1]); y <= min(cy + 1, T.cmax[1]); ++y)
                    for (int x = max(cx - 1, T.cmin[0]); x <= min(cx + 1, T.cmax[0]); ++x) {
                        uint32_t st, cn;
                        if (!hash_find(T, pack_key(T, x, y, z), st, cn)) continue;
                        for (uint32_t t = st; t < st + cn; ++t) {
                            const float4 q = gload(T.pts + t);
                            const int32_t j = __float_as_int(q.w);
                            if (j < i && dist2(p.x, p.y, p.z, q.x, q.y, q.z) <= a.e2 &&
                                (!a.mask || a.mask[j]))
                                f(0, i, j);
                        }
                    }
            own(i);
        }
        return;
    }
    const int dz = (c * 57) >> 9, r = c - 9 * dz, dy = (r * 11) >> 5;   // c / 9, r / 3
    while (todo) {
        float px = p.x, py = p.y, pz = p.z, pw = p.w;
        bool have = active;
        if (two) {
            todo = 0;
        } else {
            const int m0 = __builtin_ffsll((long long)todo) - 1;
            todo &= todo - 1;
            const int m1 = todo ? __builtin_ffsll((long long)todo) - 1 : -1;
            if (todo) todo &= todo - 1;
            const int m = half ? m1 : m0;
            have = m >= 0;
            px = shfl(p.x, m & 63);
            py = shfl(p.y, m & 63);
            pz = shfl(p.z, m & 63);
            pw = shfl(p.w, m & 63);
        }
        const int32_t i = __float_as_int(pw);
        const int x = cell_coord(px, T.inv_cell) + r - 3 * dy - 1;
        const int y = cell_coord(py, T.inv_cell) + dy - 1;
        const int z = cell_coord(pz, T.inv_cell) + dz - 1;
        uint32_t st = 0, cn = 0;
        if (!have || c >= 27 || x < T.cmin[0] || x > T.cmax[0] || y < T.cmin[1] || y > T.cmax[1] ||
            z < T.cmin[2] || z > T.cmax[2] || !hash_find(T, pack_key(T, x, y, z), st, cn))
            cn = 0;
        const int longest = wave_max_i32((int)cn);
        const int steps = readlane(wave_incl_scan((int)((cn + WAVE - 1) / WAVE)), WAVE - 1);
        if (longest <= steps) {
            for (uint32_t t = st; t < st + cn; ++t) {
                const float4 q = gload(T.pts + t);
                const int32_t j = __float_as_int(q.w);
                if (j < i && dist2(px, py, pz, q.x, q.y, q.z) <= a.e2 && (!a.mask || a.mask[j]))
                    f(half, i, j);
            }
        } else {
            unsigned long long cells = ballot(cn > 0);
            while (cells) {
                const int l = __builtin_ffsll((long long)cells) - 1;
                cells &= cells - 1;
                const float ux = readlane(px, l), uy = readlane(py, l), uz = readlane(pz, l);
                const int32_t ui = readlane(i, l);
                const int b = readlane((int)st, l), e = b + readlane((int)cn, l);
                for (int t = b + lane; t < e; t += WAVE) {
                    const float4 q = gload(T.pts + t);
                    const int32_t j = __float_as_int(q.w);
                    if (j < ui && dist2(ux, uy, uz, q.x, q.y, q.z) <= a.e2 &&
                        (!a.mask || a.mask[j]))
                        f(l / 32, ui, j);
                }
            }
        }
        done(i, have);
    }
}

// First pass: every point's parent is the smallest of its neighbours (or
// itself).  No two threads write the same word, so nothing contends, and most
// of the pairs are then in one tree already.
__global__ void __launch_bounds__(WT) k_cluster_seed(ClusterArgs a) {
    const TargetView T = load_uniform(a.views);
    if (T.n == 0 || cluster_one_pass(a, T)) {
        // (a rebuild that failed on the device left the grid empty: every
        // point its own root)
        const int64_t g = (int64_t)blockIdx.x * WT + threadIdx.x;
        if (g < a.n) a.par[g] = (int32_t)g;
        return;
    }
    int32_t least[2] = {INT32_MAX, INT32_MAX};
    cluster_pairs<false>(
        a,
        [&](int half, int32_t, int32_t j) {
            least[0] = min(least[0], half ? INT32_MAX : j);
            least[1] = min(least[1], half ? j : INT32_MAX);
        },
        [&](int32_t i, bool have) {
            const int32_t l0 = wave_min_i32(least[0]), l1 = wave_min_i32(least[1]);
            if (have && lane_id() % 32 == 0) a.par[i] = min(lane_id() ? l1 : l0, i);
            least[0] = least[1] = INT32_MAX;
        },
        [&](int32_t i) { a.par[i] = min(least[0], i); });
}

// Points every node at its root: each thread takes its node's grandparent for
// parent until that is a root, and as all do so at once the chains halve with
// every step.
__global__ void __launch_bounds__(WT) k_cluster_flatten(int32_t* __restrict__ par, int64_t n,
                                                        const uint8_t* __restrict__ mask) {
    const int64_t i = (int64_t)blockIdx.x * WT + threadIdx.x;
    if (i >= n || (mask && !mask[i])) return;
    int32_t p = parent_load(par, (int32_t)i);
    for (;;) {
        const int32_t g = parent_load(par, p);
        if (g == p) return;
        __hip_atomic_store(par + i, g, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        p = g;
    }
}

// Second pass, on flattened trees: of every pair in two trees, the larger
// root is given the smallest of the roots that it meets for parent (an atomic
// minimum: nothing is retried, and a root that another pair already gave a
// smaller one is left alone).
__global__ void __launch_bounds__(WT) k_cluster_hook(ClusterArgs a) {
    cluster_pairs<true>(
        a,
        [&](int, int32_t i, int32_t j) {
            const int32_t u = a.par[i], v = a.par[j];
            const int32_t hi = max(u, v), lo = min(u, v);
            if (lo != hi && a.par[hi] > lo) atomicMin(a.par + hi, lo);
        },
        [](int32_t, bool) {}, [](int32_t) {});
}

// Last pass: joins the trees of every pair that are still two.  Two nodes that
// ever had one parent are in one tree: an ordinary load, old as the caches may
// have it, settles nearly every pair.
//
// The passes are bound by latency: the chains of probes, candidates and parent
// walks.  One pass of joins over single points, one thread per point (a few
// thousand kept points of a scan leave most of the chip idle), took 323 us for
// the 30,011 voxels of a scan, of which those on walls take part; the same with
// 32 lanes per point and its chains halved 104, nearly all of it parent walks;
// seeded and flattened first, with the test of the parents, 85; with a hook
// before the joins 54 (9 seed, 5 + 5 flatten, 14 hook, 20 joins).
__global__ void __launch_bounds__(WT) k_cluster_union(ClusterArgs a) {
    cluster_pairs<true>(
        a,
        [&](int, int32_t i, int32_t j) {
            if (a.par[i] != a.par[j]) uf_union(a.par, i, j, a.m);
        },
        [](int32_t, bool) {}, [](int32_t) {});
}

// All passes: the parents of the grid's points, at most two or three joins
// from their roots.
void launch_cluster(hipStream_t st, ClusterArgs a) {
    const int64_t n = a.n;
    // Two points a wavefront where that leaves the chip room (32,768 wavefronts
    // are four times what it holds), more of more points: those with nothing
    // to do are then passed over by the dozen.
    a.chunk = 2;
    while (a.chunk < WAVE / 2 && n / a.chunk > 32768) a.chunk *= 2;
    if (n > CLUSTER_MANY && (!a.mask || n / a.chunk > 65536)) a.chunk = WAVE;
    const dim3 points(grid_of(n, WT)), pairs(grid_of((n + a.chunk - 1) / a.chunk, WT / WAVE));
    hipLaunchKernelGGL(k_cluster_seed, pairs, dim3(WT), 0, st, a);
    hipLaunchKernelGGL(k_cluster_flatten, points, dim3(WT), 0, st, a.par, n, a.mask);
    // (a third pass over the pairs pays while the joins are bound by latency:
    // 300,000 points of a map, eps 0.3, 420 us with the hooks and 470 without;
    // a million, eps 0.5, 1.67 and 1.48 ms)
    if (n <= CLUSTER_MANY) {
        hipLaunchKernelGGL(k_cluster_hook, pairs, dim3(WT), 0, st, a);
        hipLaunchKernelGGL(k_cluster_flatten, points, dim3(WT), 0, st, a.par, n, a.mask);
    }
    hipLaunchKernelGGL(k_cluster_union, pairs, dim3(WT), 0, st, a);
}

// Mask compaction in ascending order, in two launches: kept points per tile,
// then every tile adds up the tiles before it and writes its own points (the
// labels of the points left out too).  Up to RAW_MASK_TILES tiles; past that
// their counts are scanned in between.
constexpr int MASK_TILE = 1024;
constexpr int RAW_MASK_TILES = 4096;

__global__ void __launch_bounds__(WT) k_mask_count(const uint8_t* __restrict__ mask, int64_t n,
                                                   uint32_t* __restrict__ counts) {
    __shared__ uint32_t s_c[WT / WAVE];
    const int64_t b = (int64_t)blockIdx.x * MASK_TILE;
    uint32_t c = 0;
#pragma unroll
    for (int u = 0; u < MASK_TILE / WT; ++u) {
        const int64_t i = b + u * WT + threadIdx.x;
        c += (uint32_t)__popcll(ballot(i < n && mask[i] != 0));
    }
    if (threadIdx.x % WAVE == 0) s_c[threadIdx.x / WAVE] = c;
    __syncthreads();
    if (threadIdx.x == 0) counts[blockIdx.x] = s_c[0] + s_c[1] + s_c[2] + s_c[3];
}

__global__ void __launch_bounds__(WT) k_mask_compact(const float* __restrict__ pts,
                                                     const uint8_t* __restrict__ mask, int64_t n,
                                                     const uint32_t* __restrict__ counts, int raw,
                                                     float* __restrict__ cpts,
                                                     int32_t* __restrict__ cidx,
                                                     int32_t* __restrict__ label,
                                                     UvMeta* __restrict__ m) {
    constexpr int U = MASK_TILE / WT, NW = WT / WAVE;
    __shared__ uint32_t s_c[U][NW], s_b[NW];
    const int l = threadIdx.x % WAVE, w = threadIdx.x / WAVE;
    const int64_t b = (int64_t)blockIdx.x * MASK_TILE;
    uint32_t before = 0;
    if (raw) {
        for (int j = threadIdx.x; j < (int)blockIdx.x; j += WT) before += counts[j];
        before = (uint32_t)readlane(wave_incl_scan((int)before), WAVE - 1);
    }
    if (l == 0) s_b[w] = before;
    uint32_t in = 0;   // bit u: item u is kept
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int64_t i = b + u * WT + threadIdx.x;
        const bool k = i < n && mask[i] != 0;
        in |= k ? 1u << u : 0u;
        if (i < n && !k) label[i] = -1;
        const uint32_t c = (uint32_t)__popcll(ballot(k));
        if (l == 0) s_c[u][w] = c;
    }
    __syncthreads();
    uint32_t o = raw ? s_b[0] + s_b[1] + s_b[2] + s_b[3] : counts[blockIdx.x];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const bool k = (in >> u) & 1u;
        const unsigned long long bal = ballot(k);
        uint32_t at = o + (uint32_t)__popcll(bal & ((1ull << l) - 1ull));
#pragma unroll
        for (int v = 0; v < NW; ++v) {
            at += v < w ? s_c[u][v] : 0u;
            o += s_c[u][v];
        }
        if (k) {
            const int64_t i = b + u * WT + threadIdx.x;
            cpts[3 * (int64_t)at] = pts[3 * i];
            cpts[3 * (int64_t)at + 1] = pts[3 * i + 1];
            cpts[3 * (int64_t)at + 2] = pts[3 * i + 2];
            cidx[at] = (int32_t)i;
        }
    }
    if (blockIdx.x == gridDim.x - 1 && threadIdx.x == 0) m->kept = o;
}

// The status of a grid rebuilt on the device: the rebuild's own, then the
// range of its cells.
__device__ __forceinline__ int32_t cluster_grid_status(const TargetView* views,
                                                       const int32_t* build_status) {
    const int32_t st = build_status ? build_status[0] : (int32_t)LKC_OK;
    if (st != (int32_t)LKC_OK || !views) return st;
    return views->max_abs * views->inv_cell < (float)((1 << 20) - 4) ? (int32_t)LKC_OK
                                                                     : (int32_t)LKC_ERR_INVALID_ARG;
}

// labels: every point's root (full path compression), roots counted; with
// a mask, compacted point c labels its original index cidx[c] with the
// original index of its root (compaction keeps the order, so that is the
// smallest original index of the component).  With build_status, the grid's
// status goes into m->bad and its passes into m->passes.
__global__ void __launch_bounds__(WT) k_cluster_labels(int32_t* __restrict__ par, int64_t n,
                                                       const int32_t* __restrict__ cidx,
                                                       int32_t* __restrict__ label,
                                                       UvMeta* __restrict__ m,
                                                       const uint8_t* __restrict__ mask,
                                                       const TargetView* __restrict__ views,
                                                       const int32_t* __restrict__ build_status) {
    const int64_t i = (int64_t)blockIdx.x * WT + threadIdx.x;
    if (build_status) {
        const int32_t bad = cluster_grid_status(views, build_status);
        if (i == 0) {
            m->bad = (uint32_t)bad;
            m->passes = build_status[3];
        }
        if (bad != (int32_t)LKC_OK) return;   // (the call does it over or fails)
    }
    bool root = false;
    if (i < n && mask && !mask[i]) {
        label[i] = -1;   // (uncompacted masked call: a point left out)
    } else if (i < n) {
        int32_t x = (int32_t)i;
        while (par[x] != x) x = par[x];
        if (cidx)
            label[cidx[i]] = cidx[x];
        else
            label[i] = x;
        root = x == (int32_t)i;
    }
    const unsigned long long b = ballot(root);
    if (threadIdx.x % WAVE == 0 && b) atomicAdd(&m->n_clusters, (uint32_t)__popcll(b));
}

// The status of a clustering with no host wait (one thread): the grid
// rebuild's (build_status, when the rebuild ran on the device), then the
// cell range of the grid, then the join retries.
__global__ void k_cluster_status(const TargetView* __restrict__ Tp,
                                 const int32_t* __restrict__ build_status,
                                 const UvMeta* __restrict__ m, int64_t* __restrict__ n_clusters,
                                 int32_t* __restrict__ status) {
    if (threadIdx.x != 0) return;
    int32_t st = cluster_grid_status(Tp, build_status);
    if (st == (int32_t)LKC_OK && m->spins) st = (int32_t)LKC_ERR_HIP;
    *status = st;
    *n_clusters = st == (int32_t)LKC_OK ? (int64_t)m->n_clusters : 0;
}

UvMeta* uv_meta_dev(lkc_ctx* ctx) { return (UvMeta*)((char*)ctx->meta_dev + 192); }
UvMeta* uv_meta_host(lkc_ctx* ctx) { return (UvMeta*)((char*)ctx->meta_host + 192); }

}  // namespace

lkc_status zvote(lkc_ctx* ctx, const float* pts, int64_t n, float g, int32_t tau,
                 uint8_t* keep, int32_t* votes) {
    if (n == 0) return LKC_OK;
    hipStream_t st = ctx->stream;
    int bits = 6;
    while (((int64_t)1 << bits) < 2 * n) ++bits;
    const int64_t cap = (int64_t)1 << bits;
    lkc_status s;
    HashSlot* table = (HashSlot*)aux_scratch(ctx, sizeof(HashSlot) * (size_t)cap, &s);
    if (!table) return s;
    VoteArgs a{pts, n, g, table, bits, tau, keep, votes};
    hipLaunchKernelGGL(k_vote_clear, dim3(grid_of(cap, WT)), dim3(WT), 0, st, table, cap);
    hipLaunchKernelGGL(k_vote, dim3(grid_of(n, WT)), dim3(WT), 0, st, a);
    hipLaunchKernelGGL(k_vote_read, dim3(grid_of(n, WT)), dim3(WT), 0, st, a);
    LKC_HIP_TRY(ctx, hipGetLastError());
    return LKC_OK;
}

lkc_status euclid_cluster(lkc_ctx* ctx, const float* pts, int64_t n, float eps,
                          const uint8_t* mask, int32_t* labels, int64_t* n_clusters) {
    *n_clusters = 0;
    if (n == 0) return LKC_OK;
    hipStream_t st = ctx->stream;
    if (!ctx->cluster_grid) {
        ctx->cluster_grid = new (std::nothrow) lkc_target();
        if (!ctx->cluster_grid) return set_error(ctx, LKC_ERR_OOM, "host allocation");
    }
    size_t off = 0;
    auto carve = [&](size_t b) {
        const size_t o = off;
        off += align256(b);
        return o;
    };
    const int64_t tiles = (n + MASK_TILE - 1) / MASK_TILE;
    const size_t o_par = carve(4 * (size_t)n), o_fl = carve(mask ? 4 * (size_t)tiles : 0),
                 o_tmp = carve(mask ? 4 * ((size_t)tiles / 4096 + 2) : 0),
                 o_cp = carve(mask ? 12 * (size_t)n : 0), o_ci = carve(mask ? 4 * (size_t)n : 0);
    lkc_status s;
    char* sb = (char*)aux_scratch(ctx, off, &s);
    if (!sb) return s;
    auto* par = (int32_t*)(sb + o_par);
    UvMeta* md = uv_meta_dev(ctx);
    UvMeta* mh = uv_meta_host(ctx);
    const float* cp = pts;
    const int32_t* cidx = nullptr;
    int64_t m = n;
    if (mask) {
        // the kept points, compacted in ascending order
        auto* counts = (uint32_t*)(sb + o_fl);
        auto* cpts = (float*)(sb + o_cp);
        auto* ci = (int32_t*)(sb + o_ci);
        const int raw = tiles <= RAW_MASK_TILES ? 1 : 0;
        hipLaunchKernelGGL(k_mask_count, dim3((unsigned)tiles), dim3(WT), 0, st, mask, n, counts);
        if (!raw) scan_words(st, counts, tiles, (uint32_t*)(sb + o_tmp));
        hipLaunchKernelGGL(k_mask_compact, dim3((unsigned)tiles), dim3(WT), 0, st, pts, mask, n,
                           (const uint32_t*)counts, raw, cpts, ci, labels, md);
        LKC_HIP_TRY(ctx, hipGetLastError());
        LKC_HIP_TRY(ctx, hipMemcpyAsync(mh, md, sizeof(UvMeta), hipMemcpyDeviceToHost, st));
        LKC_HIP_TRY(ctx, hipStreamSynchronize(st));
        m = mh->kept;
        cp = cpts;
        cidx = ci;
        if (m == 0) return LKC_OK;
    }
    lkc_target& grid = *ctx->cluster_grid;
    grid.cell_size = 1.25f * eps;
    // The grid is rebuilt without a wait where its memory and sort passes
    // allow it; what such a rebuild finds wrong (a cell key that needs more
    // passes, a coordinate or a range to refuse) is built once more with one,
    // which sorts in full or gives the error.
    for (int attempt = 0;; ++attempt) {
        s = build_into(ctx, &grid, cp, m, attempt == 0);
        if (s != LKC_OK) return s;
        const bool on_device = grid.host_stale;
        const float reach = grid.view.max_abs * grid.view.inv_cell;
        if (!on_device && !(reach < (float)((1 << 20) - 4)))
            return set_error(ctx, LKC_ERR_INVALID_ARG,
                             "eps %g is too small for the cloud's extent (|p| up to %g)",
                             (double)eps, (double)grid.view.max_abs);
        hipLaunchKernelGGL(k_uv_init, dim3(1), dim3(64), 0, st, md);
        launch_cluster(st, ClusterArgs{grid.view_dev, eps * eps, nullptr, par, md, m, 0});
        hipLaunchKernelGGL(k_cluster_labels, dim3(grid_of(m, WT)), dim3(WT), 0, st, par, m,
                           cidx, labels, md, (const uint8_t*)nullptr,
                           (const TargetView*)grid.view_dev,
                           on_device ? (const int32_t*)((const char*)grid.view_dev +
                                                        view_status_offset())
                                     : nullptr);
        LKC_HIP_TRY(ctx, hipGetLastError());
        LKC_HIP_TRY(ctx, hipMemcpyAsync(mh, md, sizeof(UvMeta), hipMemcpyDeviceToHost, st));
        LKC_HIP_TRY(ctx, hipStreamSynchronize(st));
        if (on_device && mh->bad && attempt == 0) continue;
        // (the next build, with or without a wait, finds the passes of this
        // cloud, as after a build with a wait, not those of an earlier one)
        if (on_device) grid.sort_passes = mh->passes;
        if (mh->spins)
            return set_error(ctx, LKC_ERR_HIP, "%u union-find joins exceeded the retry limit",
                             mh->spins);
        *n_clusters = mh->n_clusters;
        return LKC_OK;
    }
}

lkc_status euclid_cluster_async(lkc_ctx* ctx, const float* pts, int64_t n, float eps,
                                const uint8_t* mask, int32_t* labels, int64_t* n_clusters,
                                int32_t* status) {
    hipStream_t st = ctx->stream;
    if (n == 0) {
        hipLaunchKernelGGL(k_uv_init, dim3(1), dim3(64), 0, st, uv_meta_dev(ctx));
        hipLaunchKernelGGL(k_cluster_status, dim3(1), dim3(64), 0, st, (const TargetView*)nullptr,
                           (const int32_t*)nullptr, (const UvMeta*)uv_meta_dev(ctx), n_clusters,
                           status);
        LKC_HIP_TRY(ctx, hipGetLastError());
        return LKC_OK;
    }
    if (!ctx->cluster_grid) {
        ctx->cluster_grid = new (std::nothrow) lkc_target();
        if (!ctx->cluster_grid) return set_error(ctx, LKC_ERR_OOM, "host allocation");
    }
    lkc_status s;
    auto* par = (int32_t*)aux_scratch(ctx, 4 * (size_t)n, &s);
    if (!par) return s;
    UvMeta* md = uv_meta_dev(ctx);
    hipLaunchKernelGGL(k_uv_init, dim3(1), dim3(64), 0, st, md);
    // The grid over every point (the mask applies in the joins and labels,
    // so no count comes back); a new cell size lays the key out afresh,
    // with one synchronous build.
    lkc_target& grid = *ctx->cluster_grid;
    const float cell = 1.25f * eps;
    if (grid.cell_size != cell) grid.sort_passes = 0;
    grid.cell_size = cell;
    s = build_into(ctx, &grid, pts, n, true);
    if (s != LKC_OK) return s;
    // the rebuild ran on the device (its status there) or on the host (and succeeded)
    const int32_t* bst =
        grid.host_stale ? (const int32_t*)((const char*)grid.view_dev + view_status_offset())
                        : nullptr;
    launch_cluster(st, ClusterArgs{grid.view_dev, eps * eps, mask, par, md, n, 0});
    hipLaunchKernelGGL(k_cluster_labels, dim3(grid_of(n, WT)), dim3(WT), 0, st, par, n,
                       (const int32_t*)nullptr, labels, md, mask,
                       (const TargetView*)nullptr, (const int32_t*)nullptr);
    hipLaunchKernelGGL(k_cluster_status, dim3(1), dim3(64), 0, st,
                       (const TargetView*)grid.view_dev, bst, (const UvMeta*)md, n_clusters,
                       status);
    LKC_HIP_TRY(ctx, hipGetLastError());
    return LKC_OK;
}

}  // namespace lkc
