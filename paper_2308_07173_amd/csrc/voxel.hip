// voxel.hip -- voxel filter and sliding-window submap on gfx950.
//
// Voxel filter: the paper voxel-filters its scans and maps (Sec. III-D.1;
// leaf sizes in Sec. IV).  voxel(p) = floor((p - o) / leaf) per axis in
// float32 (IEEE subtraction and correctly rounded division); one output
// point per occupied voxel, the mean of its points; voxels in (vz, vy, vx)
// order.  On the device:
//   1. voxel bounds of the finite points (per-workgroup partials, one
//      reduction workgroup); the synchronous filter reads them once to size
//      the sort key;
//   2. key in the occupied box (ascending key = (vz, vy, vx) order), points
//      left out get the largest key;
//   3. stable LSD radix sort of (key, point index) on the occupied bits (keys
//      of up to 32 bits as 32-bit words);
//   4. run starts counted per tile of sorted positions;
//   5. every tile numbers its voxels, gathers its points into LDS and writes
//      the voxels that start in it: one thread per voxel sums its run in FP64
//      in ascending point order and writes the float32 mean, the count and the
//      voxel coordinates.
// Step 5 adds in the same order as the FP64 definition, so the centroids
// are the correctly rounded float32 of the FP64 means.
//
// Submap (Sec. III-C.3: only the map points near the current race-line pose
// are queried): a flag per map point (float32 d2 <= r2, fma order of the
// search), an exclusive scan and a compaction give the indices in ascending
// order; they are HBM-streaming kernels over the map's float4 records.
#include <algorithm>
#include <cmath>

#include "lkc_internal.h"

namespace lkc {

namespace {

constexpr int VT = 256;
constexpr int VOX_CLAMP = 1 << 20;

inline size_t align256(size_t b) { return (b + 255) & ~size_t(255); }
inline unsigned grid_of(int64_t n, int bt) { return (unsigned)((n + bt - 1) / bt); }
int bit_w(unsigned long long v) { return v ? 64 - __builtin_clzll(v) : 0; }

struct VoxMeta {        // 64 bytes
    int vmin[3];
    int vmax[3];
    uint32_t n_finite;
    uint32_t bad;       // a voxel coordinate outside [-2^20, 2^20)
    uint32_t n_vox;
    uint32_t pad[7];
};
static_assert(sizeof(VoxMeta) == 64, "VoxMeta layout");

struct VoxPart {
    int vmin[3];
    int vmax[3];
    uint32_t n_finite;
    uint32_t bad;
};

__device__ __forceinline__ bool voxel_of(const float* p, float ox, float oy, float oz, float leaf,
                                         int (&v)[3], bool& bad) {
    const float x = p[0], y = p[1], z = p[2];
    bad = false;
    if (!finite3(x, y, z)) return false;
    const float q[3] = {(x - ox) / leaf, (y - oy) / leaf, (z - oz) / leaf};
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        const float f = floorf(q[d]);
        const bool ok = f >= -(float)VOX_CLAMP && f < (float)VOX_CLAMP;
        bad = bad || !ok;
        v[d] = ok ? (int)f : 0;
    }
    return true;
}

__device__ __forceinline__ int wmax_i(int v) { return ~wave_min_i32(~v); }
__device__ __forceinline__ uint32_t wsum_u(uint32_t v) {
    return (uint32_t)readlane(wave_incl_scan((int)v), WAVE - 1);
}

// Folds the block's parts (one per thread) into one, in thread 0.
template <int THREADS>
__device__ __forceinline__ VoxPart vox_fold(VoxPart p, VoxPart* sp) {
    const int w = threadIdx.x / WAVE, l = threadIdx.x % WAVE;
    for (int d = 0; d < 3; ++d) {
        p.vmin[d] = wave_min_i32(p.vmin[d]);
        p.vmax[d] = wmax_i(p.vmax[d]);
    }
    p.n_finite = wsum_u(p.n_finite);
    p.bad = wsum_u(p.bad);
    if (l == 0) sp[w] = p;
    __syncthreads();
    if (threadIdx.x == 0) {
        p = sp[0];
        for (int ww = 1; ww < THREADS / WAVE; ++ww) {
            for (int d = 0; d < 3; ++d) {
                p.vmin[d] = min(p.vmin[d], sp[ww].vmin[d]);
                p.vmax[d] = max(p.vmax[d], sp[ww].vmax[d]);
            }
            p.n_finite += sp[ww].n_finite;
            p.bad += sp[ww].bad;
        }
    }
    return p;
}

constexpr VoxPart VOX_NONE{{INT32_MAX, INT32_MAX, INT32_MAX}, {INT32_MIN, INT32_MIN, INT32_MIN}, 0, 0};

// Bound by the one read of the points: the workgroups (at most one part per
// thread of the fold below) stride over them and fold once at the end (a fold
// for every 256 points took 36 us for 3.76 M, this takes 15).
constexpr int BOUNDS_BLOCKS = 1024;

__global__ void __launch_bounds__(VT) k_vox_bounds(const float* __restrict__ pts, int64_t n,
                                                   float ox, float oy, float oz, float leaf,
                                                   VoxPart* __restrict__ parts) {
    __shared__ VoxPart sp[VT / WAVE];
    VoxPart p = VOX_NONE;
    for (int64_t i = (int64_t)blockIdx.x * VT + threadIdx.x; i < n; i += (int64_t)gridDim.x * VT) {
        int v[3] = {0, 0, 0};
        bool bad = false;
        if (!voxel_of(pts + 3 * i, ox, oy, oz, leaf, v, bad)) continue;
        p.n_finite += 1u;
        p.bad += bad ? 1u : 0u;
        if (!bad)
            for (int d = 0; d < 3; ++d) {
                p.vmin[d] = min(p.vmin[d], v[d]);
                p.vmax[d] = max(p.vmax[d], v[d]);
            }
    }
    p = vox_fold<VT>(p, sp);
    if (threadIdx.x == 0) parts[blockIdx.x] = p;
}

// (`host`: the meta record goes there too, pinned memory that the host reads
// after it waited, without a copy launch)
__global__ void __launch_bounds__(BOUNDS_BLOCKS) k_vox_bounds_final(
    const VoxPart* __restrict__ parts, int nparts, VoxMeta* __restrict__ meta,
    VoxMeta* __restrict__ host) {
    __shared__ VoxPart sp[BOUNDS_BLOCKS / WAVE];
    const VoxPart t =
        vox_fold<BOUNDS_BLOCKS>((int)threadIdx.x < nparts ? parts[threadIdx.x] : VOX_NONE, sp);
    if (threadIdx.x == 0) {
        VoxMeta m{};
        for (int d = 0; d < 3; ++d) {
            m.vmin[d] = t.vmin[d];
            m.vmax[d] = t.vmax[d];
        }
        m.n_finite = t.n_finite;
        m.bad = t.bad;
        *meta = m;
        if (host) *host = m;
    }
}

// The sorted pass of both filters.  Their keys are relative to the box minimum
// (read on the device): row-major in the occupied box (wx, wy its extents), or,
// without a host wait, with power-of-two strides of `b` bits (the same (vz,
// vy, vx) order).  Keys from `limit` on are left out and sort last: non-finite
// points, and with `b` those outside [-2^20, 2^20) or past 2^b in some axis.
struct VoxArgs {
    const float* pts;
    int64_t n;
    float ox, oy, oz, leaf;
    int b;                          // bits per axis, 0: row-major
    unsigned long long wx, wy;
    unsigned long long limit;
    VoxMeta* meta;                  // bounds (k_vox_bounds_final), n_vox, over
    void* keys;                     // Key[n]
    uint32_t* vals;
    uint32_t* counts;               // voxels starting in each tile (raw), or before it, then all
    int tiles;
    int raw;
    float* centroid;                // [cap][3]
    int32_t* count;                 // [cap] or NULL
    int32_t* voxel;                 // [cap][3] or NULL
    int64_t cap;
    int64_t* n_out;                 // device, or NULL
    int32_t* status;                // device, or NULL
    VoxMeta* host;                  // pinned, or NULL
};

template <typename Key>
__global__ void __launch_bounds__(VT) k_vox_keys(VoxArgs a) {
    const int64_t i = (int64_t)blockIdx.x * VT + threadIdx.x;
    if (i >= a.n) return;
    int v[3];
    bool bad;
    unsigned long long key = a.limit;
    if (voxel_of(a.pts + 3 * i, a.ox, a.oy, a.oz, a.leaf, v, bad) && !bad) {
        const uint32_t r0 = (uint32_t)(v[0] - a.meta->vmin[0]);
        const uint32_t r1 = (uint32_t)(v[1] - a.meta->vmin[1]);
        const uint32_t r2 = (uint32_t)(v[2] - a.meta->vmin[2]);
        if (a.b == 0) {
            key = (unsigned long long)r0 + a.wx * ((unsigned long long)r1 + a.wy * r2);
        } else {
            const uint32_t lim = 1u << a.b;
            if (r0 < lim && r1 < lim && r2 < lim)
                key = (unsigned long long)r0 | ((unsigned long long)r1 << a.b) |
                      ((unsigned long long)r2 << (2 * a.b));
            else
                atomicOr(&a.meta->pad[0], 1u);   // over
        }
    }
    ((Key*)a.keys)[i] = (Key)key;
    a.vals[i] = (uint32_t)i;
}

constexpr int VOX_ITEMS = 8;
constexpr int VOX_TILE = VT * VOX_ITEMS;
constexpr int RAW_VOX_TILES = 4096;   // up to this many tiles add up their counts themselves

// Which of this thread's VOX_ITEMS sorted positions (tile position u * VT +
// threadIdx.x) start a voxel, bit by bit.  The indices are clamped, not the
// loads skipped: a load under a condition waits for the one before it.
template <typename Key>
__device__ __forceinline__ uint32_t vox_starts(const Key* __restrict__ keys, int64_t base,
                                               int64_t n, Key limit, Key (&k)[VOX_ITEMS]) {
    Key p[VOX_ITEMS];
#pragma unroll
    for (int u = 0; u < VOX_ITEMS; ++u) {
        const int64_t i = min(base + u * VT + threadIdx.x, n - 1);
        k[u] = keys[i];
        p[u] = keys[max(i - 1, (int64_t)0)];
    }
    uint32_t starts = 0;
#pragma unroll
    for (int u = 0; u < VOX_ITEMS; ++u) {
        const int64_t i = base + u * VT + threadIdx.x;
        if (i < n && k[u] < limit && (i == 0 || k[u] != p[u])) starts |= 1u << u;
    }
    return starts;
}

// Voxels starting in each tile.
template <typename Key>
__global__ void __launch_bounds__(VT) k_vox_count(VoxArgs a) {
    __shared__ uint32_t s_c[VT / WAVE];
    Key k[VOX_ITEMS];
    const uint32_t starts = vox_starts((const Key*)a.keys, (int64_t)blockIdx.x * VOX_TILE, a.n,
                                       (Key)a.limit, k);
    const uint32_t c = wsum_u((uint32_t)__popc(starts));
    if (threadIdx.x % WAVE == 0) s_c[threadIdx.x / WAVE] = c;
    __syncthreads();
    if (threadIdx.x == 0) a.counts[blockIdx.x] = s_c[0] + s_c[1] + s_c[2] + s_c[3];
}

struct Sum3 {
    double x, y, z;
};

// One workgroup per tile of sorted positions: it numbers the voxels that start
// in the tile, gathers the tile's points into LDS with every lane, and one
// thread per voxel adds its run in FP64 in ascending point order; a run that
// goes on past the tile is gathered on, a workgroup of points at a time.  Then
// the float32 mean, the count and the voxel coordinates.  Nothing is written
// where the call fails (a voxel out of range, more voxels than the capacity).
//
// Bound by the scattered reads of the points (12 of every 128 bytes fetched).
// One thread per voxel that read its run from memory, one point after another,
// was bound by their latency: 128 us for 3.76 M points in 400 k voxels, 186
// with flags, scan and starts in launches of their own; now 59 + 5.
template <typename Key>
__global__ void __launch_bounds__(VT) k_vox_emit(VoxArgs a) {
    constexpr int NW = VT / WAVE;
    __shared__ uint32_t s_c[VOX_ITEMS][NW], s_b[3][NW];
    __shared__ uint16_t s_start[VOX_TILE + 1];
    __shared__ Key s_key[VOX_TILE];
    __shared__ float s_p[3][VOX_TILE];
    __shared__ int s_more;
    const Key* keys = (const Key*)a.keys;
    const Key limit = (Key)a.limit;
    const int tid = threadIdx.x, l = tid % WAVE, w = tid / WAVE;
    // (each XCD takes a contiguous part, whose rows of voxels share the lines
    // of points in its L2)
    const int tile = (int)xcd_tile(blockIdx.x, gridDim.x);
    const int64_t base = (int64_t)tile * VOX_TILE;
    // all first loads together
    Key k[VOX_ITEMS];
    const uint32_t starts = vox_starts(keys, base, a.n, limit, k);
    uint32_t i[VOX_ITEMS];
#pragma unroll
    for (int u = 0; u < VOX_ITEMS; ++u) i[u] = a.vals[min(base + u * VT + tid, a.n - 1)];
    const Key after = keys[min(base + VOX_TILE, a.n - 1)];   // the next tile's first
    const uint32_t m_bad = a.meta->bad, m_over = a.meta->pad[0];
    const int vmin[3] = {a.meta->vmin[0], a.meta->vmin[1], a.meta->vmin[2]};
    // voxels before this tile, and all
    uint32_t before = 0, total = 0;
    if (a.raw) {
        for (int j = tid; j < a.tiles; j += VT) {
            const uint32_t c = a.counts[j];
            before += j < tile ? c : 0u;
            total += c;
        }
        before = wsum_u(before);
        total = wsum_u(total);
    }
    uint32_t kept = 0;   // the tile's points that are not left out: its first ones
#pragma unroll
    for (int u = 0; u < VOX_ITEMS; ++u) {
        const uint32_t c = (uint32_t)__popcll(ballot((starts >> u) & 1u));
        kept += (uint32_t)__popcll(ballot(base + u * VT + tid < a.n && k[u] < limit));
        if (l == 0) s_c[u][w] = c;
    }
    if (l == 0) {
        s_b[0][w] = before;
        s_b[1][w] = total;
        s_b[2][w] = kept;
    }
    __syncthreads();
    if (a.raw) {
        before = s_b[0][0] + s_b[0][1] + s_b[0][2] + s_b[0][3];
        total = s_b[1][0] + s_b[1][1] + s_b[1][2] + s_b[1][3];
    } else {
        before = a.counts[tile];
        total = a.counts[a.tiles];
    }
    kept = s_b[2][0] + s_b[2][1] + s_b[2][2] + s_b[2][3];
    const bool bad = m_bad || m_over;
    const int32_t status = m_bad ? (int32_t)LKC_ERR_INVALID_ARG
                           : m_over || (int64_t)total > a.cap ? (int32_t)LKC_ERR_BUDGET
                                                              : (int32_t)LKC_OK;
    if (tile == 0 && tid == 0) {
        a.meta->n_vox = total;
        if (a.host) a.host->n_vox = total;
        if (a.status) *a.status = status;
        if (a.n_out) *a.n_out = bad ? 0 : (int64_t)total;
    }
    if (status != (int32_t)LKC_OK) return;
    int here = 0;   // voxels that start in this tile
#pragma unroll
    for (int u = 0; u < VOX_ITEMS; ++u) {
        const bool f = (starts >> u) & 1u;
        const unsigned long long bal = ballot(f);
        int at = here + __popcll(bal & ((1ull << l) - 1ull));
#pragma unroll
        for (int v = 0; v < NW; ++v) {
            at += v < w ? (int)s_c[u][v] : 0;
            here += (int)s_c[u][v];
        }
        if (f) {
            s_start[at] = (uint16_t)(u * VT + tid);
            s_key[at] = k[u];
        }
    }
    if (here == 0) return;
    {
        float x[VOX_ITEMS], y[VOX_ITEMS], z[VOX_ITEMS];
#pragma unroll
        for (int u = 0; u < VOX_ITEMS; ++u) {
            const float* p = a.pts + 3 * (int64_t)i[u];
            x[u] = p[0];
            y[u] = p[1];
            z[u] = p[2];
        }
#pragma unroll
        for (int u = 0; u < VOX_ITEMS; ++u) {
            s_p[0][u * VT + tid] = x[u];
            s_p[1][u * VT + tid] = y[u];
            s_p[2][u * VT + tid] = z[u];
        }
    }
    __syncthreads();
    // (eight points are read ahead of their adds, which stay in order)
    const auto add = [&](Sum3& s, int from, int to) {
        constexpr int U = 8;
        for (int j = from; j < to; j += U) {
            float x[U], y[U], z[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int t = min(j + u, VOX_TILE - 1);
                x[u] = s_p[0][t];
                y[u] = s_p[1][t];
                z[u] = s_p[2][t];
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                if (j + u < to) {
                    s.x += (double)x[u];
                    s.y += (double)y[u];
                    s.z += (double)z[u];
                }
            }
        }
    };
    const auto write = [&](int v, const Sum3& s, int64_t n_pts) {
        const int64_t o = (int64_t)before + v;
        const double c = (double)n_pts;
        a.centroid[3 * o] = (float)(s.x / c);
        a.centroid[3 * o + 1] = (float)(s.y / c);
        a.centroid[3 * o + 2] = (float)(s.z / c);
        if (a.count) a.count[o] = (int32_t)n_pts;
        if (a.voxel) {
            const Key k = s_key[v];
            int32_t x, y, z;
            if (a.b == 0) {
                const Key wx = (Key)a.wx, wy = (Key)a.wy, r = k / wx;
                x = (int32_t)(k - r * wx);
                z = (int32_t)(r / wy);
                y = (int32_t)(r - (Key)z * wy);
            } else {
                const unsigned long long m = (1ull << a.b) - 1ull, kk = k;
                x = (int32_t)(kk & m);
                y = (int32_t)((kk >> a.b) & m);
                z = (int32_t)(kk >> (2 * a.b));
            }
            a.voxel[3 * o] = x + vmin[0];
            a.voxel[3 * o + 1] = y + vmin[1];
            a.voxel[3 * o + 2] = z + vmin[2];
        }
    };
    // (the last voxel of the tile may go on past it: below)
    for (int v = tid; v < here - 1; v += VT) {
        Sum3 s{0.0, 0.0, 0.0};
        add(s, s_start[v], s_start[v + 1]);
        write(v, s, (int64_t)s_start[v + 1] - s_start[v]);
    }
    const int first = s_start[here - 1];
    const Key key = s_key[here - 1];
    const bool mine = tid == (here - 1) % VT;
    Sum3 s{0.0, 0.0, 0.0};
    if (mine) add(s, first, (int)kept);
    int64_t end = base + kept;   // the run's points up to here are added
    if (kept == VOX_TILE && end < a.n && after == key) {
        for (;;) {
            // the next points, up to the first with another key
            const int size = (int)min((int64_t)VT, a.n - end);
            __syncthreads();   // the points before are added
            if (tid == 0) s_more = size;
            Key kn = 0;
            if (tid < size) {
                kn = keys[end + tid];
                const float* p = a.pts + 3 * (int64_t)a.vals[end + tid];
                s_p[0][tid] = p[0];
                s_p[1][tid] = p[1];
                s_p[2][tid] = p[2];
            }
            __syncthreads();
            const unsigned long long other = ballot(tid < size && kn != key);
            if (l == 0 && other) atomicMin(&s_more, w * WAVE + __builtin_ffsll((long long)other) - 1);
            __syncthreads();
            const int to = s_more;
            if (mine) add(s, 0, to);
            end += to;
            if (to < size || end >= a.n) break;
        }
    }
    if (mine) write(here - 1, s, end - (base + first));
}

__global__ void __launch_bounds__(VT) k_submap_flags(const float4* __restrict__ orig, int64_t n,
                                                     float cx, float cy, float cz, float r2,
                                                     uint32_t* __restrict__ flags) {
    const int64_t i = (int64_t)blockIdx.x * VT + threadIdx.x;
    if (i >= n) return;
    const float4 p = orig[i];
    flags[i] = dist2(cx, cy, cz, p.x, p.y, p.z) <= r2 ? 1u : 0u;
}

__global__ void __launch_bounds__(VT) k_submap_compact(const float4* __restrict__ orig, int64_t n,
                                                       float cx, float cy, float cz, float r2,
                                                       const uint32_t* __restrict__ offs,
                                                       int64_t cap, int32_t* __restrict__ out,
                                                       float* __restrict__ gathered,
                                                       uint32_t* __restrict__ total) {
    const int64_t i = (int64_t)blockIdx.x * VT + threadIdx.x;
    if (i >= n) return;
    const float4 p = orig[i];
    const bool in = dist2(cx, cy, cz, p.x, p.y, p.z) <= r2;
    const uint32_t o = offs[i];
    if (in && (int64_t)o < cap) {
        if (out) out[o] = (int32_t)i;
        if (gathered) {
            gathered[3 * (int64_t)o] = p.x;
            gathered[3 * (int64_t)o + 1] = p.y;
            gathered[3 * (int64_t)o + 2] = p.z;
        }
    }
    if (i == n - 1) *total = o + (in ? 1u : 0u);
}

}  // namespace

// grow-only auxiliary scratch of the context
void* aux_scratch(lkc_ctx* ctx, size_t bytes, lkc_status* st) {
    *st = LKC_OK;
    if (ctx->aux_scratch_bytes < bytes) {
        if (ctx->aux_scratch) {
            if (hipStreamSynchronize(ctx->stream) != hipSuccess) {
                *st = set_error(ctx, LKC_ERR_HIP, "stream synchronize failed");
                return nullptr;
            }
            (void)hipFree(ctx->aux_scratch);
            ctx->aux_scratch = nullptr;
            ctx->aux_scratch_bytes = 0;
        }
        const size_t b = bytes + bytes / 4;
        if (hipMalloc(&ctx->aux_scratch, b) != hipSuccess) {
            ctx->aux_scratch = nullptr;
            *st = set_error(ctx, LKC_ERR_OOM, "auxiliary scratch of %zu bytes", b);
            return nullptr;
        }
        ctx->aux_scratch_bytes = b;
    }
    return ctx->aux_scratch;
}

namespace {

VoxMeta* vox_meta_dev(lkc_ctx* ctx) { return (VoxMeta*)((char*)ctx->meta_dev + 128); }
VoxMeta* vox_meta_host(lkc_ctx* ctx) { return (VoxMeta*)((char*)ctx->meta_host + 128); }

}  // namespace

namespace {

// Scratch of a filter of n points.
struct VoxScratch {
    unsigned long long *ka, *kb;
    uint32_t *va, *vb, *sort, *counts, *tmp;
    VoxPart* parts;
};

lkc_status vox_scratch(lkc_ctx* ctx, int64_t n, VoxScratch& v) {
    const size_t nn = (size_t)std::max<int64_t>(n, 1);
    const size_t tiles = (nn + VOX_TILE - 1) / VOX_TILE;
    size_t off = 0;
    auto carve = [&](size_t b) {
        const size_t o = off;
        off += align256(b);
        return o;
    };
    const size_t o_ka = carve(8 * nn), o_kb = carve(8 * nn), o_va = carve(4 * nn),
                 o_vb = carve(4 * nn), o_sort = carve(4 * sort_count_words(n)),
                 o_cnt = carve(4 * (tiles + 1)), o_tmp = carve(4 * (tiles / 4096 + 2)),
                 o_pp = carve(sizeof(VoxPart) * BOUNDS_BLOCKS);
    lkc_status s;
    char* b = (char*)aux_scratch(ctx, off, &s);
    if (!b) return s;
    v = VoxScratch{(unsigned long long*)(b + o_ka), (unsigned long long*)(b + o_kb),
                   (uint32_t*)(b + o_va),           (uint32_t*)(b + o_vb),
                   (uint32_t*)(b + o_sort),         (uint32_t*)(b + o_cnt),
                   (uint32_t*)(b + o_tmp),          (VoxPart*)(b + o_pp)};
    return LKC_OK;
}

void launch_vox_bounds(hipStream_t st, const VoxArgs& a, const VoxScratch& v, VoxMeta* host) {
    const int nb = (int)std::max<int64_t>(1, std::min<int64_t>(grid_of(a.n, VT), BOUNDS_BLOCKS));
    hipLaunchKernelGGL(k_vox_bounds, dim3((unsigned)nb), dim3(VT), 0, st, a.pts, a.n, a.ox, a.oy,
                       a.oz, a.leaf, v.parts);
    hipLaunchKernelGGL(k_vox_bounds_final, dim3(1), dim3(BOUNDS_BLOCKS), 0, st,
                       (const VoxPart*)v.parts, nb, a.meta, host);
}

__global__ void k_vox_end(uint32_t* counts, int tiles) { counts[tiles] = 0u; }

// Keys, sort and output of a.n > 0 points, `bits` key bits (`limit` among them).
template <typename Key>
lkc_status vox_sorted(lkc_ctx* ctx, VoxArgs a, const VoxScratch& v, int bits) {
    hipStream_t st = ctx->stream;
    a.keys = v.ka;
    a.vals = v.va;
    a.counts = v.counts;
    a.tiles = (int)((a.n + VOX_TILE - 1) / VOX_TILE);
    a.raw = a.tiles <= RAW_VOX_TILES ? 1 : 0;
    hipLaunchKernelGGL(k_vox_keys<Key>, dim3(grid_of(a.n, VT)), dim3(VT), 0, st, a);
    bool in_b = false;
    const lkc_status s = sort_pairs(ctx, (Key*)v.ka, v.va, (Key*)v.kb, v.vb, a.n, bits, v.sort, &in_b);
    if (s != LKC_OK) return s;
    if (in_b) {
        a.keys = v.kb;
        a.vals = v.vb;
    }
    hipLaunchKernelGGL(k_vox_count<Key>, dim3((unsigned)a.tiles), dim3(VT), 0, st, a);
    if (!a.raw) {
        // (one more entry, for the sum of all)
        hipLaunchKernelGGL(k_vox_end, dim3(1), dim3(1), 0, st, a.counts, a.tiles);
        scan_words(st, a.counts, (int64_t)a.tiles + 1, v.tmp);
    }
    hipLaunchKernelGGL(k_vox_emit<Key>, dim3((unsigned)a.tiles), dim3(VT), 0, st, a);
    LKC_HIP_TRY(ctx, hipGetLastError());
    return LKC_OK;
}

// The status and count of no points at all (one thread).
__global__ void k_vox_none(VoxArgs a) {
    *a.status = (int32_t)LKC_OK;
    *a.n_out = 0;
}

}  // namespace

lkc_status voxel_filter(lkc_ctx* ctx, const float* pts, int64_t n, const float* origin,
                        float leaf, float* centroid, int32_t* count, int32_t* voxel, int64_t cap,
                        int64_t* n_out) {
    *n_out = 0;
    if (n == 0) return LKC_OK;
    hipStream_t st = ctx->stream;
    VoxScratch v;
    lkc_status s = vox_scratch(ctx, n, v);
    if (s != LKC_OK) return s;
    VoxMeta* mh = vox_meta_host(ctx);
    VoxArgs a{};
    a.pts = pts;
    a.n = n;
    a.ox = origin[0];
    a.oy = origin[1];
    a.oz = origin[2];
    a.leaf = leaf;
    a.meta = vox_meta_dev(ctx);
    a.centroid = centroid;
    a.count = count;
    a.voxel = voxel;
    a.cap = cap;
    a.host = mh;
    launch_vox_bounds(st, a, v, mh);
    LKC_HIP_TRY(ctx, hipGetLastError());
    LKC_HIP_TRY(ctx, hipStreamSynchronize(st));
    if (mh->bad)
        return set_error(ctx, LKC_ERR_INVALID_ARG,
                         "%u points fall in a voxel outside [-2^20, 2^20) per axis", mh->bad);
    if (mh->n_finite == 0) return LKC_OK;
    unsigned long long w[3];
    for (int d = 0; d < 3; ++d) w[d] = (unsigned long long)(mh->vmax[d] - mh->vmin[d]) + 1ull;
    a.wx = w[0];
    a.wy = w[1];
    a.limit = w[0] * w[1] * w[2];          // <= 2^63: the key of non-finite points
    const int bits = bit_w(a.limit);
    s = bits <= 32 ? vox_sorted<uint32_t>(ctx, a, v, bits)
                   : vox_sorted<unsigned long long>(ctx, a, v, bits);
    if (s != LKC_OK) return s;
    LKC_HIP_TRY(ctx, hipStreamSynchronize(st));
    const int64_t nv = mh->n_vox;
    *n_out = nv;
    if (nv > cap)
        return set_error(ctx, LKC_ERR_BUDGET, "%lld voxels exceed the output capacity %lld",
                         (long long)nv, (long long)cap);
    return LKC_OK;
}

lkc_status voxel_filter_async(lkc_ctx* ctx, const float* pts, int64_t n, const float* origin,
                              float leaf, int axis_bits, float* centroid, int32_t* count,
                              int32_t* voxel, int64_t cap, int64_t* n_out, int32_t* status) {
    hipStream_t st = ctx->stream;
    VoxScratch v;
    lkc_status s = vox_scratch(ctx, n, v);
    if (s != LKC_OK) return s;
    VoxArgs a{};
    a.pts = pts;
    a.n = n;
    a.ox = origin[0];
    a.oy = origin[1];
    a.oz = origin[2];
    a.leaf = leaf;
    a.b = axis_bits;
    a.limit = 1ull << (3 * axis_bits);
    a.meta = vox_meta_dev(ctx);
    a.centroid = centroid;
    a.count = count;
    a.voxel = voxel;
    a.cap = cap;
    a.n_out = n_out;
    a.status = status;
    if (n == 0) {
        hipLaunchKernelGGL(k_vox_none, dim3(1), dim3(1), 0, st, a);
        LKC_HIP_TRY(ctx, hipGetLastError());
        return LKC_OK;
    }
    launch_vox_bounds(st, a, v, nullptr);
    const int bits = 3 * axis_bits + 1;
    return bits <= 32 ? vox_sorted<uint32_t>(ctx, a, v, bits)
                      : vox_sorted<unsigned long long>(ctx, a, v, bits);
}

lkc_status submap_extract(lkc_ctx* ctx, const lkc_target* t, const float* center, float radius,
                          int32_t* idx, float* gathered, int64_t cap, int64_t* n_out) {
    *n_out = 0;
    const int64_t n = t->view.n;
    if (n == 0) return LKC_OK;
    hipStream_t st = ctx->stream;
    size_t off = 0;
    auto carve = [&](size_t b) {
        const size_t o = off;
        off += align256(b);
        return o;
    };
    const size_t o_fl = carve(4 * (size_t)n), o_tmp = carve(4 * ((size_t)n / 4096 + 2));
    lkc_status s;
    char* b = (char*)aux_scratch(ctx, off, &s);
    if (!b) return s;
    auto* flags = (uint32_t*)(b + o_fl);
    auto* tmp = (uint32_t*)(b + o_tmp);
    VoxMeta* md = vox_meta_dev(ctx);
    VoxMeta* mh = vox_meta_host(ctx);
    const float r2 = radius * radius;
    const unsigned g = grid_of(n, VT);
    hipLaunchKernelGGL(k_submap_flags, dim3(g), dim3(VT), 0, st, (const float4*)t->view.orig, n,
                       center[0], center[1], center[2], r2, flags);
    scan_words(st, flags, n, tmp);
    hipLaunchKernelGGL(k_submap_compact, dim3(g), dim3(VT), 0, st, (const float4*)t->view.orig,
                       n, center[0], center[1], center[2], r2, (const uint32_t*)flags, cap, idx,
                       gathered, &md->n_vox);
    LKC_HIP_TRY(ctx, hipGetLastError());
    LKC_HIP_TRY(ctx, hipMemcpyAsync(mh, md, sizeof(VoxMeta), hipMemcpyDeviceToHost, st));
    LKC_HIP_TRY(ctx, hipStreamSynchronize(st));
    *n_out = mh->n_vox;
    if (*n_out > cap)
        return set_error(ctx, LKC_ERR_BUDGET, "%lld window points exceed the capacity %lld",
                         (long long)*n_out, (long long)cap);
    return LKC_OK;
}

lkc_status submap_build(lkc_ctx* ctx, const lkc_target* map, const float* center, float radius,
                        int32_t* idx, int64_t cap, int64_t* n_out, lkc_target* out) {
    // the window's points, gathered in ascending map order, then built
    const int64_t n = map->view.n;
    float* pts = nullptr;
    if (n > 0) LKC_HIP_TRY(ctx, hipMalloc(&pts, 12 * (size_t)n));
    lkc_status s = submap_extract(ctx, map, center, radius, idx, pts, idx ? cap : n, n_out);
    if (s == LKC_OK) s = build_into(ctx, out, pts, *n_out);
    if (pts) {
        (void)hipStreamSynchronize(ctx->stream);
        (void)hipFree(pts);
    }
    return s;
}

}  // namespace lkc
