// search.hip -- k-nearest-points search and per-point covariance on gfx950.
//
// The step the paper moves to the GPU (Sec. III-C.1, the paragraph after
// Eq. eq_trans_likelihood, and Sec. IV-E.1): for every query point find its
// corresponding nearest points, then estimate the covariance that models
// the point as a Gaussian in GICP.
//
// Search -- two kernels:
//   * the group search (k_group) takes 64 queries per wavefront (queries
//     sorted by the Morton code of their cell; self queries are the target's
//     own sorted points), one lane per query with its top-k in registers:
//     the group streams the point runs of its block of cells once, each
//     candidate broadcast to all lanes, and answers every lane whose result
//     the block proves exact;
//   * the wavefront-per-query search (k_wave: the whole search with algorithm 2
//     and of launches that takes_group leaves to it) answers the rest: the 27
//     cells around the query probed a lane each, then Chebyshev rings, lanes
//     enumerating a ring's cells in parallel and probing the cell hash; the
//     surviving runs streamed 64 candidates at a time (one coalesced read) and
//     appended with one ballot to an unordered list of keys in LDS, which is
//     cut back by a distance that enough of them do not exceed and sorted once
//     at the end by counting; it stops once the unvisited region lies beyond
//     the k-th distance (or the radius), and a query whose rings would outgrow
//     the occupied cells finishes with one sweep of the cell table, so uncapped
//     searches stay bounded.  Small targets, and sparse ones of middling size,
//     are taken as a whole, through the boxes of their 16-point runs.
// Ordering everywhere is lexicographic on (float32 d2, original index), so
// both kernels, every launch shape and every visiting order give the same
// bits.
//
// Covariance -- two passes over the neighbours relative to the query point
// (centred, 1/n), then the smallest eigenvector of the 3x3 in closed form
// (float32) for the GICP plane regulariser; fused into both searches and
// standalone in k_cov, one lane per query in each (k_wave and k_cov gather the
// neighbours, and take the weights, with all lanes beforehand).
#include <climits>
#include <cmath>
#include <mutex>

#include "lkc_internal.h"

namespace lkc {

namespace {

constexpr float INF = __builtin_huge_valf();

struct SearchParams {
    int k;
    float r2;        // squared radius (INF if uncapped)
    int capped;
};

// ---------------------------------------------------- wavefront candidates --

__device__ __forceinline__ int lanes_below(unsigned long long m) {
    return (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32),
                                          __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
}
// Orders this wavefront's LDS writes before its later reads by other lanes
// (the LDS serves a wavefront in order: only the compiler has to be told).
__device__ __forceinline__ void wave_lds_fence() {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// The candidates of one query, whole wavefront: an unordered list of exact
// keys (float32 d2 bits above the original index) in LDS and the squared
// distance beyond which none can matter.  A batch of 64 candidates is
// appended with one ballot; the list is cut back when it outgrows a wavefront
// or a tighter bound is wanted, and sorted once, at the end, by counting.
// The cut needs a distance that at least k and not many more entries do not
// exceed: on the surfaces a LiDAR sees the counts grow about linearly with
// d2, so interpolating between two counts finds it in two or three ballots
// (a search over the distance's bits takes about twenty).
//
// LIM: entries that stay between cuts, 64, or 128 for k > WIDE_K, whose cuts
// would otherwise have no room between k and LIM: nearly every batch then cut
// the list, to one entry exactly (k = 64, a self search of 100,000 points in
// one cell: 38.7 ms, with 128 6.8).
constexpr int WIDE_K = 56;

template <int LIM>
struct WaveList {
    static constexpr int CAP = LIM + WAVE;   // entries (LDS keys)
    static constexpr int REGS = CAP / WAVE;
    static constexpr int SLACK_ENTRIES = 8;
    unsigned long long* buf;
    float bound;               // (uniform) farther candidates are not among the k nearest
    int n;                     // (uniform) entries
    int k;
    bool dirty;                // (uniform) entries since the last cut

    // Cuts the list back to about k + SLACK_ENTRIES, at most `most`, entries;
    // CLOSE: to about k, from between the nearest entry and the farthest (a query
    // far from the target has all its candidates there).
    template <int R, bool CLOSE = false>
    __device__ __forceinline__ void cut(int most) {
        constexpr int SLACK = CLOSE ? 0 : SLACK_ENTRIES;
        const int lane = lane_id();
        // (k <= WIDE_K with LIM = 64: no entry too many)
        const int keep = LIM == WAVE ? k + SLACK : min(k + SLACK, most);
        const int aim = LIM == WAVE ? k + SLACK / 2 : min(k + SLACK / 2, keep);
        wave_lds_fence();
        unsigned long long e[R];
        float d[R], far = 0.0f, near = INF;
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const bool have = lane + r * WAVE < n;
            e[r] = have ? buf[lane + r * WAVE] : ~0ull;
            // (an absent entry's distance is a NaN: below nothing)
            d[r] = __uint_as_float((uint32_t)(e[r] >> 32));
            far = fmaxf(far, have ? d[r] : 0.0f);
            near = fminf(near, have ? d[r] : INF);
        }
        const auto within_d = [&](float t) {
            int c = 0;
#pragma unroll
            for (int r = 0; r < R; ++r) c += __popcll(ballot(d[r] <= t));
            return c;
        };
        float lo = 0.0f, up = wave_max_nonneg(far);
        int c_lo = 0, c_up = n;
        if (CLOSE) {
            lo = wave_min_nonneg(near);
            c_lo = within_d(lo);
            if (c_lo >= k) {
                up = lo;
                c_up = c_lo;
            }
        }
        for (int it = 0; it < 6 && c_up > keep; ++it) {
            const float t =
                lo + (up - lo) * ((float)(aim - c_lo) * __builtin_amdgcn_rcpf((float)(c_up - c_lo)));
            const int c = within_d(t);
            if (c >= k) {
                up = t;
                c_up = c;
            } else {
                lo = t;
                c_lo = c;
            }
        }
        unsigned long long m[R];
#pragma unroll
        for (int r = 0; r < R; ++r) m[r] = ballot(d[r] <= up);
        if (c_up > most) {
            // many equal distances: tell the keys apart bit by bit
            unsigned long long ul = 0, uu = ~0ull >> 1;
            for (int bit = 62; bit >= 0 && c_up > most; --bit) {
                const unsigned long long t = ul | ((1ull << bit) - 1ull);
                int c = 0;
#pragma unroll
                for (int r = 0; r < R; ++r) c += __popcll(ballot(e[r] <= t));
                if (c >= k) {
                    uu = t;
                    c_up = c;
                } else {
                    ul |= 1ull << bit;
                }
            }
#pragma unroll
            for (int r = 0; r < R; ++r) m[r] = ballot(e[r] <= uu);
        }
        if (c_up < n) {
            int at = 0;
#pragma unroll
            for (int r = 0; r < R; ++r) {
                if ((m[r] >> lane) & 1ull) buf[at + lanes_below(m[r])] = e[r];
                at += __popcll(m[r]);
            }
        }
        n = c_up;
        bound = fminf(bound, up);
        dirty = false;
    }
    // Takes the lanes' candidates; at most LIM entries stay.
    __device__ __forceinline__ void add(bool valid, float d, int32_t i) {
        const bool pass = valid && d <= bound;
        const unsigned long long m = ballot(pass);
        if (!m) return;
        if (pass)
            buf[n + lanes_below(m)] = ((unsigned long long)__float_as_uint(d) << 32) | (uint32_t)i;
        n += __popcll(m);
        dirty = true;
        if (n > LIM) cut<REGS>(LIM);
    }
    // Tightens the bound once the list holds k entries.
    __device__ __forceinline__ void tighten() {
        if (dirty && n >= k) cut<(LIM == WAVE ? REGS : REGS - 1)>(LIM);
    }
    // The same where the bound decides which cells of a ring are probed: one of
    // the (k + 8)-th distance lets many more pass when k is small (32,768 points
    // 10 m apart against themselves, k = 5: 560 loads a query, 1,538 us; so
    // 1,265.  40,000 queries 8 m off 10,000 points of a sweep, k = 1: 1,088, so
    // 806).
    __device__ __forceinline__ void tighten_close() {
        if (dirty && n >= k) cut<(LIM == WAVE ? REGS : REGS - 1), true>(LIM);
    }
    // At most a wavefront's entries.
    __device__ __forceinline__ void finish() {
        if (LIM > WAVE && n > WAVE) cut<REGS - 1>(WAVE);
    }
    // Whether k candidates are nearer than d2, or the radius is.
    __device__ __forceinline__ bool within(float d2) {
        if (d2 > bound) return true;
        if (n < k) return false;
        wave_lds_fence();
        const int lane = lane_id();
        int c = 0;
#pragma unroll
        for (int r = 0; r < LIM / WAVE; ++r) {
            const float d = __uint_as_float(
                lane + r * WAVE < n ? (uint32_t)(buf[lane + r * WAVE] >> 32) : ~0u);
            c += __popcll(ballot(d < d2));
        }
        return c >= k;
    }
};

// The nearest candidate alone (k = 1): each lane keeps its own best.
struct WaveNearest {
    static constexpr int k = 1;
    float bound;               // (uniform)
    float d;
    int32_t i;
    __device__ __forceinline__ void add(bool valid, float cd, int32_t ci) {
        if (valid && cd <= bound && key_less(cd, ci, d, i)) {
            d = cd;
            i = ci;
        }
    }
    __device__ __forceinline__ void tighten() { bound = fminf(bound, wave_min_nonneg(d)); }
    __device__ __forceinline__ void tighten_close() { tighten(); }
    __device__ __forceinline__ bool within(float d2) { return d2 > bound || ballot(d < d2) != 0; }
};

struct WaveQuery {
    float x, y, z;
    int skip;   // 64-record chunk of the points that has been taken already (-1: none)
};

// Stream the concatenated point runs of the cells held by lanes with `want`
// into the list, two batches of 64 candidates in flight.
template <typename List>
__device__ __forceinline__ void scan_points(const TargetView& T, const WaveQuery& q, bool want,
                                            int st, int total, int excl, List& L) {
    const int lane = lane_id();
    const int delta = st - excl;   // candidate f of the concatenation is point f + delta
    unsigned long long pend = ballot(want);
    int open = 0;                  // (uniform) delta of the last cell begun
    const auto next = [&](int b0) -> int {
        const int f = b0 + lane;
        int dl = open;
        while (pend) {
            const int cl = __builtin_ffsll((long long)pend) - 1;
            const int o = readlane(excl, cl);
            if (o >= b0 + WAVE) break;
            pend &= pend - 1;
            open = readlane(delta, cl);
            dl = f >= o ? open : dl;
        }
        const int src = f + dl;
        return f < total && (src >> 6) != q.skip ? src : -1;
    };
#pragma unroll 1
    for (int b0 = 0; b0 < total; b0 += 2 * WAVE) {
        const bool two = b0 + WAVE < total;
        const int s0 = next(b0);
        const int s1 = two ? next(b0 + WAVE) : -1;
        const float4 p0 = gload(T.pts + max(s0, 0));
        float4 p1 = p0;
        if (two) p1 = gload(T.pts + max(s1, 0));
        L.add(s0 >= 0, dist2(q.x, q.y, q.z, p0.x, p0.y, p0.z), __float_as_int(p0.w));
        if (two) L.add(s1 >= 0, dist2(q.x, q.y, q.z, p1.x, p1.y, p1.z), __float_as_int(p1.w));
    }
}

// The same through the cells' aligned 16-point runs: a lane tests one run's
// box against the bound, and four surviving runs make a batch.
template <typename List>
__device__ __forceinline__ void scan_runs(const TargetView& T, const WaveQuery& q, bool want,
                                          int st, int cn, float margin, List& L) {
    const int lane = lane_id();
    const int first = st / BOX_PTS, en = st + cn;
    const int nr = want ? (en - 1) / BOX_PTS - first + 1 : 0;
    const int incl = wave_incl_scan(nr), excl = incl - nr;
    const int total = readlane(incl, WAVE - 1);
    const int delta = first - excl;
    unsigned long long pend = ballot(want);
    int o_delta = 0, o_st = 0, o_en = 0;
#pragma unroll 1
    for (int b0 = 0; b0 < total; b0 += WAVE) {
        // this lane's run: the points [p0, p1) of one cell
        const int f = b0 + lane;
        int dl = o_delta, cs = o_st, ce = o_en;
        while (pend) {
            const int cl = __builtin_ffsll((long long)pend) - 1;
            const int o = readlane(excl, cl);
            if (o >= b0 + WAVE) break;
            pend &= pend - 1;
            o_delta = readlane(delta, cl);
            o_st = readlane(st, cl);
            o_en = readlane(en, cl);
            dl = f >= o ? o_delta : dl;
            cs = f >= o ? o_st : cs;
            ce = f >= o ? o_en : ce;
        }
        const int r = f + dl;
        const int p0 = max(r * BOX_PTS, cs), p1 = min((r + 1) * BOX_PTS, ce);
        const bool some = f < total && (p0 >> 6) != q.skip;
        float ld = INF;
        if (some) {
            const float4 lo = gload(T.boxes + 2 * r);
            const float4 hi = gload(T.boxes + 2 * r + 1);
            const float gx = fmaxf(fmaxf(lo.x - (q.x + margin), (q.x - margin) - hi.x), 0.0f);
            const float gy = fmaxf(fmaxf(lo.y - (q.y + margin), (q.y - margin) - hi.y), 0.0f);
            const float gz = fmaxf(fmaxf(lo.z - (q.z + margin), (q.z - margin) - hi.z), 0.0f);
            ld = fmaf(gx, gx, fmaf(gy, gy, gz * gz));
        }
        unsigned long long todo = ballot(some);
        for (;;) {
            // (the bound tightens as batches are added)
            todo &= ballot(ld <= L.bound * (1.0f + 2e-6f));
            if (!todo) break;
            int from = -1;
#pragma unroll
            for (int u = 0; u < WAVE / BOX_PTS; ++u) {
                if (todo) {
                    const int c = __builtin_ffsll((long long)todo) - 1;
                    todo &= todo - 1;
                    from = lane / BOX_PTS == u ? c : from;
                }
            }
            const int s = shfl(p0, from & 63) + lane % BOX_PTS, e = shfl(p1, from & 63);
            const bool valid = from >= 0 && s < e;
            const float4 p = gload(T.pts + (valid ? s : 0));
            L.add(valid, dist2(q.x, q.y, q.z, p.x, p.y, p.z), __float_as_int(p.w));
        }
    }
}

// Cells of many points go through their runs' boxes (one more dependent load,
// then only the near runs), cells of few are streamed whole.
constexpr int RUN_SCAN_MIN = 4 * WAVE;

template <typename List>
__device__ __forceinline__ void scan_cells(const TargetView& T, const WaveQuery& q, bool want,
                                           uint32_t start, uint32_t count, float margin, List& L) {
    const int c = want ? (int)count : 0;
    const int incl = wave_incl_scan(c);
    const int total = readlane(incl, WAVE - 1);
    if (total > RUN_SCAN_MIN)
        scan_runs(T, q, want, (int)start, (int)count, margin, L);
    else
        scan_points(T, q, want, (int)start, total, incl - c, L);
}

// The points of one cell.
template <typename List>
__device__ __forceinline__ void scan_one(const TargetView& T, const WaveQuery& q, int st, int cn,
                                         List& L) {
    const int lane = lane_id();
#pragma unroll 1
    for (int b0 = 0; b0 < cn; b0 += 2 * WAVE) {
        const bool two = b0 + WAVE < cn;
        const int f0 = b0 + lane, f1 = f0 + WAVE;
        const float4 p0 = gload(T.pts + st + min(f0, cn - 1));
        float4 p1 = p0;
        if (two) p1 = gload(T.pts + st + min(f1, cn - 1));
        L.add(f0 < cn, dist2(q.x, q.y, q.z, p0.x, p0.y, p0.z), __float_as_int(p0.w));
        if (two) L.add(f1 < cn, dist2(q.x, q.y, q.z, p1.x, p1.y, p1.z), __float_as_int(p1.w));
    }
}

// Squared distance from q to the box of cell c, shrunk by `margin` on every
// side to absorb the rounding of the float cell assignment.
__device__ __forceinline__ float box_dist2(const TargetView& T, float qx, float qy, float qz,
                                           int cx, int cy, int cz, float margin) {
    const float lx = (float)cx * T.cell - margin, hx = (float)(cx + 1) * T.cell + margin;
    const float ly = (float)cy * T.cell - margin, hy = (float)(cy + 1) * T.cell + margin;
    const float lz = (float)cz * T.cell - margin, hz = (float)(cz + 1) * T.cell + margin;
    const float dx = fmaxf(fmaxf(lx - qx, qx - hx), 0.0f);
    const float dy = fmaxf(fmaxf(ly - qy, qy - hy), 0.0f);
    const float dz = fmaxf(fmaxf(lz - qz, qz - hz), 0.0f);
    return dx * dx + dy * dy + dz * dz;
}

// Squared distance up to which no point lies outside the (2R+1)^3 block of
// cells around cell cq of query q (0 when not even the block's faces are
// clear of it).
__device__ __forceinline__ float block_clear2(float cell, const float (&q)[3], const int (&cq)[3],
                                              int R, float margin) {
    float f = INF;
    for (int a = 0; a < 3; ++a) {
        const float lo = (float)(cq[a] - R) * cell, hi = (float)(cq[a] + R + 1) * cell;
        f = fminf(f, fminf(q[a] - lo, hi - q[a]));
    }
    f = fmaxf(f - margin, 0.0f);
    return f * f * (1.0f - 1e-6f);
}

// Slack for the rounding of cell faces up to R + 2 cells from a query (`reach`:
// the largest |coordinate| of the query and the target).
__device__ __forceinline__ float wave_margin(float reach, float cell, int R) {
    return (reach + (float)(R + 2) * cell) * 1e-6f;
}

// What the wavefront search of a query starts from, all of it uniform.  The
// plans of a wavefront's next WAVE_PLANS queries are laid out together, a lane
// each: worked out one query at a time they were a quarter of the
// instructions of a k = 1 search (the same in every lane), and each began
// with a load of its own.
struct alignas(16) WavePlan {
    float x, y, z;
    int32_t qi;      // output row
    int cq[3];       // the query's cell
    int tgc;         // self queries: the query's own 64-record chunk; else the target
    int R, rmax;     // first and last ring (rmax < 0: nothing to search)
    float reach;     // largest |coordinate| of query and target
    float clear2;    // block_clear2 of the first ring
};
constexpr int WAVE_PLANS = 8;

__device__ __forceinline__ WavePlan wave_plan(const TargetView& V, float x, float y, float z,
                                              int32_t qi, int tgc, int capped, float radius) {
    WavePlan w;
    w.x = x;
    w.y = y;
    w.z = z;
    w.qi = qi;
    w.tgc = tgc;
    const float cell = V.cell, inv_cell = V.inv_cell;
    const float q[3] = {x, y, z};
    int R = 0, rmax = 0;
    // rings closer than the occupied box hold no cells: start at the first
    // ring that reaches it, end at the last
    for (int a = 0; a < 3; ++a) {
        const int c = cell_coord(q[a], inv_cell), lo = V.cmin[a], hi = V.cmax[a];
        w.cq[a] = c;
        R = max(R, max(lo - c, c - hi));
        rmax = max(rmax, max(c - lo, hi - c));
    }
    if (capped) {
        const float rc = ceilf(radius * inv_cell) + 1.0f;
        if (rc < (float)rmax) rmax = (int)rc;
    }
    w.R = R;
    w.rmax = finite3(x, y, z) && V.n_cells > 0 ? rmax : -1;
    w.reach = fmaxf(fmaxf(fabsf(x), fmaxf(fabsf(y), fabsf(z))), V.max_abs);
    w.clear2 = block_clear2(cell, q, w.cq, 1, wave_margin(w.reach, cell, 1));
    return w;
}

// The candidates of one query that hold its k nearest points, whole wavefront
// (q finite, the target not empty; L.bound starts at the radius).  `self`: the
// query is a point of the target, whose own 64-record chunk (its neighbours
// in Morton order) is taken first for a tight bound.  Then the query's own
// cell and its first ring, whose hash probes go out together (one chain of
// dependent loads rather than two; without a chunk the own cell is streamed
// first, so that its k-th distance prunes the ring), then ring by ring, or in
// one sweep of the cell table where a ring holds more cells than the table.
// (T is the copy of *Tp in scalar registers; what only a sweep reads is left
// in memory.)
template <typename List>
__device__ __forceinline__ void knn_query_wave(const TargetView& T, const TargetView* Tp,
                                               const WavePlan& w, bool self, List& L) {
    const int lane = lane_id();
    const float qx = w.x, qy = w.y, qz = w.z;
    const int cq[3] = {w.cq[0], w.cq[1], w.cq[2]};
    const float q[3] = {qx, qy, qz};
    const WaveQuery sp{qx, qy, qz, self ? w.tgc : -1};
    int R = w.R;
    const int rmax = w.rmax;
    if (self) {
        const int p = sp.skip * WAVE + lane;
        const float4 t = gload(T.pts + p);   // (64 spare records)
        L.add(p < (int)T.n, dist2(qx, qy, qz, t.x, t.y, t.z), __float_as_int(t.w));
        L.tighten();
    }
    bool found = false;
    uint32_t st = 0, cn = 0;
    float bd = INF;
    if (R == 0 && rmax >= 1) {
        const float margin = wave_margin(w.reach, T.cell, 1);
        // the 27 cells around cq, x fastest
        const int dz = (lane * 57) >> 9, r = lane - 9 * dz, dy = (r * 11) >> 5;
        const int cx = cq[0] + r - 3 * dy - 1, cy = cq[1] + dy - 1, cz = cq[2] + dz - 1;
        const bool own = lane == 13;
        if (lane < 27 && cx >= T.cmin[0] && cx <= T.cmax[0] && cy >= T.cmin[1] &&
            cy <= T.cmax[1] && cz >= T.cmin[2] && cz <= T.cmax[2]) {
            bd = box_dist2(T, qx, qy, qz, cx, cy, cz, margin) * (1.0f - 1e-6f);
            if (bd <= L.bound) found = hash_find(T, pack_key(T, cx, cy, cz), st, cn) && cn > 0;
        }
        int pass = self ? 1 : 0;
        if (!self) {
            const int oc = readlane(found ? (int)cn : 0, 13);
            if (oc <= RUN_SCAN_MIN) {
                // one cell of few points: no concatenation to work out
                if (oc > 0) {
                    scan_one(T, sp, readlane((int)st, 13), oc, L);
                    L.tighten();
                }
                pass = 1;
            }
        }
#pragma unroll 1
        for (; pass < 2; ++pass) {
            const bool want = found && (pass == 0 ? own : (self || !own) && bd <= L.bound);
            if (ballot(want)) scan_cells(T, sp, want, st, cn, margin, L);
            if (pass == 0) L.tighten();
        }
        if (L.within(w.clear2)) return;
        L.tighten_close();
        R = 2;
    }
#pragma unroll 1
    for (; R <= rmax; ++R) {
        const float margin = wave_margin(w.reach, T.cell, R);
        int lo[3], ext[3];
        int64_t total = 1;
        for (int a = 0; a < 3; ++a) {
            lo[a] = max(cq[a] - R, T.cmin[a]);
            ext[a] = max(min(cq[a] + R, T.cmax[a]) - lo[a] + 1, 0);
            total *= ext[a];
        }
        const bool sweep = total > 2 * (int64_t)T.n_cells + 256 || total > (int64_t)UINT32_MAX;
        // The ring's cells, face by face (clamped to the occupied box): the
        // two z faces whole, the y faces without the z faces' rows, the x
        // faces without both; R = 0 is the query's own cell.
        const int zi0 = max(cq[2] - R + 1, T.cmin[2]), zi1 = min(cq[2] + R - 1, T.cmax[2]);
        const int yi0 = max(cq[1] - R + 1, T.cmin[1]), yi1 = min(cq[1] + R - 1, T.cmax[1]);
        const uint32_t nz_in = (uint32_t)max(zi1 - zi0 + 1, 0), ny_in = (uint32_t)max(yi1 - yi0 + 1, 0);
        const uint32_t exy = (uint32_t)ext[0] * (uint32_t)ext[1];
        uint32_t fc[6];
        fc[0] = (R > 0 && cq[2] - R >= T.cmin[2]) ? exy : (R == 0 ? 1u : 0u);
        fc[1] = (R > 0 && cq[2] + R <= T.cmax[2]) ? exy : 0u;
        fc[2] = (R > 0 && cq[1] - R >= T.cmin[1]) ? (uint32_t)ext[0] * nz_in : 0u;
        fc[3] = (R > 0 && cq[1] + R <= T.cmax[1]) ? (uint32_t)ext[0] * nz_in : 0u;
        fc[4] = (R > 0 && cq[0] - R >= T.cmin[0]) ? ny_in * nz_in : 0u;
        fc[5] = (R > 0 && cq[0] + R <= T.cmax[0]) ? ny_in * nz_in : 0u;
        // (none when the ring misses the occupied box)
        const uint32_t steps = sweep ? (uint32_t)T.n_cells
                               : total > 0 ? fc[0] + fc[1] + fc[2] + fc[3] + fc[4] + fc[5] : 0u;
#pragma unroll 1
        for (uint32_t base = 0; base < steps; base += WAVE) {
            const uint32_t t = base + (uint32_t)lane;
            found = false;
            if (t < steps) {
                if (sweep) {
                    // every occupied cell not yet visited (Chebyshev ring >= R)
                    const unsigned long long mx = (1ull << T.sh_y) - 1ull;
                    const unsigned long long my = (1ull << (T.sh_z - T.sh_y)) - 1ull;
                    const unsigned long long key = Tp->cell_keys[t];
                    const int cx = (int)(key & mx) + T.cmin[0];
                    const int cy = (int)((key >> T.sh_y) & my) + T.cmin[1];
                    const int cz = (int)(key >> T.sh_z) + T.cmin[2];
                    const int cheb = max(abs(cx - cq[0]), max(abs(cy - cq[1]), abs(cz - cq[2])));
                    bd = box_dist2(T, qx, qy, qz, cx, cy, cz, margin) * (1.0f - 1e-6f);
                    if (cheb >= R && bd <= L.bound) {
                        st = Tp->cell_start[t];
                        cn = Tp->cell_start[t + 1] - st;
                        found = cn > 0;
                    }
                } else {
                    uint32_t u = t;
                    int f = 0;
#pragma unroll
                    for (int g = 0; g < 5; ++g) {
                        const bool past = f == g && u >= fc[g];
                        u = past ? u - fc[g] : u;
                        f = past ? g + 1 : f;
                    }
                    // rows of e cells along x (z and y faces) or along y (x faces)
                    const uint32_t e = f < 4 ? (uint32_t)ext[0] : max(ny_in, 1u);
                    const int v = (int)(u / e), r = (int)(u - (uint32_t)v * e);
                    const int cx = f < 4 ? lo[0] + r : cq[0] + (f == 5 ? R : -R);
                    const int cy = f < 2 ? lo[1] + v : f < 4 ? cq[1] + (f == 3 ? R : -R) : yi0 + r;
                    const int cz = f < 2 ? (R == 0 ? cq[2] : cq[2] + (f ? R : -R)) : zi0 + v;
                    bd = box_dist2(T, qx, qy, qz, cx, cy, cz, margin) * (1.0f - 1e-6f);
                    if (bd <= L.bound)
                        found = hash_find(T, pack_key(T, cx, cy, cz), st, cn) && cn > 0;
                }
            }
            if (ballot(found)) {
                scan_cells(T, sp, found, st, cn, margin, L);
                L.tighten_close();
            }
        }
        if (sweep || L.within(block_clear2(T.cell, q, cq, R, margin))) return;
    }
}

// Bounds the k-th distance by the farthest corners of the runs' boxes: ceil(k /
// 16) whole runs hold k points.  (In the operations of dist2, each of them
// monotonic: no point of a run is farther than its box's corner, rounding
// included.)
template <typename List>
__device__ __forceinline__ void bound_by_runs(const TargetView& T, const WaveQuery& q, List& L) {
    const int whole = (int)(T.n / BOX_PTS);
    float far = INF;   // of this lane's runs the nearest
#pragma unroll 1
    for (int r = lane_id(); r < whole; r += WAVE) {
        const float4 lo = gload(T.boxes + 2 * r);
        const float4 hi = gload(T.boxes + 2 * r + 1);
        far = fminf(far, dist2(0.0f, 0.0f, 0.0f, fmaxf(fabsf(lo.x - q.x), fabsf(hi.x - q.x)),
                               fmaxf(fabsf(lo.y - q.y), fabsf(hi.y - q.y)),
                               fmaxf(fabsf(lo.z - q.z), fabsf(hi.z - q.z))));
    }
    float b = INF;
#pragma unroll 1
    for (int held = 0; held < L.k; held += BOX_PTS) {
        b = wave_min_nonneg(far);
        const unsigned long long at = ballot(far == b);
        if (lane_id() == __builtin_ffsll((long long)at) - 1) far = INF;
    }
    L.bound = fminf(L.bound, b);
}

// The same from all points at once, through their 16-point runs (the own chunk
// of a self query first), for targets of up to RUNS_MAX_N points and sparse ones
// of up to RUNS_SPARSE_N (takes_runs).  Such a target's rings may be many and
// nearly empty: how many depends on where the queries lie, which the host does
// not know, and this is four (16) batches of boxes at most.  40,000 queries,
// k = 5, no radius, ring by ring and so:
//   2,048 points 12 m apart                                  2,277 / 57 us
//   a sweep thinned to 4,096, queries beside it, 8 m off   350 / 53, 728 / 89
//   4,096 points of a cube, 4 a cell                            54 / 66
//   6,000 (thinned sweep, cube)                          320 / 63, 56 / 72
// Up to RUN_SCAN_MIN points are streamed without the boxes.
constexpr int64_t RUNS_MAX_N = 4096, RUNS_SPARSE_N = 16384;

template <typename List>
__device__ __forceinline__ void knn_query_runs(const TargetView& T, const WavePlan& w, bool self,
                                               List& L) {
    const int lane = lane_id(), n = (int)T.n;
    const WaveQuery sp{w.x, w.y, w.z, self ? w.tgc : -1};
    if (n <= RUN_SCAN_MIN) {
        scan_one(T, sp, 0, n, L);
        return;
    }
    if (self) {
        const int p = sp.skip * WAVE + lane;
        const float4 t = gload(T.pts + p);   // (64 spare records)
        L.add(p < n, dist2(w.x, w.y, w.z, t.x, t.y, t.z), __float_as_int(t.w));
        L.tighten();
    }
    bound_by_runs(T, sp, L);
    scan_runs(T, sp, lane == 0, 0, n, 0.0f, L);
}

// ------------------------------------------------------------- covariance --

struct CovOut {
    float mean[3];
    float cov[6];   // xx xy xz yy yz zz
    float reg[6];
    bool valid;
};

// Unit eigenvector of the smallest eigenvalue of a symmetric 3x3 C (xx xy
// xz yy yz zz), by the closed form of its characteristic cubic (O. K. Smith,
// "Eigenvalues of a symmetric 3x3 matrix", CACM 4(4), 1961): with
// q = tr C / 3 and p^2 = |C - qI|_F^2 / 6, the eigenvalues are
// q + 2p cos(phi + 2 pi j / 3), phi = acos(det((C - qI) / p) / 2) / 3, and
// j = 1 gives the smallest, lambda.  Its eigenvector is the largest cross
// product of two rows of C - lambda I; the Rayleigh quotient of that vector
// refines lambda (acos loses digits when two eigenvalues are close) and the
// cross product is taken once more.  When lambda is (nearly) repeated, the
// rows of C - lambda I are (nearly) parallel to the other eigenvector and
// any vector orthogonal to the largest row spans the smallest eigenvalues'
// plane; C = qI (or 0) gives x.  No iteration: every lane runs the same
// instructions.  C is first scaled by a power of two (exactly) so that its
// largest entry lies in [1, 2).
__device__ __forceinline__ void eig_cross(const float (&c)[6], float lam, float (&e)[3],
                                          float& best, float& nrow) {
    const float m0[3] = {c[0] - lam, c[1], c[2]}, m1[3] = {c[1], c[3] - lam, c[4]},
                m2[3] = {c[2], c[4], c[5] - lam};
    const auto cross = [](const float (&u)[3], const float (&w)[3], float (&o)[3]) {
        o[0] = u[1] * w[2] - u[2] * w[1];
        o[1] = u[2] * w[0] - u[0] * w[2];
        o[2] = u[0] * w[1] - u[1] * w[0];
    };
    const auto norm2 = [](const float (&u)[3]) { return u[0] * u[0] + u[1] * u[1] + u[2] * u[2]; };
    float t[3];
    cross(m0, m1, e);
    best = norm2(e);
    cross(m0, m2, t);
    float nt = norm2(t);
    if (nt > best) {
        best = nt;
        e[0] = t[0]; e[1] = t[1]; e[2] = t[2];
    }
    cross(m1, m2, t);
    nt = norm2(t);
    if (nt > best) {
        best = nt;
        e[0] = t[0]; e[1] = t[1]; e[2] = t[2];
    }
    // the largest row
    const float n0 = norm2(m0), n1 = norm2(m1), n2 = norm2(m2);
    const float* rr = m0;
    nrow = n0;
    if (n1 > nrow) { nrow = n1; rr = m1; }
    if (n2 > nrow) { nrow = n2; rr = m2; }
    // rows (nearly) parallel: orthogonal to the largest row, through the
    // axis it has least of
    if (!(best > 1e-6f * nrow * nrow)) {
        if (nrow > 0.0f) {
            const float ax = fabsf(rr[0]), ay = fabsf(rr[1]), az = fabsf(rr[2]);
            const int k = (ax <= ay && ax <= az) ? 0 : (ay <= az ? 1 : 2);
            const float ek[3] = {k == 0 ? 1.0f : 0.0f, k == 1 ? 1.0f : 0.0f, k == 2 ? 1.0f : 0.0f};
            const float r3[3] = {rr[0], rr[1], rr[2]};
            cross(r3, ek, e);
            best = norm2(e);
        } else {
            e[0] = 1.0f; e[1] = 0.0f; e[2] = 0.0f;
            best = 1.0f;
        }
        nrow = -1.0f;   // degenerate: no refinement
    }
}

__device__ __forceinline__ void smallest_eigvec(const float (&cin)[6], float (&v0)[3]) {
    // scaled by a power of two (exact) to bring the largest entry to [1, 2):
    // the eigenvectors are unchanged and tiny covariances do not underflow
    float mx = 0.0f;
#pragma unroll
    for (int i = 0; i < 6; ++i) mx = fmaxf(mx, fabsf(cin[i]));
    if (!(mx > 0.0f)) {
        v0[0] = 1.0f;
        v0[1] = 0.0f;
        v0[2] = 0.0f;
        return;
    }
    const float sc = __int_as_float((254 - ((__float_as_int(mx) >> 23) & 0xff)) << 23);
    float c[6];
#pragma unroll
    for (int i = 0; i < 6; ++i) c[i] = cin[i] * sc;
    const float xx = c[0], xy = c[1], xz = c[2], yy = c[3], yz = c[4], zz = c[5];
    const float q = (xx + yy + zz) * (1.0f / 3.0f);
    const float d0 = xx - q, d1 = yy - q, d2 = zz - q;
    const float p1 = xy * xy + xz * xz + yz * yz;
    const float p2 = d0 * d0 + d1 * d1 + d2 * d2 + 2.0f * p1;
    float lam = q;
    if (p2 > 0.0f) {
        const float p = sqrtf(p2 * (1.0f / 6.0f));
        const float ip = 1.0f / p;
        const float b00 = d0 * ip, b11 = d1 * ip, b22 = d2 * ip;
        const float b01 = xy * ip, b02 = xz * ip, b12 = yz * ip;
        const float det = b00 * (b11 * b22 - b12 * b12) - b01 * (b01 * b22 - b12 * b02) +
                          b02 * (b01 * b12 - b11 * b02);
        const float r = fminf(fmaxf(0.5f * det, -1.0f), 1.0f);
        const float phi = acosf(r) * (1.0f / 3.0f);
        lam = q + 2.0f * p * cosf(phi + 2.09439510239319549f);   // + 2 pi / 3
    }
    float e[3], best, nrow;
    eig_cross(c, lam, e, best, nrow);
    if (nrow > 0.0f) {
        // Rayleigh quotient of e, then the cross product again
        const float ce0 = xx * e[0] + xy * e[1] + xz * e[2];
        const float ce1 = xy * e[0] + yy * e[1] + yz * e[2];
        const float ce2 = xz * e[0] + yz * e[1] + zz * e[2];
        lam = (e[0] * ce0 + e[1] * ce1 + e[2] * ce2) / best;
        eig_cross(c, lam, e, best, nrow);
    }
    const float inv = 1.0f / sqrtf(best);
    v0[0] = e[0] * inv;
    v0[1] = e[1] * inv;
    v0[2] = e[2] * inv;
}

__device__ __forceinline__ void cov_empty(CovOut& out) {
    for (int a = 0; a < 3; ++a) out.mean[a] = 0.0f;
    for (int e = 0; e < 6; ++e) out.cov[e] = 0.0f;
    out.reg[0] = 1.f; out.reg[1] = 0.f; out.reg[2] = 0.f;
    out.reg[3] = 1.f; out.reg[4] = 0.f; out.reg[5] = 1.f;
    out.valid = false;
}

// GICP plane regulariser I - (1 - eps) v0 v0^T (v0: smallest eigenvector
// of out.cov) for n >= 3 neighbours, else I.
__device__ __forceinline__ void cov_regularise(int n, float eps, CovOut& out) {
    out.valid = n >= 3;
    if (out.valid) {
        float v0[3];
        smallest_eigvec(out.cov, v0);
        const float w = 1.0f - eps;
        out.reg[0] = 1.0f - w * v0[0] * v0[0];
        out.reg[1] = -w * v0[0] * v0[1];
        out.reg[2] = -w * v0[0] * v0[2];
        out.reg[3] = 1.0f - w * v0[1] * v0[1];
        out.reg[4] = -w * v0[1] * v0[2];
        out.reg[5] = 1.0f - w * v0[2] * v0[2];
    } else {
        out.reg[0] = 1.f; out.reg[1] = 0.f; out.reg[2] = 0.f;
        out.reg[3] = 1.f; out.reg[4] = 0.f; out.reg[5] = 1.f;
    }
}

// Two-pass centred covariance of n neighbours relative to origin o, for at
// most NMAX neighbours whose offsets from o are in registers (all loads were
// in flight together).  The same operations in the same order in every kernel
// (covariance_offsets below), so their results agree bit for bit.
template <int NMAX>
__device__ __forceinline__ void covariance_n(float ox, float oy, float oz, int n,
                                             const float (&ux)[NMAX], const float (&uy)[NMAX],
                                             const float (&uz)[NMAX], float eps, CovOut& out) {
    if (n <= 0) {
        cov_empty(out);
        return;
    }
    float sx = 0.f, sy = 0.f, sz = 0.f;
#pragma unroll
    for (int j = 0; j < NMAX; ++j) {
        if (j < n) {
            sx += ux[j];
            sy += uy[j];
            sz += uz[j];
        }
    }
    const float inv_n = 1.0f / (float)n;
    const float mx = sx * inv_n, my = sy * inv_n, mz = sz * inv_n;
    float cxx = 0.f, cxy = 0.f, cxz = 0.f, cyy = 0.f, cyz = 0.f, czz = 0.f;
#pragma unroll
    for (int j = 0; j < NMAX; ++j) {
        if (j < n) {
            const float dx = ux[j] - mx, dy = uy[j] - my, dz = uz[j] - mz;
            cxx = fmaf(dx, dx, cxx);
            cxy = fmaf(dx, dy, cxy);
            cxz = fmaf(dx, dz, cxz);
            cyy = fmaf(dy, dy, cyy);
            cyz = fmaf(dy, dz, cyz);
            czz = fmaf(dz, dz, czz);
        }
    }
    out.cov[0] = cxx * inv_n;
    out.cov[1] = cxy * inv_n;
    out.cov[2] = cxz * inv_n;
    out.cov[3] = cyy * inv_n;
    out.cov[4] = cyz * inv_n;
    out.cov[5] = czz * inv_n;
    out.mean[0] = ox + mx;
    out.mean[1] = oy + my;
    out.mean[2] = oz + mz;
    cov_regularise(n, eps, out);
}

// Exponent of the kernel descriptor for squared distance d2.
__device__ __forceinline__ float weight_exponent(const CovWeight& W, float d2) {
    return W.kind == LKC_WEIGHT_LAPLACIAN ? sqrtf(d2) * W.scale : d2 * W.scale;
}

// Kernel-descriptor weighted covariance (the paper's table of kernel
// descriptors, Sec. III-C.1): neighbour j of the query at o gets
// w_j = K(o, t_j) / max_j K(o, t_j) = exp(-(e_j - min e)); the rescaling
// leaves the normalised estimate unchanged, keeps the weights in (0, 1] and
// makes the sum >= 1.  Three passes relative to o: the smallest exponent,
// the weighted mean, the weighted centred second moment; both divided by
// the weight sum.  Validity and the regulariser are those of the plain
// estimate.  For k_group; covariance_offsets takes the same operations in the
// same order elsewhere, so that the results agree bit for bit.
template <typename Fetch>
__device__ __forceinline__ void covariance_weighted(float ox, float oy, float oz, int n,
                                                    Fetch fetch, const CovWeight& W, float eps,
                                                    CovOut& out) {
    if (n <= 0) {
        cov_empty(out);
        return;
    }
    float emin = INF;
    for (int j = 0; j < n; ++j) {
        const float4 t = fetch(j);
        emin = fminf(emin, weight_exponent(W, dist2(ox, oy, oz, t.x, t.y, t.z)));
    }
    float sw = 0.f, sx = 0.f, sy = 0.f, sz = 0.f;
    for (int j = 0; j < n; ++j) {
        const float4 t = fetch(j);
        const float w = expf(emin - weight_exponent(W, dist2(ox, oy, oz, t.x, t.y, t.z)));
        sw += w;
        sx = fmaf(w, t.x - ox, sx);
        sy = fmaf(w, t.y - oy, sy);
        sz = fmaf(w, t.z - oz, sz);
    }
    const float mx = sx / sw, my = sy / sw, mz = sz / sw;
    float cxx = 0.f, cxy = 0.f, cxz = 0.f, cyy = 0.f, cyz = 0.f, czz = 0.f;
    for (int j = 0; j < n; ++j) {
        const float4 t = fetch(j);
        const float w = expf(emin - weight_exponent(W, dist2(ox, oy, oz, t.x, t.y, t.z)));
        const float dx = (t.x - ox) - mx, dy = (t.y - oy) - my, dz = (t.z - oz) - mz;
        const float wx = w * dx, wy = w * dy, wz = w * dz;
        cxx = fmaf(wx, dx, cxx);
        cxy = fmaf(wx, dy, cxy);
        cxz = fmaf(wx, dz, cxz);
        cyy = fmaf(wy, dy, cyy);
        cyz = fmaf(wy, dz, cyz);
        czz = fmaf(wz, dz, czz);
    }
    out.cov[0] = cxx / sw;
    out.cov[1] = cxy / sw;
    out.cov[2] = cxz / sw;
    out.cov[3] = cyy / sw;
    out.cov[4] = cyz / sw;
    out.cov[5] = czz / sw;
    out.mean[0] = ox + mx;
    out.mean[1] = oy + my;
    out.mean[2] = oz + mz;
    cov_regularise(n, eps, out);
}

// The same estimates, in the same operations and order, from neighbours whose
// offsets from o (and weights) have been taken before: fetch(j) returns
// (t_j - o, w_j).
template <bool WEIGHTED, typename Fetch>
__device__ __forceinline__ void covariance_offsets(float ox, float oy, float oz, int n, Fetch fetch,
                                                   float eps, CovOut& out) {
    if (n <= 0) {
        cov_empty(out);
        return;
    }
    float sw = 0.f, sx = 0.f, sy = 0.f, sz = 0.f;
#pragma unroll 4
    for (int j = 0; j < n; ++j) {
        const float4 u = fetch(j);
        if (WEIGHTED) {
            sw += u.w;
            sx = fmaf(u.w, u.x, sx);
            sy = fmaf(u.w, u.y, sy);
            sz = fmaf(u.w, u.z, sz);
        } else {
            sx += u.x;
            sy += u.y;
            sz += u.z;
        }
    }
    const float inv_n = 1.0f / (float)n;
    const float mx = WEIGHTED ? sx / sw : sx * inv_n, my = WEIGHTED ? sy / sw : sy * inv_n,
                mz = WEIGHTED ? sz / sw : sz * inv_n;
    float c[6] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll 4
    for (int j = 0; j < n; ++j) {
        const float4 u = fetch(j);
        const float dx = u.x - mx, dy = u.y - my, dz = u.z - mz;
        const float wx = WEIGHTED ? u.w * dx : dx, wy = WEIGHTED ? u.w * dy : dy,
                    wz = WEIGHTED ? u.w * dz : dz;
        c[0] = fmaf(wx, dx, c[0]);
        c[1] = fmaf(wx, dy, c[1]);
        c[2] = fmaf(wx, dz, c[2]);
        c[3] = fmaf(wy, dy, c[3]);
        c[4] = fmaf(wy, dz, c[4]);
        c[5] = fmaf(wz, dz, c[5]);
    }
#pragma unroll
    for (int e = 0; e < 6; ++e) out.cov[e] = WEIGHTED ? c[e] / sw : c[e] * inv_n;
    out.mean[0] = ox + mx;
    out.mean[1] = oy + my;
    out.mean[2] = oz + mz;
    cov_regularise(n, eps, out);
}

struct CovPtrs {
    float* mean;
    float* cov;
    float* reg;
    uint8_t* valid;
};

__device__ __forceinline__ void store_sym(float* dst, const float (&s)[6]) {
    dst[0] = s[0]; dst[1] = s[1]; dst[2] = s[2];
    dst[3] = s[1]; dst[4] = s[3]; dst[5] = s[4];
    dst[6] = s[2]; dst[7] = s[4]; dst[8] = s[5];
}

__device__ __forceinline__ void store_cov(const CovPtrs& o, int64_t qi, const CovOut& c) {
    if (o.mean) {
        o.mean[3 * qi + 0] = c.mean[0];
        o.mean[3 * qi + 1] = c.mean[1];
        o.mean[3 * qi + 2] = c.mean[2];
    }
    if (o.cov) store_sym(o.cov + 9 * qi, c.cov);
    if (o.reg) store_sym(o.reg + 9 * qi, c.reg);
    o.valid[qi] = c.valid ? 1 : 0;
}

struct KnnPtrs {
    int32_t* idx;
    float* d2;
    int32_t* count;
};

// ---------------------------------------------------------- group search --
//
// Lane-per-query search over queries sorted by grid cell.  A wavefront takes
// 64 consecutive sorted queries (a "group": they sit in one or a few
// neighbouring cells), probes the cells of the group's block (its cells
// grown by R on every side) in parallel, and streams every surviving cell's
// point run once for the whole group: the candidate address is the same in
// all lanes, so each load is one coalesced read.  Each lane keeps its own
// sorted top-k (+ SLACK spare entries) in registers as 32-bit packed keys
// (the float d2 bits with the low ID_BITS replaced by the candidate's name,
// see below), decoded to the exact (d2, index) order at the end.  A lane
// whose result the block cannot prove exact (the k-th distance, or the
// radius, reaches past the block), or whose packed order is ambiguous, is
// handed to the wavefront-per-query search through a fallback list.

constexpr int GROUP_W = 2;       // lanes within this many cells of a round's anchor take part
constexpr int64_t WHOLE_N = 4096;  // targets this small are streamed whole by every group

// Batcher's odd-even merge sort on P = 2^ceil(log2 K) inputs, keeping the
// comparators between the first K (the others would compare with +inf
// padding and never swap).  Built at compile time.
template <int K>
struct SortNet {
    static constexpr int P = K <= 8 ? 8 : (K <= 16 ? 16 : (K <= 32 ? 32 : 64));
    int a[P * 8], b[P * 8];
    int n;
    constexpr SortNet() : a(), b(), n(0) {
        for (int p = 1; p < P; p += p)
            for (int k = p; k >= 1; k /= 2)
                for (int j = k % p; j + k <= P - 1; j += 2 * k)
                    for (int i = 0; i <= k - 1 && i <= P - j - k - 1; ++i)
                        if ((i + j) / (2 * p) == (i + j + k) / (2 * p) && i + j + k < K) {
                            a[n] = i + j;
                            b[n] = i + j + k;
                            ++n;
                        }
    }
};

struct GroupArgs {
    const TargetView* views;          // device array, one per target
    const float* queries;             // [q][3]; NULL: the queries are the target's own points
    const uint32_t* order;            // sorted slot -> query index (NULL with self queries)
    // query keys, target index in bits >= tshift: sorted for the group
    // search, by query without it (NULL: one target)
    const unsigned long long* skeys;
    int tshift;
    int R;                            // block reach in cells
    int64_t n_slots;
    SearchParams sp;
    KnnPtrs ko;
    CovPtrs co;
    float eps;
    CovWeight wt;                     // covariance weights (fused mode 2)
    uint32_t* fb_list;                // slots handed to the wavefront search (NULL: every slot)
    uint32_t* fb_count;
    uint32_t* counters;               // per-XCD work counters (persistent mode) or NULL
    uint32_t* prof;                   // optional per-group counters (PROF_WORDS each) or NULL
    int split;                        // waves per group (1, 2 or 4)
    int rounds;                       // anchor rounds per group (lanes left fall back)
    int cov_slots;                    // rows a wavefront of the wavefront search keeps for their covariances
    int moved;                        // the wavefront search moves its queries by `move`
    RigidF move;
};

// Waves sharing a group: each streams the chunks it owns (chunk index
// modulo the split) and publishes its lanes' k-th distances here; the others
// prune with the smallest of them, which is still an upper bound of the
// final k-th distance (each list holds k distinct candidates).
struct SplitShare {
    volatile float* thr;     // [split][64]
    volatile uint32_t* flag; // [split][64]: lanes a wave cannot answer exactly
    uint32_t* dist;          // [split / 2][K][64]: merge buffers (d2 bits)
    uint32_t* pos;           // [split / 2][K][64]: and the entries' positions
    int sub;                 // this wave's index in the group
    int split_mask;          // split - 1
};

__device__ __forceinline__ float shared_thr(const SplitShare& sh, int lane, float own) {
    for (int w = 0; w <= sh.split_mask; ++w)
        if (w != sh.sub) own = fminf(own, sh.thr[w * WAVE + lane]);
    return own;
}

// per-group profile words: clock cycles, probe rounds, cells streamed,
// 64-point chunks loaded, candidates tested, insertion pops, member lanes,
// fallback lanes, insertions (over all lanes), pops in which no lane
// inserted; then insertions and candidates split by phase: the cells holding
// the queries, the surrounding cells, a small target streamed whole; then
// insertions from the group's own chunk (self queries); then the lanes
// handed on because their decoded entries stayed out of order or tied, because
// the last entry shared the k-th distance's bucket, or because the wave ran
// out of chunk names; then clock cycles of the first wavefront in the
// streaming (probes and chunks), in decoding and merging the lists, and in
// the covariances; then the 16-point runs tested against the members'
// bounds and those some member's bound kept
constexpr int PROF_WORDS = 25;
// A profile counter that compiles away in the unprofiled kernels (their
// counters are never read, so the arithmetic feeding them is dead).
template <bool ON>
struct ProfCount {
    uint32_t v = 0;
    __device__ ProfCount& operator++() {
        if (ON) ++v;
        return *this;
    }
    __device__ void operator++(int) {
        if (ON) ++v;
    }
    __device__ ProfCount& operator+=(uint32_t x) {
        if (ON) v += x;
        return *this;
    }
    __device__ operator uint32_t() const { return ON ? v : 0u; }
};
template <bool ON>
struct GroupProf {
    ProfCount<ON> probes, cells, chunks, cands, pops, inserts, dead;
    ProfCount<ON> ins0, ins1, ins2, cand0, cand1, cand2, own;
    ProfCount<ON> amb_order, amb_bucket, amb_names;
    ProfCount<ON> t_walk, t_final, t_cov, runs_grp, runs_kept;
};

struct SlotQuery {
    int64_t qi;   // output row
    float x, y, z;
    int tgt;
};

__device__ __forceinline__ SlotQuery load_slot(const GroupArgs& a, const TargetView& T, int64_t slot) {
    SlotQuery s;
    s.tgt = a.skeys ? (int)(a.skeys[slot] >> a.tshift) : 0;
    if (a.queries) {
        s.qi = a.order ? (int64_t)gload(a.order + slot) : slot;
        s.x = gload(a.queries + 3 * s.qi);
        s.y = gload(a.queries + 3 * s.qi + 1);
        s.z = gload(a.queries + 3 * s.qi + 2);
    } else {
        const float4 p = gload(T.pts + slot);
        s.qi = __float_as_int(p.w);
        s.x = p.x;
        s.y = p.y;
        s.z = p.z;
    }
    return s;
}

// Packed insertion keys.  While a block is streamed, a lane keeps its
// nearest candidates as 32-bit keys: the float32 bits of d2 with the low
// ID_BITS bits replaced by the candidate's name (the ordinal of its 64-point
// chunk in the wave's stream of this round, and its lane in that chunk).
// Non-negative floats order as their bits, so the key order is the d2 order
// up to buckets of 2^-9 relative width, and the name order inside a bucket.
// A sorted list of such keys takes a candidate with one v_med3_u32 per entry
// (the median of the entry before, the candidate and the entry itself is the
// entry's new value), where a sorted list of exact 64-bit (d2, index) keys
// costs a compare and four selects per entry.  The list holds SLACK entries
// past the k-th.  When the block is done every entry is decoded to its exact
// (d2, index) key and the k smallest of those are the exact result, unless
// the last entry's bucket is the exact k-th distance's bucket: a candidate
// the list dropped may then tie with the k-th inside the bucket, and the lane
// is handed to the wavefront-per-query search.  Ordinals start at 1, so
// that a real key is never 0, the value of the front pads of a list for
// k < K.
constexpr int SLACK = 4;
constexpr int ID_BITS = 14;
constexpr uint32_t ID_MASK = (1u << ID_BITS) - 1u;
constexpr int MAX_CHUNKS = 1 << (ID_BITS - 6);   // chunk ordinals (0 unused)

__device__ __forceinline__ uint32_t med3_u32(uint32_t a, uint32_t x, uint32_t b) {
    uint32_t r;
    asm("v_med3_u32 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(x), "v"(b));
    return r;
}

// The position of the lowest set bit of x, ~0u when x is 0.
__device__ __forceinline__ uint32_t ffbl_u32(uint32_t x) {
    uint32_t r;
    asm("v_ffbl_b32 %0, %1" : "=v"(r) : "v"(x));
    return r;
}

// 2 b + (d <= t): the compare's lane mask is the add's carry in (the two
// wait states are the ones a mask written by a VALU compare needs before a
// VALU instruction reads it).
__device__ __forceinline__ uint32_t shift_in_le(uint32_t b, float d, float t) {
    uint32_t r;
    unsigned long long m;
    asm("v_cmp_le_f32_e64 %1, %3, %4\n\ts_nop 1\n\tv_addc_co_u32_e64 %0, %1, %2, %2, %1"
        : "=v"(r), "=&s"(m)
        : "v"(b), "v"(d), "v"(t));
    return r;
}

typedef uint32_t u32x16 __attribute__((ext_vector_type(16)));

// The 128 bytes at p (wavefront-uniform, read-only) as two 64-byte scalar
// loads.  The wait stays inside the statement: the compiler takes an asm
// statement's outputs as written when it ends.
__device__ __forceinline__ void load_boxes64(const float4* p, u32x16& a, u32x16& b) {
    asm volatile("s_load_dwordx16 %0, %2, 0x0\n\ts_load_dwordx16 %1, %2, 0x40\n\ts_waitcnt lgkmcnt(0)"
                 : "=&s"(a), "=&s"(b)
                 : "s"(p)
                 : "memory");
}

// Insert x into the ascending list L; a no-op when x is not below L[N-1].
template <int N>
__device__ __forceinline__ void pk_insert(uint32_t (&L)[N], uint32_t x) {
#pragma unroll
    for (int j = N - 1; j >= 1; --j) L[j] = med3_u32(L[j - 1], x, L[j]);
    L[0] = min(L[0], x);
}

// Insert x (below D[K-1]) into the ascending 32-bit list D, its payload xp
// moving into P alongside.
template <int K>
__device__ __forceinline__ void insert_p(uint32_t (&D)[K], uint32_t (&P)[K], uint32_t x,
                                         uint32_t xp) {
    bool c_hi = x < D[K - 1];
#pragma unroll
    for (int j = K - 1; j >= 1; --j) {
        const bool c_lo = x < D[j - 1];
        const uint32_t tp = c_hi ? xp : P[j];
        P[j] = c_lo ? P[j - 1] : tp;
        D[j] = med3_u32(D[j - 1], x, D[j]);
        c_hi = c_lo;
    }
    P[0] = c_hi ? xp : P[0];
    D[0] = min(D[0], x);
}

// A lane's pruning bound: the top of its k-th entry's bucket (the radius
// while it holds fewer than k entries), never above its bound lcap.  The
// k-th entry sits at K - 1: k < K lists start with K - k zero pads.
template <int K>
__device__ __forceinline__ float pk_bound(const uint32_t (&L)[K + SLACK], float r2, float lcap) {
    // all three are non-negative floats (an empty entry's ~0u is above
    // every one), which order as their bits
    return __uint_as_float(
        min(min(L[K - 1] | ID_MASK, __float_as_uint(r2)), __float_as_uint(lcap)));
}

// Sort 32-bit keys ascending in registers.
template <int N>
__device__ __forceinline__ void sort_u32(uint32_t (&L)[N]) {
    constexpr SortNet<N> net{};
#pragma unroll
    for (int c = 0; c < net.n; ++c) {
        const uint32_t x = L[net.a[c]], y = L[net.b[c]];
        L[net.a[c]] = min(x, y);
        L[net.b[c]] = max(x, y);
    }
}

// Stream the reordered points [s0, e0) through every member lane's list.
// The run is walked in aligned 64-point chunks made of four 16-point runs
// with their own bounding boxes; a 16-point run whose box is farther from
// every member's query than that member's own bound (never above the
// radius) is skipped.  (A test of the run's box against the members' query
// box would be implied by this one: it only ever saved the per-lane test,
// at a cost above that test's.)  A kept chunk
// is named (its ordinal in this wave's stream, recorded in s_tab; fixed_ord
// names a chunk the caller registered); each candidate is broadcast from its lane and
// tested by every lane, which only sets a bit per passing candidate; the
// insertions follow as "pops" in which every lane inserts its own next
// passing candidate, so a chunk costs as many insertion steps as its busiest
// lane needs rather than one per candidate that any lane wants.  A wave that
// runs out of names sets n_ch past MAX_CHUNKS (its members fall back).
template <int K, bool PROF>
__device__ __forceinline__ void scan_run(const TargetView& T, int s0, int e0, bool member,
                                         float qx, float qy, float qz, float r2, float lcap,
                                         float3 qlo, float3 qhi, uint32_t (&L)[K + SLACK],
                                         GroupProf<PROF>& gp, int skip_cb,
                                         const SplitShare& sh, int& n_ch, uint32_t* s_tab,
                                         int fixed_ord = -1, int win_k = 0, int win_n = 0) {
    const int lane = lane_id();
#pragma unroll 1
    for (int cb = s0 & ~(WAVE - 1); cb < e0; cb += WAVE) {
        if (cb == skip_cb) continue;   // streamed first, as the group's own chunk
        if (((cb / WAVE) & sh.split_mask) != sh.sub) continue;   // the other wave's chunk
        // the chunk's load goes out with its boxes' (lane t holds point t,
        // one coalesced read; padded: reads past n stay in bounds)
        const float4 c = gload(T.pts + cb + lane);
        // and so do the boxes of its four runs (two 64-byte scalar loads; the
        // boxes carry 4 spare runs)
        u32x16 bw[2];
        load_boxes64(T.boxes + 2 * (cb / BOX_PTS), bw[0], bw[1]);
        uint32_t keep = 0;
        float lthr = pk_bound<K>(L, r2, lcap);
        if (sh.split_mask) lthr = shared_thr(sh, lane, lthr);
        // a run is kept when its box is within some member's bound of that
        // member's query box widened by the margin (non-members: never)
        const float bthr = member ? lthr * (1.0f + 2e-6f) : -1.0f;
#pragma unroll
        for (int q4 = 0; q4 < WAVE / BOX_PTS; ++q4) {
            const int sb = cb + q4 * BOX_PTS;
            if (sb + BOX_PTS <= s0 || sb >= e0) continue;
            const u32x16& w = bw[q4 >> 1];
            const int o = 8 * (q4 & 1);
            const float3 blo = make_float3(__uint_as_float(w[o]), __uint_as_float(w[o + 1]),
                                           __uint_as_float(w[o + 2]));
            const float3 bhi = make_float3(__uint_as_float(w[o + 4]), __uint_as_float(w[o + 5]),
                                           __uint_as_float(w[o + 6]));
            gp.runs_grp++;
            const float gx = fmaxf(fmaxf(blo.x - qhi.x, qlo.x - bhi.x), 0.0f);
            const float gy = fmaxf(fmaxf(blo.y - qhi.y, qlo.y - bhi.y), 0.0f);
            const float gz = fmaxf(fmaxf(blo.z - qhi.z, qlo.z - bhi.z), 0.0f);
            const float ld = fmaf(gx, gx, fmaf(gy, gy, gz * gz));
            if (ballot(ld <= bthr)) {
                keep |= 1u << q4;
                gp.runs_kept++;
            }
        }
        if (!keep) continue;
        int ord = fixed_ord;
        if (ord < 0) {
            if (n_ch >= MAX_CHUNKS) {
                n_ch = MAX_CHUNKS + 1;
                continue;
            }
            ord = n_ch++;   // n_ch starts at 1
            if (lane == 0) s_tab[ord] = (uint32_t)(cb / WAVE);
        }
        gp.chunks++;
        // non-members never pass (d2 >= 0)
        const float tthr = member ? lthr : -1.0f;
        uint32_t blo = 0, bhi = 0;
        const int lo = max(s0, cb) - cb, hi = min(e0, cb + WAVE) - cb;
#pragma unroll 1
        for (int q4 = 0; q4 < WAVE / BOX_PTS; ++q4) {
            if (!((keep >> q4) & 1u)) continue;
            const int t1 = min(hi, (q4 + 1) * BOX_PTS);
            gp.cands += (uint32_t)max(0, t1 - max(lo, q4 * BOX_PTS));
            // Descending: each test doubles the word and adds its outcome,
            // so candidate t ends at bit t - t0.
            const int t0 = max(lo, q4 * BOX_PTS);
            uint32_t b = 0;
#pragma unroll 2
            for (int t = t1 - 1; t >= t0; --t) {
                const float cx = readlane(c.x, t), cy = readlane(c.y, t), cz = readlane(c.z, t);
                b = shift_in_le(b, dist2(qx, qy, qz, cx, cy, cz), tthr);
            }
            b <<= (t0 & 31);
            if (q4 < 2)
                blo |= b;
            else
                bhi |= b;
        }
        unsigned long long bits = ((unsigned long long)bhi << 32) | blo;
        if (win_k) {
            // a member's window of win_k slots (of the win_n active ones)
            // is already in its list
            const int w0 = min(max(lane - (win_k - 1) / 2, 0), win_n - win_k);
            bits &= member ? ~(((1ull << win_k) - 1ull) << w0) : ~0ull;
        }
        if (!ballot(bits != 0ull)) continue;
        const uint32_t name0 = (uint32_t)ord << 6;
        // Each lane's next passing candidate (lane 63 when none: read, not
        // inserted) is fetched one pop ahead, so the fetch overlaps the
        // insertion chain of the current one.
        auto fetch = [&](uint32_t jj, float& fx, float& fy, float& fz) {
            const int ja = (int)(jj << 2);
            fx = __int_as_float(__builtin_amdgcn_ds_bpermute(ja, __float_as_int(c.x)));
            fy = __int_as_float(__builtin_amdgcn_ds_bpermute(ja, __float_as_int(c.y)));
            fz = __int_as_float(__builtin_amdgcn_ds_bpermute(ja, __float_as_int(c.z)));
        };
        // The lowest set bit of a lane's mask, ~0u when it is empty: the
        // empty lane's key is then ~0u, which inserts nothing, and its fetch
        // reads lane 63.
        auto first = [](unsigned long long m) -> uint32_t {
            return min(ffbl_u32((uint32_t)m), ffbl_u32((uint32_t)(m >> 32)) | 32u);
        };
        auto insert = [&](uint32_t jj, float px, float py, float pz) {
            gp.pops++;
            // d2 <= the lane's bound <= r2: within the radius
            const uint32_t db = __float_as_uint(dist2(qx, qy, qz, px, py, pz));
            const uint32_t x = (db & ~ID_MASK) | name0 | jj;
            if (PROF) {
                const unsigned long long im = ballot(x < L[K + SLACK - 1]);
                gp.inserts += (uint32_t)__popcll(im);
                gp.dead += im ? 0u : 1u;
            }
            pk_insert<K + SLACK>(L, x);
        };
        // Unrolled by two so that the candidate fetched ahead needs no copy.
        uint32_t j = first(bits);
        bits &= bits - 1ull;
        float cx, cy, cz;
        fetch(j, cx, cy, cz);
        for (;;) {
            const uint32_t jn = first(bits);
            bits &= bits - 1ull;
            float nx, ny, nz;
            fetch(jn, nx, ny, nz);
            insert(j, cx, cy, cz);
            if (!ballot(jn != ~0u)) break;
            j = first(bits);
            bits &= bits - 1ull;
            fetch(j, cx, cy, cz);
            insert(jn, nx, ny, nz);
            if (!ballot(j != ~0u)) break;
        }
        // publish the lane's bound to the group's other waves
        if (sh.split_mask) sh.thr[sh.sub * WAVE + lane] = pk_bound<K>(L, r2, lcap);
    }
}

// A lane's row of K words, four to a store (rows are only known to be aligned
// to a word).  Every lane's row lies in lines of its own, and a store takes a
// cycle of the address unit for each line: word by word, the two rows of a
// k = 20 query were 40 of the group search's 49 stores, and the address units
// busy 66 % of the batched launch (3.76 M queries, 1.19 ms); in quads 41 %
// (1.07 ms), and the instructions issued bound it again.
typedef uint32_t row4 __attribute__((ext_vector_type(4), aligned(4)));

template <int K>
__device__ __forceinline__ void store_row(uint32_t* dst, const uint32_t (&v)[K]) {
    static_assert(K % 4 == 0, "rows of whole quads");
#pragma unroll
    for (int j = 0; j < K; j += 4) *(row4*)(dst + j) = row4{v[j], v[j + 1], v[j + 2], v[j + 3]};
}

// Write one query's neighbour row from the ascending exact d2 bits D and
// the points' positions P in the reordered array (K - k pads first, ~0u
// empty): d2 and the count; the indices too unless the fused covariance
// writes them as it gathers the points (positions left in s_pos, column c
// at s_pos[(K - k + c) * 64 + lane]).  Returns the count.
template <int K, int FUSED>
__device__ __forceinline__ int emit_row(const GroupArgs& a, const TargetView& T, int64_t qi,
                                        int k, const uint32_t (&D)[K], const uint32_t (&P)[K],
                                        uint32_t* s_pos) {
    int cnt = 0;
    int32_t* ip = a.ko.idx + qi * k - (K - k);   // entry j is column j - (K - k)
    float* dp = a.ko.d2 + qi * k - (K - k);
    const int lane = lane_id();
    if (k == K) {
        // no pads: whole rows
        uint32_t d[K];
#pragma unroll
        for (int j = 0; j < K; ++j) {
            const bool have = D[j] != ~0u;
            d[j] = have ? D[j] : __float_as_uint(INF);
            cnt += have ? 1 : 0;
            if (FUSED) s_pos[j * WAVE + lane] = P[j];
        }
        store_row((uint32_t*)dp, d);
        if (!FUSED) {
#pragma unroll
            for (int j = 0; j < K; ++j)
                d[j] = D[j] != ~0u ? __float_as_uint(gload(T.pts + P[j]).w) : ~0u;
            store_row((uint32_t*)ip, d);
        }
        a.ko.count[qi] = cnt;
        return cnt;
    }
#pragma unroll
    for (int j = 0; j < K; ++j) {
        if (P[j] != ~0u) {   // not a pad
            const bool have = D[j] != ~0u;
            dp[j] = have ? __uint_as_float(D[j]) : INF;
            if (!FUSED) ip[j] = have ? __float_as_int(gload(T.pts + P[j]).w) : -1;
            if (FUSED && !have) ip[j] = -1;
            cnt += have ? 1 : 0;
        }
        if (FUSED) s_pos[j * WAVE + lane] = P[j];
    }
    a.ko.count[qi] = cnt;
    return cnt;
}

// The covariance of a written row: its first cnt neighbours, gathered from
// the reordered points (the copy the search has just streamed through the
// caches; the same values as the caller-order copy) by the positions in sp
// (column c at sp[c * 64], LDS), then the row's indices.  Restrict-qualified
// so that the gathers of a pass can all be in flight together.
// (k == K: the row is written whole, -1 past cnt, here; else only its first cnt
// entries, the rest by emit_row.)
template <int K, int FUSED>
__device__ __forceinline__ void cov_gather(const float4* __restrict__ pts,
                                           const uint32_t* __restrict__ sp,
                                           uint32_t* __restrict__ irow, const GroupArgs& a,
                                           int64_t qi, float qx, float qy, float qz, int k,
                                           int cnt) {
    CovOut c;
    if (FUSED == 1) {
        // each neighbour gathered once, its index written on the way (eight
        // gathers in flight: with all of them the offsets and the indices do
        // not fit the registers)
        float ux[K], uy[K], uz[K];
#pragma unroll
        for (int j0 = 0; j0 < K; j0 += 4) {
            uint32_t w[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int j = j0 + u;
                w[u] = ~0u;
                ux[j] = uy[j] = uz[j] = 0.0f;
                if (j < cnt) {
                    const float4 t = gload(pts + sp[j * WAVE]);
                    ux[j] = t.x - qx;
                    uy[j] = t.y - qy;
                    uz[j] = t.z - qz;
                    w[u] = __float_as_uint(t.w);
                }
            }
            if (k == K) {
                store_row(irow + j0, w);
            } else {
#pragma unroll
                for (int u = 0; u < 4; ++u)
                    if (j0 + u < cnt) irow[j0 + u] = w[u];
            }
            if (j0 % 8 == 4) __builtin_amdgcn_sched_barrier(0);
        }
        covariance_n<K>(qx, qy, qz, cnt, ux, uy, uz, a.eps, c);
    } else {
        const auto fetch = [&](int j) { return gload(pts + sp[j * WAVE]); };
        covariance_weighted(qx, qy, qz, cnt, fetch, a.wt, a.eps, c);
#pragma unroll 4
        for (int j = 0; j < cnt; ++j) irow[j] = __float_as_uint(gload(pts + sp[j * WAVE]).w);
        if (k == K)
            for (int j = cnt; j < k; ++j) irow[j] = ~0u;
    }
    store_cov(a.co, qi, c);
}

template <int K, int FUSED>
__device__ __forceinline__ void emit_cov(const GroupArgs& a, const TargetView& T, int64_t qi,
                                         float qx, float qy, float qz, int k, int cnt,
                                         const uint32_t* s_pos) {
    cov_gather<K, FUSED>(T.pts, s_pos + (K - k) * WAVE + lane_id(), (uint32_t*)a.ko.idx + qi * k, a, qi, qx,
                         qy, qz, k, cnt);
}

// An empty result row (non-finite query, empty target).
template <int FUSED>
__device__ __forceinline__ void emit_empty(const GroupArgs& a, int64_t qi, int k) {
#pragma unroll 1
    for (int j = 0; j < k; ++j) {
        a.ko.idx[qi * k + j] = -1;
        a.ko.d2[qi * k + j] = INF;
    }
    a.ko.count[qi] = 0;
    if (FUSED) {
        CovOut c;
        cov_empty(c);
        store_cov(a.co, qi, c);
    }
}

template <int K, int FUSED, bool PROF>
__device__ __forceinline__ void group_body(const GroupArgs& a, int64_t group, const SplitShare& sh,
                           uint32_t* s_tab, uint32_t* s_pos) {
    constexpr int KP = K + SLACK;
    const int lane = lane_id();
    const int64_t slot = group * WAVE + lane;
    const bool active = slot < a.n_slots;
    int gt = a.skeys ? (int)(load_uniform(a.skeys + group * WAVE) >> a.tshift) : 0;
    gt = __builtin_amdgcn_readfirstlane(gt);
    const TargetView T = load_uniform(a.views + gt);
    SlotQuery s{-1, 0.f, 0.f, 0.f, gt};
    if (active) s = load_slot(a, T, slot);
    const bool fin = active && finite3(s.x, s.y, s.z);
    const int cx = fin ? cell_coord(s.x, T.inv_cell) : 0;
    const int cy = fin ? cell_coord(s.y, T.inv_cell) : 0;
    const int cz = fin ? cell_coord(s.z, T.inv_cell) : 0;
    const bool same = fin && s.tgt == gt;
    const float r2 = a.sp.r2;
    const int k = a.sp.k;
    const int pad = K - k;
    // An empty target answers every query with an empty list.
    const bool empty_tgt = same && T.n_cells == 0;
    bool placed = empty_tgt;   // searched by one of the rounds below
    bool to_fb = false;        // handed to the wavefront-per-query search
    int row_cnt = -1;          // count of the row this wave wrote (-1: none)
    GroupProf<PROF> gp{};
    const unsigned long long t_start = PROF ? __builtin_amdgcn_s_memtime() : 0ull;
    // Rounds: each picks an anchor cell among the unplaced lanes and searches
    // for every unplaced lane within GROUP_W cells of it, so a group whose sorted
    // queries straddle two clusters can be served in two rounds rather than
    // handing one cluster to the wavefront-per-query search.  Every round
    // streams a whole block, so the launch sets the number of rounds.
    // Self queries: a window of k consecutive slots holding the lane's own
    // point are k target points, so the largest of their distances bounds
    // the lane's k-th distance from above (k = 1: its own point, distance
    // 0); every later test prunes against that bound.
    float lcap = INF;
    const int n_act = (int)min((int64_t)WAVE, a.n_slots - group * WAVE);
    const bool win = !a.queries && k <= 32 && n_act >= k;   // (uniform) the windows exist
    if (win) {
        // the lane's window: slots [w0, w0 + k) of the group
        const int w0 = min(max(lane - (k - 1) / 2, 0), n_act - k);
        float m = 0.0f;
#pragma unroll 1
        for (int j = 0; j < k; ++j) {
            const int src = w0 + j;
            m = fmaxf(m, dist2(s.x, s.y, s.z, shfl(s.x, src), shfl(s.y, src), shfl(s.z, src)));
        }
        lcap = m;
    }
    unsigned long long pending = T.n_cells > 0 ? ballot(same) : 0ull;
#pragma unroll 1
    for (int round = 0; round < a.rounds && pending; ++round) {
        // The anchor box is GROUP_W cells around the first pending lane's
        // cell.  A single-round launch (whose leftover lanes all fall back)
        // takes instead the box that holds the most pending lanes, of three:
        // around the first pending lane's cell, the last one's, and the
        // middle of the pending lanes' cells.
        const bool pend = (pending >> lane) & 1ull;
        auto takes = [&](int x, int y, int z) {
            return pend && abs(cx - x) <= GROUP_W && abs(cy - y) <= GROUP_W &&
                   abs(cz - z) <= GROUP_W;
        };
        const int L0 = __builtin_ffsll((long long)pending) - 1;
        const int L1 = 63 - __builtin_clzll(pending);
        int ax = readlane(cx, L0), ay = readlane(cy, L0), az = readlane(cz, L0);
        if (a.rounds == 1) {
            int best = __popcll(ballot(takes(ax, ay, az)));
            {
                const int bx = readlane(cx, L1), by = readlane(cy, L1), bz = readlane(cz, L1);
                const int c = __popcll(ballot(takes(bx, by, bz)));
                if (c > best) {
                    best = c;
                    ax = bx;
                    ay = by;
                    az = bz;
                }
            }
            {
                const auto middle = [&](int c) {
                    return (wave_min_i32(pend ? c : INT_MAX) + wave_max_i32(pend ? c : INT_MIN)) >> 1;
                };
                const int bx = middle(cx);
                const int by = middle(cy);
                const int bz = middle(cz);
                const int c = __popcll(ballot(takes(bx, by, bz)));
                if (c > best) {
                    ax = bx;
                    ay = by;
                    az = bz;
                }
            }
        }
        // A small target is streamed whole, in one round, for every lane.
        const bool whole = T.n <= WHOLE_N;
        const bool member = whole ? pend : takes(ax, ay, az);
        const unsigned long long mm = ballot(member);
        pending &= ~mm;
        placed = placed || member;
        const float bx0 = wave_min_ordered(member ? s.x : INF), bx1 = wave_max_ordered(member ? s.x : -INF);
        const float by0 = wave_min_ordered(member ? s.y : INF), by1 = wave_max_ordered(member ? s.y : -INF);
        const float bz0 = wave_min_ordered(member ? s.z : INF), bz1 = wave_max_ordered(member ? s.z : -INF);
        const float b0[3] = {bx0, by0, bz0}, b1[3] = {bx1, by1, bz1};
        int blo[3], bhi[3], lo[3], ext[3];
        int64_t total = 1;
        for (int d = 0; d < 3; ++d) {
            blo[d] = cell_coord(b0[d], T.inv_cell) - a.R;
            bhi[d] = cell_coord(b1[d], T.inv_cell) + a.R;
            lo[d] = max(blo[d], T.cmin[d]);
            const int hi = min(bhi[d], T.cmax[d]);
            ext[d] = hi - lo[d] + 1;
            total *= ext[d] > 0 ? ext[d] : 0;
        }
        const float qabs = fmaxf(fmaxf(fmaxf(fabsf(bx0), fabsf(bx1)), fmaxf(fabsf(by0), fabsf(by1))),
                                 fmaxf(fabsf(bz0), fabsf(bz1)));
        const float margin = (fmaxf(qabs, T.max_abs) + 2.0f * T.cell) * 1e-6f;
        // the lane's query widened by the margin (the runs' box tests)
        const float3 qlo = make_float3(s.x - margin, s.y - margin, s.z - margin);
        const float3 qhi = make_float3(s.x + margin, s.y + margin, s.z + margin);
        // this round's lists: K - k zero pads, then empty entries
        uint32_t L[KP];
#pragma unroll
        for (int j = 0; j < KP; ++j) L[j] = ~0u;
#pragma unroll 1
        for (int j = 0; j < pad; ++j) pk_insert<KP>(L, 0u);
        int n_ch = 1;
        const unsigned long long t_round = PROF ? __builtin_amdgcn_s_memtime() : 0ull;
        // Self queries: the group's 64 slots are 64 consecutive points of
        // the target's Morton order, i.e. the queries themselves and each
        // other's nearest points; streaming that chunk first fills every
        // list with near neighbours, so later candidates rarely pass.
        int own_cb = -1;
        if (!a.queries) {
            own_cb = (int)(group * WAVE);
            if (((own_cb / WAVE) & sh.split_mask) == sh.sub) {
                // the own chunk is this wave's chunk 1
                n_ch = 2;
                if (lane == 0) s_tab[1] = (uint32_t)(own_cb / WAVE);
                // The wave that streams the own chunk starts each member's
                // list with its window (the keys of its points within the
                // radius) and streams the rest of the chunk.
                int win_k = 0;
                if (win) {
                    const int w0 = min(max(lane - (k - 1) / 2, 0), n_act - k);
#pragma unroll 1
                    for (int j = 0; j < k; ++j) {
                        const int src = w0 + j;
                        const float px = shfl(s.x, src), py = shfl(s.y, src), pz = shfl(s.z, src);
                        const float d = dist2(s.x, s.y, s.z, px, py, pz);
                        // a window point beyond the radius is no neighbour
                        const uint32_t key = member && d <= r2
                                                 ? (__float_as_uint(d) & ~ID_MASK) | (1u << 6) |
                                                       (uint32_t)src
                                                 : ~0u;
                        pk_insert<KP>(L, key);
                    }
                    win_k = k;
                    gp.inserts += (uint32_t)__popcll(ballot(member)) * (uint32_t)k;
                }
                const uint32_t i0 = gp.inserts;
                scan_run<K>(T, own_cb, (int)min((int64_t)own_cb + WAVE, T.n), member, s.x, s.y,
                            s.z, r2, lcap, qlo, qhi, L, gp, -1, sh, n_ch, s_tab, 1,
                            win_k, n_act);
                gp.own += gp.inserts - i0;
            }
        }
        if (whole) {
            const uint32_t i0 = gp.inserts, c0 = gp.cands;
            scan_run<K>(T, 0, (int)T.n, member, s.x, s.y, s.z, r2, lcap, qlo, qhi,
                        L, gp, own_cb, sh, n_ch, s_tab);
            gp.ins2 += gp.inserts - i0;
            gp.cand2 += gp.cands - c0;
        }
        const float ie0 = 1.0f / (float)max(ext[0], 1), ie1 = 1.0f / (float)max(ext[1], 1);
        for (int pass = 0; pass < (whole ? 0 : 2); ++pass) {
            for (int64_t base = 0; base < total; base += WAVE) {
                gp.probes++;
                // the members' largest k-th bound (their lists only tighten
                // between probes)
                float own = pk_bound<K>(L, r2, lcap);
                if (sh.split_mask) own = shared_thr(sh, lane, own);
                const float gthr = wave_max_dpp(member ? own : -INF);
                const int64_t t = base + lane;
                bool want = false;
                uint32_t st = 0, cn = 0;
                if (t < total) {
                    // the block has at most (5 + 2 * 4)^3 cells: the quotients
                    // by float reciprocal ((a + 0.5) / b lies at least 0.5 / b
                    // from an integer; exact for a < 2^22)
                    const uint32_t tu = (uint32_t)t, e0 = (uint32_t)ext[0],
                                   e1 = (uint32_t)ext[1];
                    const uint32_t t0 = (uint32_t)(((float)tu + 0.5f) * ie0);
                    const uint32_t t1 = (uint32_t)(((float)t0 + 0.5f) * ie1);
                    const int c3[3] = {lo[0] + (int)(tu - t0 * e0), lo[1] + (int)(t0 - t1 * e1),
                                       lo[2] + (int)t1};
                    float bd = 0.0f;
                    for (int d = 0; d < 3; ++d) {
                        const float cl = (float)c3[d] * T.cell - margin;
                        const float ch = (float)(c3[d] + 1) * T.cell + margin;
                        const float g = fmaxf(fmaxf(cl - b1[d], b0[d] - ch), 0.0f);
                        bd += g * g;
                    }
                    const bool inside = bd == 0.0f;
                    if (inside == (pass == 0) && bd <= r2 && bd * (1.0f - 1e-6f) <= gthr)
                        want = hash_find(T, pack_key(T, c3[0], c3[1], c3[2]), st, cn) && cn > 0;
                }
                // the cells holding the queries first (they set tight k-th
                // distances), the surrounding cells after them
                unsigned long long wm = ballot(want);
                const uint32_t i0 = gp.inserts, c0 = gp.cands;
                while (wm) {
                    const int cl = __builtin_ffsll((long long)wm) - 1;
                    wm &= wm - 1;
                    const int s0 = readlane((int)st, cl);
                    const int e0 = s0 + readlane((int)cn, cl);
                    gp.cells++;
                    scan_run<K>(T, s0, e0, member, s.x, s.y, s.z, r2, lcap, qlo, qhi, L, gp,
                                own_cb, sh, n_ch, s_tab);
                }
                if (pass == 0) {
                    gp.ins0 += gp.inserts - i0;
                    gp.cand0 += gp.cands - c0;
                } else {
                    gp.ins1 += gp.inserts - i0;
                    gp.cand1 += gp.cands - c0;
                }
            }
        }
        const unsigned long long t_dec = PROF ? __builtin_amdgcn_s_memtime() : 0ull;
        // Decode every entry to its exact d2 bits (in place) and its
        // position in the reordered points (pads get position ~0u).  The
        // packed order is the exact order except inside a bucket, which
        // rarely holds more than two entries: four alternating odd-even
        // transposition phases fix up to four; a lane still out of order, or
        // whose order among equal distances the index would decide, or a
        // full list whose last entry shares the exact k-th distance's
        // bucket (a candidate it dropped may tie inside the bucket), or a
        // wave that ran out of chunk names, hands its lane on.
        const uint32_t last = L[KP - 1];
        uint32_t P[KP];
#pragma unroll
        for (int j = 0; j < KP; ++j) {
            const uint32_t e = L[j];
            uint32_t pos = e == 0u ? ~0u : 0u;
            if (member && e != 0u && e != ~0u) {
                const uint32_t id = e & ID_MASK;
                pos = s_tab[id >> 6] * (uint32_t)WAVE + (id & 63u);
                const float4 p = gload(T.pts + pos);
                L[j] = __float_as_uint(dist2(s.x, s.y, s.z, p.x, p.y, p.z));
            }
            P[j] = pos;
            if ((j % 12) == 11) __builtin_amdgcn_sched_barrier(0);   // bounded loads in flight
        }
        const auto cmpx_p = [&](int j) {
            const uint32_t d0 = L[j - 1], d1 = L[j], p0 = P[j - 1], p1 = P[j];
            const bool sw = d1 < d0;
            L[j - 1] = min(d0, d1);
            L[j] = max(d0, d1);
            P[j - 1] = sw ? p1 : p0;
            P[j] = sw ? p0 : p1;
        };
#pragma unroll
        for (int ph = 0; ph < 4; ++ph) {
#pragma unroll
            for (int j = 1 + (ph & 1); j < KP; j += 2) cmpx_p(j);
        }
        bool amb = false;
#pragma unroll
        for (int j = 1; j < KP; ++j) {
            // out of order, or two real entries at one distance up to the
            // (k+1)-th (pads and empty entries excepted)
            const bool real = P[j - 1] != ~0u && L[j] != ~0u;
            amb = amb || L[j] < L[j - 1] || (j <= K && real && L[j] == L[j - 1]);
        }
        const bool amb_b = last != ~0u && L[K - 1] != ~0u &&
                           (last >> ID_BITS) <= (L[K - 1] >> ID_BITS);
        if (PROF) {
            gp.amb_order += (uint32_t)__popcll(ballot(member && amb));
            gp.amb_bucket += (uint32_t)__popcll(ballot(member && !amb && amb_b));
            gp.amb_names += n_ch > MAX_CHUNKS ? (uint32_t)__popcll(ballot(member)) : 0u;
        }
        amb = member && (amb || n_ch > MAX_CHUNKS || amb_b);
        uint32_t D[K], Q[K];   // the first K: the row
#pragma unroll
        for (int j = 0; j < K; ++j) {
            D[j] = L[j];
            Q[j] = P[j];
        }
        if (sh.split_mask) {
            // every wave has streamed its chunks: merge the lists pairwise
            // through LDS (wave w + stride hands its lists to wave w, which
            // inserts the entries below its k-th distance; each list is
            // ascending, so a lane stops at its first miss, which must not
            // tie with the k-th); a lane is handed on if it is in any wave
#pragma unroll 1
            for (int stride = 1; stride <= sh.split_mask; stride <<= 1) {
                const int slot = sh.sub / (2 * stride);
                uint32_t* bd = sh.dist + (int64_t)slot * K * WAVE;
                uint32_t* bp = sh.pos + (int64_t)slot * K * WAVE;
                __syncthreads();
                if (sh.sub % (2 * stride) == stride) {
#pragma unroll
                    for (int j = 0; j < K; ++j) {
                        bd[j * WAVE + lane] = D[j];
                        bp[j * WAVE + lane] = Q[j];
                    }
                }
                __syncthreads();
                if (sh.sub % (2 * stride) == 0) {
#pragma unroll 1
                    for (int j = pad; j < K; ++j) {
                        const uint32_t x = bd[j * WAVE + lane];
                        const bool ins = member && x < D[K - 1];
                        amb = amb || (member && x != ~0u && x == D[K - 1]);
                        if (!ballot(ins)) break;
                        if (ins) insert_p<K>(D, Q, x, bp[j * WAVE + lane]);
                    }
                }
            }
            // equal distances brought together by the merge
#pragma unroll
            for (int j = 1; j < K; ++j)
                amb = amb || (member && Q[j - 1] != ~0u && D[j] != ~0u && D[j] == D[j - 1]);
            sh.flag[sh.sub * WAVE + lane] = amb ? 1u : 0u;
            __syncthreads();
            for (int w = 0; w <= sh.split_mask; ++w) amb = amb || sh.flag[w * WAVE + lane] != 0u;
            __syncthreads();   // the flags are rewritten next round
        }
        if (PROF) {
            const unsigned long long t_now = __builtin_amdgcn_s_memtime();
            gp.t_walk += (uint32_t)(t_dec - t_round);
            gp.t_final += (uint32_t)(t_now - t_dec);
        }
        if (member) {
            // exactness: every point outside the (unclamped) block is at least f away
            bool covers = true;
            float f = INF;
            const float q3[3] = {s.x, s.y, s.z};
            for (int d = 0; d < 3; ++d) {
                covers = covers && blo[d] <= T.cmin[d] && bhi[d] >= T.cmax[d];
                f = fminf(f, fminf(q3[d] - (float)blo[d] * T.cell,
                                   (float)(bhi[d] + 1) * T.cell - q3[d]));
            }
            f -= margin;
            const float f2 = f > 0.0f ? f * f * (1.0f - 1e-6f) : 0.0f;
            const bool full = D[K - 1] != ~0u;
            const bool ok = whole || covers || (full && f2 > __uint_as_float(D[K - 1])) ||
                            (a.sp.capped && f2 > r2);
            if (!ok || amb) {
                to_fb = true;
            } else if (sh.sub == 0) {
                row_cnt = emit_row<K, FUSED>(a, T, s.qi, k, D, Q, s_pos);
            }
        }
    }
    if (PROF && lane == 0) {
        // every wave of the group adds what it streamed (the buffer is
        // cleared before the launch)
        uint32_t* pw = a.prof + group * PROF_WORDS;
        const uint32_t add[15] = {gp.chunks,    gp.cands, gp.pops,  gp.inserts,    gp.dead,
                                  gp.ins0,      gp.ins1,  gp.ins2,  gp.cand0,      gp.cand1,
                                  gp.cand2,     gp.own,   gp.amb_order, gp.amb_bucket,
                                  gp.amb_names};
        const int at[15] = {3, 4, 5, 8, 9, 10, 11, 12, 13, 14, 15, 16, 17, 18, 19};
        for (int i = 0; i < 15; ++i) atomicAdd(pw + at[i], add[i]);
    }
    if (sh.sub) return;   // the other waves of a split group are done
    to_fb = to_fb || (fin && !placed);
    const unsigned long long fm = ballot(to_fb);
    if (PROF) {
        // (the ballot outside the lane-0 branch, so that it sees every lane)
        const unsigned long long pm = ballot(placed);
        if (lane == 0) {
            uint32_t* pw = a.prof + group * PROF_WORDS;
            pw[0] = (uint32_t)(__builtin_amdgcn_s_memtime() - t_start);
            pw[1] = gp.probes;
            pw[2] = gp.cells;
            pw[6] = (uint32_t)__popcll(pm);
            pw[7] = (uint32_t)__popcll(fm);
        }
    }
    if (fm) {
        const int leader = __builtin_ffsll((long long)fm) - 1;
        uint32_t base = 0;
        if (lane == leader) base = atomicAdd(a.fb_count, (uint32_t)__popcll(fm));
        base = (uint32_t)__shfl((int)base, leader);
        if (to_fb)
            a.fb_list[base + __popcll(fm & ((1ull << lane) - 1ull))] = (uint32_t)slot;
    }
    // covariances of the written rows (after the rounds: the lists are dead)
    const unsigned long long t_cov0 = PROF ? __builtin_amdgcn_s_memtime() : 0ull;
    if (FUSED && row_cnt >= 0) emit_cov<K, FUSED>(a, T, s.qi, s.x, s.y, s.z, k, row_cnt, s_pos);
    if (PROF && lane == 0 && sh.sub == 0) {
        uint32_t* pw = a.prof + group * PROF_WORDS;
        pw[20] = gp.t_walk;
        pw[21] = gp.t_final;
        pw[22] = (uint32_t)(__builtin_amdgcn_s_memtime() - t_cov0);
        pw[23] = gp.runs_grp;
        pw[24] = gp.runs_kept;
    }
    // non-finite queries and queries against an empty target: empty results
    if (active && (!fin || empty_tgt)) emit_empty<FUSED>(a, s.qi, k);
}
// PROF: record the per-group profile words (a.prof is set).
// Dynamic LDS of the group search (32-bit words): each wave's chunk names;
// the positions of the rows' neighbours (fused covariance; one wave emits
// in a split group); in a split group the merge buffers (d2 bits and
// positions), the shared k-th bounds and the lane flags.
__host__ __device__ inline size_t group_lds_words(int K, int fused, int split, int waves) {
    const size_t w = WAVE;
    size_t n = (size_t)waves * MAX_CHUNKS;
    if (fused) n += (size_t)(split > 1 ? 1 : waves) * K * w;
    if (split > 1) n += 2 * (size_t)(split / 2) * K * w + 2 * (size_t)split * w;
    return n;
}

template <int K, int FUSED, bool PROF>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(K <= 20 ? 4 : 2)))
k_group(GroupArgs a) {
    const int wpb = blockDim.x / WAVE;
    // (wavefront-uniform: scalar registers and branches for what follows)
    const int wid = __builtin_amdgcn_readfirstlane((int)(threadIdx.x / WAVE));
    const int64_t n_groups = (a.n_slots + WAVE - 1) / WAVE;
    extern __shared__ uint32_t s_dyn[];
    uint32_t* s_tab = s_dyn + wid * MAX_CHUNKS;
    uint32_t* s_free = s_dyn + wpb * MAX_CHUNKS;
    uint32_t* s_pos = nullptr;
    if (FUSED) {
        s_pos = s_free + (a.split > 1 ? 0 : wid) * K * WAVE;
        s_free += (a.split > 1 ? 1 : wpb) * K * WAVE;
    }
    // One call site, so that the body is inlined: its arguments then stay
    // in scalar registers (a called function takes them in vector registers
    // and reaches the kernel arguments through a stack copy).
    SplitShare sh{nullptr, nullptr, nullptr, nullptr, 0, 0};
    int64_t g;
    if (a.split > 1) {
        // one group per workgroup of `split` waves
        uint32_t* s_md = s_free;
        uint32_t* s_mp = s_md + (a.split / 2) * K * WAVE;
        float* s_thr = (float*)(s_mp + (a.split / 2) * K * WAVE);
        uint32_t* s_flag = (uint32_t*)(s_thr + a.split * WAVE);
        s_thr[threadIdx.x] = a.sp.r2;
        __syncthreads();
        sh = SplitShare{s_thr, s_flag, s_md, s_mp, wid, a.split - 1};
        // Groups of separate queries: each XCD takes a contiguous range, so
        // its L2 holds that range's part of the target.  Self queries (the
        // target is one scan, a few MB): groups are dealt round-robin over
        // the XCDs, which spreads the dense regions' heavy groups.
        g = a.queries ? (int64_t)xcd_tile(blockIdx.x, gridDim.x) : (int64_t)blockIdx.x;
    } else {
        // many groups: dealt round-robin over the XCDs, so that every XCD
        // gets a share of the dense regions
        g = (int64_t)blockIdx.x * wpb + wid;
    }
    // persistent: the groups are split into 8 contiguous ranges, one per XCD
    // (workgroups are dealt round-robin over the XCDs); a wave drains its own
    // XCD's range, then helps the others
    const bool persist = a.split <= 1 && a.counters != nullptr;
    const int lane = lane_id();
    const int x0 = blockIdx.x % 8;
    int xs = 0;
    for (;;) {
        if (persist) {
            g = -1;
            while (xs < 8) {
                const int x = (x0 + xs) % 8;
                const int64_t g_lo = n_groups * x / 8, g_hi = n_groups * (x + 1) / 8;
                uint32_t t = 0;
                if (lane == 0) t = atomicAdd(&a.counters[x], 1u);
                t = (uint32_t)__builtin_amdgcn_readfirstlane((int)t);
                if (g_lo + (int64_t)t < g_hi) {
                    g = g_lo + t;
                    break;
                }
                ++xs;
            }
            if (g < 0) break;
        }
        if (g < n_groups) group_body<K, FUSED, PROF>(a, g, sh, s_tab, s_pos);
        if (!persist) break;
    }
}

// A kept row's query (LDS).
struct WaveSlot {
    float x, y, z;
    int cnt;
    int32_t qi;
    union {
        int tg;       // target; once its points are gathered:
        float emin;   // smallest weight exponent
    };
};
static_assert(sizeof(WaveSlot) == 24, "WaveSlot layout");

// Words of a neighbour kept for its covariance: its index, then its offset
// from the query (and its weight).
__host__ __device__ constexpr int row_words(int fused) { return fused == 2 ? 4 : 3; }

// LDS of one wavefront: its plans, the candidate list, the slots, their rows.  With 5,300
// bytes of slots and rows six workgroups of four fit a CU's 160 KB, of which
// they take multiples of 1,280 bytes (k = 20: 20 rows; with a few hundred bytes
// more it is five, and the 65k-point match took 152 us instead of 125).
constexpr int WAVE_SLOTS = 32, WAVE_ROW_BYTES = 5300;

// (the room of a longer list is taken from the rows)
__host__ __device__ inline int wave_list_bytes(int k) {
    return 8 * (k > WIDE_K ? WaveList<2 * WAVE>::CAP : WaveList<WAVE>::CAP);
}
__host__ __device__ inline int wave_slots(int k, int fused) {
    const int fit = (WAVE_ROW_BYTES + wave_list_bytes(1) - wave_list_bytes(k)) / (4 * k * row_words(fused) + (int)sizeof(WaveSlot));
    return fit < WAVE_SLOTS ? fit : WAVE_SLOTS;
}
__host__ __device__ inline size_t wave_lds_bytes(int k, int slots, int fused) {
    const size_t rows = fused ? (size_t)slots * (4 * k * row_words(fused) + sizeof(WaveSlot)) : 0;
    return WAVE_PLANS * sizeof(WavePlan) + (size_t)wave_list_bytes(k) + ((rows + 15) & ~(size_t)15);
}

// Gathers the points of a wavefront's kept rows; offsets and weights in place
// of the indices.
template <int FUSED>
__device__ __forceinline__ void wave_rows(const GroupArgs& a, int k, int ns, WaveSlot* slots,
                                          float* rows) {
    constexpr int RW = row_words(FUSED);
    const int lane = lane_id();
    wave_lds_fence();
    const float ik = 1.0f / (float)k;
#pragma unroll 1
    for (int t = lane; t < ns * k; t += WAVE) {
        // (t + 0.5) / k lies at least 0.5 / k from an integer
        const int sl = (int)(((float)t + 0.5f) * ik), j = t - sl * k;
        const WaveSlot q = slots[sl];
        if (j < q.cnt) {
            float* r = rows + t * RW;
            const float4 p = gload(a.views[q.tg].orig + __float_as_int(r[0]));
            r[0] = p.x - q.x;
            r[1] = p.y - q.y;
            r[2] = p.z - q.z;
            if (FUSED == 2) r[3] = weight_exponent(a.wt, dist2(q.x, q.y, q.z, p.x, p.y, p.z));
        }
    }
    wave_lds_fence();
    if (FUSED == 2) {
        if (lane < ns) {
            float emin = INF;
            for (int j = 0; j < slots[lane].cnt; ++j)
                emin = fminf(emin, rows[(lane * k + j) * RW + 3]);
            slots[lane].emin = emin;
        }
        wave_lds_fence();
#pragma unroll 1
        for (int t = lane; t < ns * k; t += WAVE) {
            const int sl = (int)(((float)t + 0.5f) * ik), j = t - sl * k;
            if (j < slots[sl].cnt) rows[t * RW + 3] = expf(slots[sl].emin - rows[t * RW + 3]);
        }
        wave_lds_fence();
    }
}

// The covariance of one kept row, by one lane.
template <int FUSED>
__device__ __forceinline__ void wave_cov(const GroupArgs& a, const WaveSlot& q, const float* r) {
    constexpr int RW = row_words(FUSED);
    CovOut c;
    covariance_offsets<FUSED == 2>(
        q.x, q.y, q.z, q.cnt,
        [&](int j) {
            return make_float4(r[j * RW], r[j * RW + 1], r[j * RW + 2],
                               FUSED == 2 ? r[j * RW + RW - 1] : 0.0f);
        },
        a.eps, c);
    store_cov(a.co, q.qi, c);
}

// Wavefront-per-query search of the slots in `a.fb_list` (those the group
// search handed over; their number is only known on the device), or of every
// slot when there is no list.  Persistent: the XCDs take chunks of consecutive
// slots in turn (1 / 256 to 1 / 128 of all), whose part of the target their L2
// then holds, and an XCD's wavefronts stride over its chunks.  So a stretch of
// slots that cost far more than others, as in a list that is in cell order,
// falls to all XCDs (with one contiguous eighth each, 130,000 queries without a
// radius, k = 20, of 16,000 map points took 4,218 us; so 1,519).
//
// The rows of up to a.cov_slots queries of a wavefront are kept in LDS; at the
// end (or when they are full) their points are gathered and their offsets and
// weights taken with every lane, and the sums and eigenvectors follow for all
// queries of the workgroup, one lane per query.  (When every wavefront took the
// sums of its own rows, exponents and weights included, 30,000 queries with
// Laplacian weights took 94 us; this took 68.)
//
// Bound by the chain of dependent loads of each query (hash slots, points)
// with few queries, by VALU issue with many (65,536 queries against a 2
// M-point map: 0.107 ms; 0.125 before the plans were shared).
// The list of 99,000 queries that the group search hands over in a batch of
// 3.76 M takes 54 us (the wavefront search before it: 154).
//
// LIST: the entries its lists keep, 64 or 128; 1: k = 1 without covariances, no
// list.  RUNS: knn_query_runs answers.
template <int FUSED, int LIST, bool RUNS>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(6))) k_wave(GroupArgs a) {
    alignas(16) extern __shared__ unsigned long long s_wave[];
    const int lane = lane_id();
    const int wid = __builtin_amdgcn_readfirstlane((int)(threadIdx.x / WAVE));
    const int k = a.sp.k;
    constexpr bool ONE = LIST == 1;
    using List = WaveList<ONE ? WAVE : LIST>;
    constexpr int RW = row_words(FUSED);
    __shared__ WavePlan s_one[ONE ? 4 * WAVE_PLANS : 1];
    const size_t per_wave = wave_lds_bytes(k, a.cov_slots, FUSED);
    const auto plans_of = [&](int w) { return (WavePlan*)((char*)s_wave + w * per_wave); };
    const auto list_of = [&](int w) { return (unsigned long long*)(plans_of(w) + WAVE_PLANS); };
    const auto slots_of = [&](int w) { return (WaveSlot*)(list_of(w) + List::CAP); };
    const auto rows_of = [&](int w) { return (float*)(slots_of(w) + a.cov_slots); };   // [slot][k][RW]
    WavePlan* plans = ONE ? s_one + wid * WAVE_PLANS : plans_of(wid);
    unsigned long long* buf = list_of(wid);
    WaveSlot* slots = slots_of(wid);
    float* rows = rows_of(wid);
    // (wavefront-uniform, as the compiler has to know: scalar registers and
    // branches for all that follows)
    const int64_t n = a.fb_list ? (int64_t)(uint32_t)__builtin_amdgcn_readfirstlane(
                                      (int)*(volatile uint32_t*)a.fb_count)
                                : a.n_slots;
    // this XCD's slots: of every 8 chunks of 2^sh one, and an eighth of the rest
    // (the grid is a multiple of 8)
    const int x = blockIdx.x % 8, sh = max(2, 56 - __builtin_clzll((unsigned long long)(n | 128)));
    const int64_t dealt = n >> (sh + 3) << sh, rest = n - 8 * dealt, first = 8 * dealt + rest * x / 8;
    const int64_t mine = dealt + rest * (x + 1) / 8 - rest * x / 8;
    const auto query_at = [&](int64_t p) {
        return p < dealt ? ((p >> sh) << (sh + 3)) + ((int64_t)x << sh) + (p & (((int64_t)1 << sh) - 1))
                         : first + p - dealt;
    };
    const int64_t step = (int64_t)(gridDim.x / 8) * (blockDim.x / WAVE);
    int64_t p = (int64_t)(blockIdx.x / 8) * (blockDim.x / WAVE) + wid;
    int ns = 0;   // kept rows
    const bool self = a.queries == nullptr;
    const float radius = sqrtf(a.sp.r2);
    int b = WAVE_PLANS;   // the current query's plan
#pragma unroll 1
    for (; p < mine; p += step) {
        if (++b >= WAVE_PLANS) {
            b = 0;
            wave_lds_fence();
            const int64_t lp = p + (int64_t)lane * step, li = query_at(lp);
            if (lane < WAVE_PLANS && lp < mine) {
                const int64_t slot = a.fb_list ? (int64_t)gload(a.fb_list + li) : li;
                const int tg = a.skeys ? (int)(a.skeys[slot] >> a.tshift) : 0;
                const TargetView& V = a.views[tg];
                SlotQuery s{-1, 0.f, 0.f, 0.f, tg};
                if (!self || slot < V.n) s = load_slot(a, V, slot);
                if (ONE && a.moved) rigid_apply(a.move, s.x, s.y, s.z);
                // (a self query of a target that a failed rebuild left empty)
                const bool none = s.qi < 0;
                if (none) s.qi = slot;
                WavePlan w = wave_plan(V, s.x, s.y, s.z, (int32_t)s.qi,
                                       self ? (int)(slot / WAVE) : tg, a.sp.capped, radius);
                if (none) w.rmax = -1;
                plans[lane] = w;
            }
            wave_lds_fence();
        }
        WavePlan s;
        {
            const int4* from = (const int4*)(plans + b);
            int w[12];
#pragma unroll
            for (int e = 0; e < 3; ++e) {
                const int4 v = from[e];
                w[4 * e] = __builtin_amdgcn_readfirstlane(v.x);
                w[4 * e + 1] = __builtin_amdgcn_readfirstlane(v.y);
                w[4 * e + 2] = __builtin_amdgcn_readfirstlane(v.z);
                w[4 * e + 3] = __builtin_amdgcn_readfirstlane(v.w);
            }
            static_assert(sizeof w == sizeof s, "WavePlan layout");
            __builtin_memcpy(&s, w, sizeof s);
        }
        const int tg = self ? 0 : s.tgc;
        const TargetView T = load_uniform(a.views + tg);
        const bool search = s.rmax >= 0;
        if (ONE) {
            WaveNearest L{a.sp.r2, INF, IDX_SENTINEL};
            if (search) {
                if (RUNS) knn_query_runs(T, s, self, L);
                else knn_query_wave(T, a.views + tg, s, self, L);
            }
            const float d = wave_min_nonneg(L.d);
            const int32_t best = wave_min_i32(L.d == d ? L.i : IDX_SENTINEL);
            if (lane == 0) {
                const bool have = best != IDX_SENTINEL;
                a.ko.idx[(int64_t)s.qi] = have ? best : -1;
                a.ko.d2[s.qi] = have ? d : INF;
                a.ko.count[s.qi] = have ? 1 : 0;
            }
            continue;
        }
        List L{buf, a.sp.r2, 0, k, false};
        if (search) {
            if (RUNS) knn_query_runs(T, s, self, L);
            else knn_query_wave(T, a.views + tg, s, self, L);
        }
        // each entry's place among the k smallest, by counting
        L.finish();
        wave_lds_fence();
        const unsigned long long my = lane < L.n ? buf[lane] : ~0ull;
        buf[lane] = my;
        wave_lds_fence();
        int rank = 0;
        for (int j = 0; j < L.n; j += 4) {
#pragma unroll
            for (int u = 0; u < 4; ++u) rank += buf[j + u] < my ? 1 : 0;
        }
        const int cnt = min(L.n, k);
        const bool in = lane < L.n && rank < k;
        int32_t* irow = a.ko.idx + (int64_t)s.qi * k;
        float* drow = a.ko.d2 + (int64_t)s.qi * k;
        if (in) {
            irow[rank] = (int32_t)(uint32_t)my;
            drow[rank] = __uint_as_float((uint32_t)(my >> 32));
        }
        if (lane >= cnt && lane < k) {
            irow[lane] = -1;
            drow[lane] = INF;
        }
        if (lane == 0) a.ko.count[s.qi] = cnt;
        if (FUSED) {
            if (in) rows[(ns * k + rank) * RW] = __uint_as_float((uint32_t)my);
            if (lane == 0)
                slots[ns] = WaveSlot{s.x, s.y, s.z, cnt, s.qi, {tg}};
            if (++ns == a.cov_slots && p + step < mine) {
                wave_rows<FUSED>(a, k, ns, slots, rows);
                if (lane < ns) wave_cov<FUSED>(a, slots[lane], rows + lane * k * RW);
                ns = 0;
                wave_lds_fence();
            }
        }
    }
    if (FUSED) {
        // the workgroup's rows together (every wavefront gets here)
        __shared__ int s_ns[4];
        wave_rows<FUSED>(a, k, ns, slots, rows);
        if (lane == 0) s_ns[wid] = ns;
        __syncthreads();
        int sl = (int)threadIdx.x, w = 0;
        while (w < 4 && sl >= s_ns[w]) sl -= s_ns[w++];
        if (w < 4) wave_cov<FUSED>(a, slots_of(w)[sl], rows_of(w) + sl * k * RW);
    }
}

// Sort keys of the queries: target index above the query's cell in the
// target's grid (clamped to one cell around the occupied box, packed
// x-fastest).  scans/n_scans map a query to its target (NULL: target 0).
struct QueryKeyArgs {
    const float* queries;
    int64_t q;
    const TargetView* views;
    const BatchScan* scans;
    const BatchHeader* hdr;
    int tshift;
    int sub_bits;
    int w[3];   // bits of each axis's clamped cell coordinate
    void* keys;                 // Key[q]
    uint32_t* vals;
    uint32_t* words;            // 16 work words to clear, or NULL
};

// The cell coordinates' bits interleaved from the lowest level up, x first,
// an axis dropping out once its w[a] bits are used: the Morton order of the
// cells in w[0] + w[1] + w[2] bits (a flat box needs no key bits for the
// levels only its long axes have).
// (The levels of three axes, of the two longer ones and of the longest alone
// are spread by masks; bit by bit the keys of 3.76 M queries took 36 us, so
// 27.7.  The widths are the same for all lanes.)
__device__ __forceinline__ unsigned long long morton_compact(const uint32_t (&v)[3],
                                                             const int (&w)[3]) {
    const int lo = min(w[0], min(w[1], w[2])), hi = max(w[0], max(w[1], w[2]));
    const int mid = w[0] + w[1] + w[2] - lo - hi;
    const uint32_t m = (1u << lo) - 1u;
    unsigned long long key =
        lo <= 10 ? (unsigned long long)(spread3_10(v[0] & m) | (spread3_10(v[1] & m) << 1) |
                                        (spread3_10(v[2] & m) << 2))
                 : morton3(v[0] & m, v[1] & m, v[2] & m);
    if (hi > lo) {
        // the two longer axes, in their order, and the longest
        const bool no0 = w[0] == lo, no1 = !no0 && w[1] == lo;
        const uint32_t a = no0 ? v[1] : v[0], b = no0 || no1 ? v[2] : v[1];
        const int wa = no0 ? w[1] : w[0];
        const uint32_t m2 = (1u << (mid - lo)) - 1u;
        if (mid > lo)
            key |= (spread2((a >> lo) & m2) | (spread2((b >> lo) & m2) << 1)) << (3 * lo);
        const uint32_t top = ((wa == hi ? a : b) >> mid) & ((1u << (hi - mid)) - 1u);
        key |= (unsigned long long)top << (2 * mid + lo);
    }
    return key;
}

template <typename Key>
__global__ void __launch_bounds__(256) k_query_keys(QueryKeyArgs a) {
    if (a.words && blockIdx.x == 0 && threadIdx.x < 16) a.words[threadIdx.x] = 0u;
    __shared__ int s_lo;
    const int64_t i0 = (int64_t)blockIdx.x * blockDim.x;
    const int64_t i = i0 + threadIdx.x;
    int tg = 0;
    if (a.scans) {
        // The last scan starting at or before the workgroup's first query,
        // found once; each thread then steps to its own (the scans are
        // consecutive ranges, so a workgroup spans few of them).
        if (threadIdx.x == 0) {
            int lo = 0, hi = a.hdr->n_scans - 1;
            while (lo < hi) {
                const int mid = (lo + hi + 1) >> 1;
                if (a.scans[mid].q_offset <= i0)
                    lo = mid;
                else
                    hi = mid - 1;
            }
            s_lo = lo;
        }
        __syncthreads();
        if (i < a.q) {
            const int ns = a.hdr->n_scans;
            int lo = s_lo;
            while (lo + 1 < ns && a.scans[lo + 1].q_offset <= i) ++lo;
            tg = a.scans[lo].target_index;
        }
    }
    if (i >= a.q) return;
    const TargetView& T = a.views[tg];
    const float x = a.queries[3 * i], y = a.queries[3 * i + 1], z = a.queries[3 * i + 2];
    unsigned long long key;
    if (finite3(x, y, z)) {
        uint32_t v[3];
        const float p3[3] = {x, y, z};
        for (int d = 0; d < 3; ++d) {
            const int c = cell_coord(p3[d], T.inv_cell);
            const int range = max(T.cmax[d] - T.cmin[d], 0) + 2;
            v[d] = (uint32_t)min(max(c - (T.cmin[d] - 1), 0), range);
        }
        const int sb = a.sub_bits;
        // (the sub-cell's levels below the cell's, of all three axes)
        const int w[3] = {a.w[0] + sb, a.w[1] + sb, a.w[2] + sb};
        v[0] = v[0] << sb | sub_cell(x, T.inv_cell, sb);
        v[1] = v[1] << sb | sub_cell(y, T.inv_cell, sb);
        v[2] = v[2] << sb | sub_cell(z, T.inv_cell, sb);
        key = morton_compact(v, w);
    } else {
        key = (1ull << a.tshift) - 1ull;
    }
    ((Key*)a.keys)[i] = (Key)(((unsigned long long)tg << a.tshift) | key);
    a.vals[i] = (uint32_t)i;
}

// LDS words of one query's neighbours in k_cov: an odd number, so that lanes
// reading theirs do not meet in a bank.
__host__ __device__ constexpr int cov_stride(int k, bool weighted) {
    return (k * (weighted ? 4 : 3)) | 1;
}

// Covariances of neighbour lists given by original index (the layout the
// search writes).  A workgroup takes `nq` queries (at most 64): every lane
// loads list entries and their points, four of each at a time, into LDS (with
// weights, then their exponents and weights); one wavefront follows with the
// sums and the eigenvectors, a lane per query.  Which of the four does it
// alternates, so that the workgroups of a CU use all its SIMDs.  Bound by the
// two dependent loads and by that one lane's chain; with a lane per query from
// the start (two gathers of every neighbour and index loads k words apart)
// 65,536 lists of 20 took 18.2 us, this 9.9.
template <bool WEIGHTED>
__global__ void __launch_bounds__(256) k_cov(TargetView T, const float* __restrict__ queries,
                                             const int32_t* __restrict__ idx,
                                             const int32_t* __restrict__ count, int64_t q, int k,
                                             int nq, float eps, CovWeight wt, CovPtrs co) {
    extern __shared__ float s_rows[];   // [query][neighbour][3 or 4], cov_stride apart
    __shared__ float4 s_o[64];          // the query, and its smallest exponent
    __shared__ int s_n[64];
    constexpr int RW = WEIGHTED ? 4 : 3;
    const int stride = cov_stride(k, WEIGHTED), tid = (int)threadIdx.x;
    const int64_t q0 = (int64_t)xcd_tile(blockIdx.x, gridDim.x) * nq;
    const int here = (int)min((int64_t)nq, q - q0), total = here * k;
    const float ik = 1.0f / (float)k;
    // (t + 0.5) / k lies at least 0.5 / k from an integer
    const auto slot_of = [&](int t) { return (int)(((float)t + 0.5f) * ik); };
    if (tid < here) {
        float4 o = make_float4(0.f, 0.f, 0.f, 0.f);
        if (queries) {
            o.x = queries[3 * (q0 + tid)];
            o.y = queries[3 * (q0 + tid) + 1];
            o.z = queries[3 * (q0 + tid) + 2];
        }
        s_o[tid] = o;
        s_n[tid] = min(max(count[q0 + tid], 0), k);
    }
    __syncthreads();
    const uint32_t* nb = (const uint32_t*)idx + q0 * k;
    const int last = (int)min(T.n, (int64_t)0x7fffffff) - 1;
    if (last < 0) {
        if (tid < here) s_n[tid] = 0;
    } else if (ballot(lane_id() < here && s_n[lane_id()] > 0)) {   // (not for empty lists alone)
        for (int t0 = tid; t0 < total; t0 += 4 * 256) {
            int v[4];
            float4 p[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) v[u] = (int)gload(nb + min(t0 + u * 256, total - 1));
#pragma unroll
            for (int u = 0; u < 4; ++u) p[u] = gload(T.orig + min(max(v[u], 0), last));
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int t = t0 + u * 256;
                if (t < total) {
                    const int sl = slot_of(t), j = t - sl * k;
                    float* r = s_rows + sl * stride + j * RW;
                    r[0] = p[u].x;
                    r[1] = p[u].y;
                    r[2] = p[u].z;
                    // (a list ends at its first entry that names no point)
                    if (v[u] < 0 || v[u] > last) atomicMin(&s_n[sl], j);
                }
            }
        }
    }
    __syncthreads();
    if (!queries) {
        if (tid < here && s_n[tid] > 0) {
            const float* r = s_rows + tid * stride;
            s_o[tid] = make_float4(r[0], r[1], r[2], 0.f);
        }
        __syncthreads();
    }
    if (WEIGHTED) {
        for (int t = tid; t < total; t += 256) {
            const int sl = slot_of(t), j = t - sl * k;
            const float4 o = s_o[sl];
            float* r = s_rows + sl * stride + j * RW;
            if (j < s_n[sl])
                r[RW - 1] = weight_exponent(wt, dist2(o.x, o.y, o.z, r[0], r[1], r[2]));
        }
        __syncthreads();
        if (tid < here) {
            float emin = INF;
            for (int j = 0; j < s_n[tid]; ++j)
                emin = fminf(emin, s_rows[tid * stride + j * RW + RW - 1]);
            s_o[tid].w = emin;
        }
        __syncthreads();
        for (int t = tid; t < total; t += 256) {
            const int sl = slot_of(t), j = t - sl * k;
            float* r = s_rows + sl * stride + j * RW;
            if (j < s_n[sl]) r[RW - 1] = expf(s_o[sl].w - r[RW - 1]);
        }
        __syncthreads();
    }
    const int lane = lane_id();
    if (tid / WAVE != (int)((blockIdx.x / 256) & 3) || lane >= here) return;
    const float4 o = s_o[lane];
    const float* r = s_rows + lane * stride;
    CovOut c;
    covariance_offsets<WEIGHTED>(
        o.x, o.y, o.z, s_n[lane],
        [&](int j) {
            const float* e = r + j * RW;
            return make_float4(e[0] - o.x, e[1] - o.y, e[2] - o.z, WEIGHTED ? e[RW - 1] : 0.f);
        },
        eps, c);
    store_cov(co, q0 + lane, c);
}

SearchParams make_params(int k, float radius) {
    SearchParams sp;
    sp.k = k;
    sp.capped = std::isinf(radius) ? 0 : 1;
    sp.r2 = sp.capped ? radius * radius : INF;
    return sp;
}

}  // namespace


namespace {

__global__ void k_set_words(uint32_t* __restrict__ w, int n, uint32_t first) {
    const int i = threadIdx.x;
    if (i < n) w[i] = (i == 0) ? first : 0u;
}

inline size_t align256(size_t b) { return (b + 255) & ~size_t(255); }

int bitw(uint32_t v) { return v ? 32 - __builtin_clz(v) : 0; }

struct Scratch {
    unsigned long long *ka, *kb;
    uint32_t *va, *vb, *counts, *words, *fb_list;
};

// Offsets of the search scratch of n queries: sort keys and values (two
// buffers each), radix counts, work words, fallback list.
struct ScratchLayout {
    size_t ka, kb, va, vb, counts, words, fb, bytes;
};

ScratchLayout scratch_layout(int64_t n) {
    const size_t nn = (size_t)(n > 0 ? n : 1);
    ScratchLayout L{};
    size_t off = 0;
    auto carve = [&](size_t b) {
        const size_t o = off;
        off += align256(b);
        return o;
    };
    L.ka = carve(8 * nn);
    L.kb = carve(8 * nn);
    L.va = carve(4 * nn);
    L.vb = carve(4 * nn);
    L.counts = carve(4 * sort_count_words(n));
    L.words = carve(256);
    L.fb = carve(4 * nn);
    L.bytes = off;
    return L;
}

void carve_scratch(char* b, const ScratchLayout& L, Scratch& s) {
    s.ka = (unsigned long long*)(b + L.ka);
    s.kb = (unsigned long long*)(b + L.kb);
    s.va = (uint32_t*)(b + L.va);
    s.vb = (uint32_t*)(b + L.vb);
    s.counts = (uint32_t*)(b + L.counts);
    s.words = (uint32_t*)(b + L.words);
    s.fb_list = (uint32_t*)(b + L.fb);
}

lkc_status search_scratch(lkc_ctx* ctx, int64_t n, Scratch& s) {
    const ScratchLayout L = scratch_layout(n);
    if (ctx->search_scratch_bytes < L.bytes) {
        if (ctx->search_scratch) {
            LKC_HIP_TRY(ctx, hipStreamSynchronize(ctx->stream));
            (void)hipFree(ctx->search_scratch);
            ctx->search_scratch = nullptr;
            ctx->search_scratch_bytes = 0;
            ctx->last_fallback_count = nullptr;
        }
        const size_t bytes = L.bytes + L.bytes / 4;   // headroom for slightly larger calls
        hipError_t e = hipMalloc(&ctx->search_scratch, bytes);
        if (e != hipSuccess) {
            ctx->search_scratch = nullptr;
            return set_error(ctx, LKC_ERR_OOM, "search scratch of %zu bytes: %s", bytes,
                             hipGetErrorString(e));
        }
        ctx->search_scratch_bytes = bytes;
    }
    carve_scratch((char*)ctx->search_scratch, L, s);
    return LKC_OK;
}

// The allocation-free search (lkc_knn_cov_noalloc) keeps its scratch -- the
// sort keys and values, radix counts, work words and fallback list of up to
// NOALLOC_MAX_QUERIES queries -- in this file-scope device array.  Each
// device holds its own copy until the process ends; host code reaches it
// only through the address hipGetSymbolAddress returns for that device
// (the array's name is no device address on the host).
constexpr int64_t NOALLOC_MAX_QUERIES = 131072;
constexpr size_t NOALLOC_BYTES = size_t(4) << 20;
__device__ __align__(256) unsigned char scratch[NOALLOC_BYTES];

constexpr int NOALLOC_MAX_DEVICES = 64;
std::mutex g_noalloc_mu;
void* g_noalloc_ptr[NOALLOC_MAX_DEVICES] = {};

int choose_k_tile(int k) {
    if (k <= 8) return 8;
    if (k <= 16) return 16;
    if (k <= 20) return 20;
    if (k <= 32) return 32;
    return 0;
}

template <int FUSED>
void launch_group(int K, dim3 grid, dim3 block, hipStream_t st, const GroupArgs& a) {
    const size_t lds = sizeof(uint32_t) * group_lds_words(K, FUSED, a.split, (int)(block.x / WAVE));
    switch (K) {
        case 8:
            if (a.prof) hipLaunchKernelGGL((k_group<8, FUSED, true>), grid, block, lds, st, a);
            else hipLaunchKernelGGL((k_group<8, FUSED, false>), grid, block, lds, st, a);
            break;
        case 16:
            if (a.prof) hipLaunchKernelGGL((k_group<16, FUSED, true>), grid, block, lds, st, a);
            else hipLaunchKernelGGL((k_group<16, FUSED, false>), grid, block, lds, st, a);
            break;
        case 20:
            if (a.prof) hipLaunchKernelGGL((k_group<20, FUSED, true>), grid, block, lds, st, a);
            else hipLaunchKernelGGL((k_group<20, FUSED, false>), grid, block, lds, st, a);
            break;
        default:
            if (a.prof) hipLaunchKernelGGL((k_group<32, FUSED, true>), grid, block, lds, st, a);
            else hipLaunchKernelGGL((k_group<32, FUSED, false>), grid, block, lds, st, a);
            break;
    }
}

struct SearchJob {
    const TargetView* views_dev;
    const TargetView* host_views;
    int n_targets;
    const float* queries;   // NULL: self queries over target 0's points
    int64_t n_slots;
    const BatchScan* scans_dev;
    const BatchHeader* hdr_dev;
    int32_t k;
    float radius;
    float eps;
    int fused;      // 0 search only, 1 plain covariance, 2 weighted covariance
    KnnPtrs ko;
    CovPtrs co;
    CovWeight wt;
    const RigidF* move;   // k = 1 without covariances, wavefront search: moves the queries
};

// The layout of the queries' sort keys against n targets.
struct QueryKeyBits {
    int w[3];       // bits of each axis's clamped cell coordinate
    int sub_bits;   // Morton bits per axis of the sub-cell
    int tshift;     // bits below the target index
    int tbits;      // bits of the target index
};

// LKC_ERR_UNSUPPORTED where the keys have too few bits for the targets' boxes:
// of a search that may sort its queries, for every number of them, so that it
// does not depend on that number whether a target can be searched.
lkc_status query_key_bits(lkc_ctx* ctx, const TargetView* views, int n, QueryKeyBits& kb) {
    kb.w[0] = kb.w[1] = kb.w[2] = 1;
    for (int t = 0; t < n; ++t) {
        const TargetView& V = views[t];
        for (int d = 0; d < 3; ++d)
            kb.w[d] = std::max(kb.w[d], bitw((uint32_t)(std::max(V.cmax[d] - V.cmin[d], 0) + 2)));
    }
    const int wsum = kb.w[0] + kb.w[1] + kb.w[2];
    // Morton key of the (clamped) query cell, then of its sub-cell (as
    // many sub-cell bits, from 2 to 4 per axis, as the fewest 8-bit sort
    // passes holding the key with 2 of them allow)
    kb.tbits = n > 1 ? bitw((uint32_t)(n - 1)) : 0;
    const int sub_lo = std::max(0, std::min(2, (63 - kb.tbits - wsum) / 3));
    const int room = std::min(63, 8 * ((kb.tbits + wsum + 3 * sub_lo + 7) / 8)) - kb.tbits;
    kb.sub_bits = std::max(sub_lo, std::min(4, (room - wsum) / 3));
    kb.tshift = wsum + 3 * kb.sub_bits;
    if (kb.tshift + kb.tbits > 63)
        return set_error(ctx, LKC_ERR_UNSUPPORTED, "query sort key needs %d bits",
                         kb.tshift + kb.tbits);
    return LKC_OK;
}

// Whether the group search takes a launch of n queries.  The group search
// needs the fewest instructions a query (some 125 VALU against 660, k = 20 on a
// map) but sorts the queries first and lasts as long as its slowest group; the
// wavefront search is one launch whose work is even.  Measured,
// group / wavefront, us of the whole call, r = 2 m, 1 m cells:
//   queries against a map of 2 M points (5.3 a cell)      k = 20    k = 5     k = 32
//                                       20,000       153 / 38  113 / 32  192 / 42
//                                       65,536       196 / 106 147 / 81  347 / 115
//                                       98,304       233 / 154 170 / 118 329 / 178
//                                      131,072       252 / 202 182 / 154 367 / 223
//                                      196,608       293 / 294 230 / 225 402 / 331
//   against one of 100 k (2.2 a cell)
//                                       65,536       170 / 125 127 / 78  273 / 148
//                                       98,304       181 / 184 137 / 115 258 / 226
//                                      131,072       196 / 244 149 / 151 300 / 290
//                                      163,840       213 / 296 174 / 185 276 / 363
//     (0.8 m cells, 1.8 a cell, 98,304: 199 / 240, k = 10 173 / 175)
//   a sweep against itself              60,000       191 / 106 114 / 85  352 / 122
//                                      117,965       340 / 218 194 / 182 438 / 262
//   two sweeps against themselves      131,072       334 / 271 227 / 185 545 / 318
//                                      163,840       404 / 312 285 / 241 557 / 380
//   a sweep against itself, k = 1       65,536        59 / 68
// So the line lies at 384 queries per CU (98,304), 320 against targets of fewer
// than 1.8 points a cell; at 512 for self queries (sorted already, but of uneven
// density), 128 for their k = 1 (the own chunk answers it); above k = 20, where a
// group's lists leave room for two wavefronts a SIMD only, at 768, and 512
// against targets of fewer than 2.5 points a cell.  Against dense targets it is
// on the safe side.  (A volume of 30 points a cell against itself, 131,072, k =
// 5: 179 / 190.)
bool may_group(int K, int algorithm) { return K > 0 && algorithm != 2; }

bool takes_group(const lkc_ctx* ctx, int k, int algorithm, bool self, int64_t n,
                 const TargetView* views, int n_targets) {
    const int K = choose_k_tile(k);
    if (!may_group(K, algorithm)) return false;
    if (algorithm == 1) return true;
    int64_t points = 0, cells = 0;
    for (int t = 0; t < n_targets; ++t) {
        points += views[t].n;
        cells += views[t].n_cells;
    }
    const int per_cu = self     ? (K > 20 ? 768 : k == 1 ? 128 : 512)
                       : K > 20 ? (2 * points < 5 * cells ? 512 : 768)
                                : (10 * points < 18 * cells ? 320 : 384);
    return n > (int64_t)ctx->num_cus * per_cu;
}

// Whether a query's rings of cells may be many.
bool many_rings(const TargetView& V, float radius) { return !(radius <= 2.0f * V.cell); }

// Whether the wavefront search takes a target as a whole (knn_query_runs):
// small ones, and larger ones of which a box is mostly empty cells, where rings
// may be many.  40,000 queries without a radius, by rings and so, us:
//   10,000 points 10 m apart (800 cells of the box a point)  k = 5 2,499 / 91
//   10,000 of a map (21)     k = 1 37 / 69   k = 5 298 / 72   k = 20 1,115 / 80
//   16,000 of a sweep (11)   k = 1 93 / 109  k = 5 155 / 107  k = 20 673 / 106
//   16,000 of a cube (1)     k = 1 41 / 108  k = 5 65 / 113   k = 20 124 / 129
bool takes_runs(const TargetView& V, int k, float radius) {
    if (V.n <= RUNS_MAX_N) return true;
    if (V.n > RUNS_SPARSE_N || k < 4 || !many_rings(V, radius)) return false;
    double box = 1.0;   // (of a rebuild without a wait not known: 0)
    for (int d = 0; d < 3; ++d) box *= (double)V.cmax[d] - (double)V.cmin[d] + 1.0;
    return box >= 8.0 * (double)V.n;
}

// `fixed`: scratch the caller provides (then nothing is allocated and the
// per-group profile is off).
lkc_status run_search(lkc_ctx* ctx, const SearchJob& j, const LaunchCfg& cfg,
                      const Scratch* fixed = nullptr) {
    if (j.n_slots == 0) return LKC_OK;
    hipStream_t st = ctx->stream;
    const int K = choose_k_tile(j.k);
    bool few = false, many = false, rings = false;
    for (int t = 0; t < j.n_targets; ++t) {
        (takes_runs(j.host_views[t], j.k, j.radius) ? few : many) = true;
        rings = rings || many_rings(j.host_views[t], j.radius);
    }
    // (a batch over both kinds of target whose rings may be many: the group
    // search streams the small ones whole, the rings of a wavefront would not end)
    const bool group = takes_group(ctx, j.k, cfg.algorithm, j.queries == nullptr, j.n_slots,
                                   j.host_views, j.n_targets) ||
                       (few && many && rings && may_group(K, cfg.algorithm));
    const bool keyed = j.queries && (group || j.n_targets > 1);
    // (the wavefront search of one target needs no scratch)
    Scratch sc{};
    lkc_status s = LKC_OK;
    if (fixed)
        sc = *fixed;
    else if (group || keyed)
        s = search_scratch(ctx, j.n_slots, sc);
    if (s != LKC_OK) return s;
    GroupArgs a{};
    a.views = j.views_dev;
    a.queries = j.queries;
    a.order = nullptr;
    a.skeys = nullptr;
    a.tshift = 0;
    a.n_slots = j.n_slots;
    a.sp = make_params(j.k, j.radius);
    a.ko = j.ko;
    a.co = j.co;
    a.eps = j.eps;
    a.wt = j.wt;
    a.moved = j.move != nullptr;
    if (j.move) a.move = *j.move;
    // Self queries: a group of consecutive target points that straddles two
    // clusters is cheap to serve in a second round (measured: fewer
    // wavefront-per-query searches and a shorter search); past three rounds
    // the groups that take them set the launch's tail (on a 118k-point scan,
    // 4 rounds: 0.220 ms and 1,998 handed on; 3: 0.207 ms and 2,476; the
    // wavefront search's time hardly changes).  For external queries the
    // extra rounds cost more than the fallback they save.
    a.rounds = j.queries ? 1 : 3;
    a.fb_list = sc.fb_list;
    a.fb_count = sc.words;
    a.counters = nullptr;
    a.prof = (!fixed && ctx->prof_buf && (j.n_slots + WAVE - 1) / WAVE <= ctx->prof_groups)
                 ? (uint32_t*)ctx->prof_buf : nullptr;
    // (cleared before every search, also one that no group takes part in)
    if (a.prof)
        LKC_HIP_TRY(ctx, hipMemsetAsync(a.prof, 0,
                                        sizeof(uint32_t) * PROF_WORDS *
                                            (size_t)((j.n_slots + WAVE - 1) / WAVE),
                                        st));
    ctx->last_fallback_count = group ? sc.words : nullptr;
    ctx->last_all_wave = !group;
    ctx->last_queries = j.n_slots;
    ctx->ev_valid = ctx->timing;
    if (ctx->timing) LKC_HIP_TRY(ctx, hipEventRecord(ctx->ev[0], st));
    const unsigned wpb = (unsigned)cfg.waves_per_block;
    // Separate queries get keys: the group search sorts them by cell, and a
    // batch over several targets carries each query's target in the key's
    // top bits (the wavefront-per-query search reads it unsorted).
    QueryKeyBits kb{};
    if (j.queries && (keyed || may_group(K, cfg.algorithm))) {
        s = query_key_bits(ctx, j.host_views, j.n_targets, kb);
        if (s != LKC_OK) return s;
    }
    const int tshift = kb.tshift, tbits = kb.tbits;
    bool words32 = false;
    if (keyed) {
        // (one target: every scan's target is 0, no lookup)
        QueryKeyArgs qa{j.queries, j.n_slots, j.views_dev, j.n_targets > 1 ? j.scans_dev : nullptr,
                        j.hdr_dev, tshift,
                        kb.sub_bits, {kb.w[0], kb.w[1], kb.w[2]}, sc.ka, sc.va, group ? sc.words : nullptr};
        // (the sorted keys are read again only for the targets of several)
        words32 = group && j.n_targets == 1 && tshift <= 32;
        const dim3 kgrid((unsigned)((j.n_slots + 255) / 256));
        if (words32)
            hipLaunchKernelGGL(k_query_keys<uint32_t>, kgrid, dim3(256), 0, st, qa);
        else
            hipLaunchKernelGGL(k_query_keys<unsigned long long>, kgrid, dim3(256), 0, st, qa);
    }
    if (group) {
        if (!j.queries)
            hipLaunchKernelGGL(k_set_words, dim3(1), dim3(64), 0, st, sc.words, 16, 0u);
        if (j.queries) {
            // sort the queries by their key
            bool in_b = false;
            s = words32 ? sort_pairs(ctx, (uint32_t*)sc.ka, sc.va, (uint32_t*)sc.kb, sc.vb,
                                     j.n_slots, tshift, sc.counts, &in_b)
                        : sort_pairs(ctx, sc.ka, sc.va, sc.kb, sc.vb, j.n_slots, tshift + tbits,
                                     sc.counts, &in_b);
            if (s != LKC_OK) return s;
            a.order = in_b ? sc.vb : sc.va;
            a.skeys = j.n_targets > 1 ? (in_b ? sc.kb : sc.ka) : nullptr;
            a.tshift = tshift;
        }
        int R = cfg.group_reach;
        if (R <= 0) {
            R = 1;
            if (a.sp.capped)
                for (int t = 0; t < j.n_targets; ++t) {
                    const float c = j.host_views[t].cell;
                    const int rt = (int)std::ceil(std::sqrt(a.sp.r2) / c);
                    R = std::max(R, std::min(rt, 2));
                }
        }
        a.R = R;
        if (ctx->timing) LKC_HIP_TRY(ctx, hipEventRecord(ctx->ev[1], st));
        const int64_t n_groups = (j.n_slots + WAVE - 1) / WAVE;
        unsigned blocks, threads = wpb * WAVE;
        a.split = 1;
        if (cfg.persistent > 0) {
            a.counters = sc.words + 8;
            blocks = (unsigned)(ctx->num_cus * cfg.persistent);
        } else if (cfg.group_split > 1 ||
                   (cfg.group_split == 0 && 2 * n_groups <= 16 * (int64_t)ctx->num_cus)) {
            // few groups: the slowest one sets the kernel time, so several
            // waves share each group (as many as still fit at four waves per
            // SIMD)
            a.split = cfg.group_split > 1 ? cfg.group_split
                      : (4 * n_groups <= 16 * (int64_t)ctx->num_cus ? 4 : 2);
            blocks = (unsigned)n_groups;
            threads = (unsigned)(a.split * WAVE);
        } else {
            blocks = (unsigned)((n_groups + wpb - 1) / wpb);
        }
        if (j.fused == 2)
            launch_group<2>(K, dim3(blocks), dim3(threads), st, a);
        else if (j.fused == 1)
            launch_group<1>(K, dim3(blocks), dim3(threads), st, a);
        else
            launch_group<0>(K, dim3(blocks), dim3(threads), st, a);
    } else {
        // every query goes to the wavefront-per-query search
        a.fb_list = nullptr;
        if (j.queries && j.n_targets > 1) {
            // slots are the queries themselves: the unsorted keys give each
            // one's target
            a.skeys = sc.ka;
            a.tshift = tshift;
        }
        if (ctx->timing) LKC_HIP_TRY(ctx, hipEventRecord(ctx->ev[1], st));
    }
    if (ctx->timing) LKC_HIP_TRY(ctx, hipEventRecord(ctx->ev[2], st));
    // six 4-wave workgroups per CU fill the kernel's occupancy (a query's
    // search is a chain of dependent loads, so more resident waves shorten
    // the list each one works through); no more than the queries need
    const unsigned full = (unsigned)ctx->num_cus * 6;
    const int64_t need = group ? full : (j.n_slots + 3) / 4;
    const dim3 wgrid(((unsigned)std::min<int64_t>(full, need) + 7) & ~7u);
    a.cov_slots = wave_slots(j.k, j.fused);
    const size_t lds = 4 * wave_lds_bytes(j.k, a.cov_slots, j.fused);
    const bool runs = !many;
    const auto pick = [&](void (*cells)(GroupArgs), void (*all)(GroupArgs)) { return runs ? all : cells; };
    const bool wide = j.k > WIDE_K;
    void (*wave)(GroupArgs) =
        j.fused == 2   ? (wide ? pick(k_wave<2, 128, false>, k_wave<2, 128, true>)
                               : pick(k_wave<2, 64, false>, k_wave<2, 64, true>))
        : j.fused == 1 ? (wide ? pick(k_wave<1, 128, false>, k_wave<1, 128, true>)
                               : pick(k_wave<1, 64, false>, k_wave<1, 64, true>))
        : j.k == 1     ? pick(k_wave<0, 1, false>, k_wave<0, 1, true>)
        : wide         ? pick(k_wave<0, 128, false>, k_wave<0, 128, true>)
                       : pick(k_wave<0, 64, false>, k_wave<0, 64, true>);
    hipLaunchKernelGGL(wave, wgrid, dim3(256), j.fused == 0 && j.k == 1 ? 0 : lds, st, a);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return hip_error(ctx, e, "search launch");
    if (ctx->timing) LKC_HIP_TRY(ctx, hipEventRecord(ctx->ev[3], st));
    return LKC_OK;
}

lkc_status check_cfg(lkc_ctx* ctx, const LaunchCfg& c) {
    if (c.algorithm < 0 || c.algorithm > 2)
        return set_error(ctx, LKC_ERR_INVALID_ARG, "algorithm must be 0 (auto), 1 or 2");
    if (c.group_reach < 0 || c.group_reach > 4)
        return set_error(ctx, LKC_ERR_INVALID_ARG, "group_reach must be in [0, 4]");
    if (c.waves_per_block < 1 || c.waves_per_block > 4)   // kernels are built for <= 256 threads
        return set_error(ctx, LKC_ERR_INVALID_ARG, "waves_per_block must be in [1, 4]");
    if (c.merge_min < 1 || c.merge_min > 65)
        return set_error(ctx, LKC_ERR_INVALID_ARG, "merge_min must be in [1, 65]");
    if (c.persistent < 0 || c.persistent > 32)
        return set_error(ctx, LKC_ERR_INVALID_ARG, "persistent must be in [0, 32]");
    if (c.group_split < 0 || c.group_split > 4 || c.group_split == 3)
        return set_error(ctx, LKC_ERR_INVALID_ARG, "group_split must be 0, 1, 2 or 4");
    if (c.group_split > 1 && c.persistent > 0)
        return set_error(ctx, LKC_ERR_INVALID_ARG, "group_split > 1 needs persistent 0");
    return LKC_OK;
}

}  // namespace

lkc_status check_launch_cfg(lkc_ctx* ctx, const LaunchCfg& c) { return check_cfg(ctx, c); }

lkc_status reserve_search(lkc_ctx* ctx, int64_t max_queries) {
    Scratch sc;
    return search_scratch(ctx, max_queries, sc);
}

LaunchCfg resolve_cfg(const lkc_launch_cfg* c) {
    // two waves per workgroup by default: on large launches of 64-query
    // groups they measured a few per cent faster than four (a workgroup's
    // slots free up sooner) and than one
    LaunchCfg r{0, 0, 2, 12, 0, 0};
    if (c) {
        // (an option of the group search asks for it)
        const bool shaped = c->group_reach || c->waves_per_block || c->persistent || c->group_split;
        r.algorithm = c->algorithm == 0 && shaped ? 1 : c->algorithm;
        r.group_reach = c->group_reach;
        if (c->waves_per_block != 0) r.waves_per_block = c->waves_per_block;
        if (c->merge_min != 0) r.merge_min = c->merge_min;
        r.persistent = c->persistent;
        r.group_split = c->group_split;
    }
    return r;
}

bool knn_takes_group(const lkc_ctx* ctx, const lkc_target* t, int32_t k, int64_t q,
                     const LaunchCfg& cfg) {
    return takes_group(ctx, k, cfg.algorithm, false, q, &t->view, 1);
}

lkc_status check_query_keys(lkc_ctx* ctx, const lkc_target* t, int32_t k, const LaunchCfg& cfg) {
    QueryKeyBits kb;
    return may_group(choose_k_tile(k), cfg.algorithm) ? query_key_bits(ctx, &t->view, 1, kb) : LKC_OK;
}

lkc_status launch_knn(lkc_ctx* ctx, const lkc_target* t, const float* queries, int64_t q,
                      int32_t k, float radius, int32_t* idx, float* d2, int32_t* count,
                      const LaunchCfg& cfg, const RigidF* move) {
    lkc_status s = check_cfg(ctx, cfg);
    if (s != LKC_OK) return s;
    SearchJob j{t->view_dev, &t->view, 1, queries, q, nullptr, nullptr, k, radius, 0.0f, 0,
                KnnPtrs{idx, d2, count}, CovPtrs{nullptr, nullptr, nullptr, nullptr}};
    j.move = move;
    return run_search(ctx, j, cfg);
}

lkc_status launch_knn_cov(lkc_ctx* ctx, const lkc_target* t, const float* queries, int64_t q,
                          int32_t k, float radius, float eps, int32_t* idx, float* d2,
                          int32_t* count, float* mean, float* cov, float* reg, uint8_t* valid,
                          const LaunchCfg& cfg, const CovWeight& wt) {
    lkc_status s = check_cfg(ctx, cfg);
    if (s != LKC_OK) return s;
    const int mode = valid == nullptr ? 0 : wt.kind == LKC_WEIGHT_NONE ? 1 : 2;
    SearchJob j{t->view_dev, &t->view, 1, queries, q, nullptr, nullptr, k, radius, eps,
                mode, KnnPtrs{idx, d2, count}, CovPtrs{mean, cov, reg, valid}, wt};
    return run_search(ctx, j, cfg);
}

lkc_status noalloc_init(lkc_ctx* ctx) {
    const int dev = ctx->device;
    if (dev < 0 || dev >= NOALLOC_MAX_DEVICES)
        return set_error(ctx, LKC_ERR_UNSUPPORTED, "device %d beyond the %d the library serves",
                         dev, NOALLOC_MAX_DEVICES);
    if (scratch_layout(NOALLOC_MAX_QUERIES).bytes > NOALLOC_BYTES)
        return set_error(ctx, LKC_ERR_UNSUPPORTED, "allocation-free scratch layout too large");
    std::lock_guard<std::mutex> lock(g_noalloc_mu);
    if (g_noalloc_ptr[dev]) return LKC_OK;
    int cur = -1;
    LKC_HIP_TRY(ctx, hipGetDevice(&cur));
    if (cur != dev) LKC_HIP_TRY(ctx, hipSetDevice(dev));
    void* p = nullptr;
    const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (cur != dev) (void)hipSetDevice(cur);
    if (e != hipSuccess || !p) return hip_error(ctx, e, "hipGetSymbolAddress(scratch)");
    g_noalloc_ptr[dev] = p;
    return LKC_OK;
}

lkc_status launch_knn_cov_noalloc(lkc_ctx* ctx, const lkc_target* t, const float* queries,
                                  int64_t q, int32_t k, float radius, float eps, int32_t* idx,
                                  float* d2, int32_t* count, float* mean, float* cov,
                                  float* reg, uint8_t* valid, const LaunchCfg& cfg) {
    lkc_status s = check_cfg(ctx, cfg);
    if (s != LKC_OK) return s;
    if (q > NOALLOC_MAX_QUERIES)
        return set_error(ctx, LKC_ERR_BUDGET,
                         "lkc_knn_cov_noalloc takes at most %lld queries (got %lld)",
                         (long long)NOALLOC_MAX_QUERIES, (long long)q);
    if ((s = noalloc_init(ctx)) != LKC_OK) return s;   // set once per device
    void* base;
    {
        std::lock_guard<std::mutex> lock(g_noalloc_mu);
        base = g_noalloc_ptr[ctx->device];
    }
    Scratch sc;
    carve_scratch((char*)base, scratch_layout(q), sc);
    SearchJob j{t->view_dev, &t->view, 1, queries, q, nullptr, nullptr, k, radius, eps,
                valid != nullptr ? 1 : 0, KnnPtrs{idx, d2, count}, CovPtrs{mean, cov, reg, valid}};
    return run_search(ctx, j, cfg, &sc);
}

lkc_status launch_knn_self(lkc_ctx* ctx, const lkc_target* t, int32_t k, float radius,
                           float eps, int32_t* idx, float* d2, int32_t* count, float* mean,
                           float* cov, float* reg, uint8_t* valid, const LaunchCfg& cfg) {
    lkc_status s = check_cfg(ctx, cfg);
    if (s != LKC_OK) return s;
    SearchJob j{t->view_dev, &t->view, 1, nullptr, t->view.n, nullptr, nullptr, k, radius, eps,
                valid != nullptr ? 1 : 0, KnnPtrs{idx, d2, count}, CovPtrs{mean, cov, reg, valid}};
    return run_search(ctx, j, cfg);
}

constexpr int64_t COV_SLICE = 1 << 23;   // workgroups of one k_cov launch

lkc_status launch_cov(lkc_ctx* ctx, const lkc_target* t, const float* queries,
                      const int32_t* idx, const int32_t* count, int64_t q, int32_t k, float eps,
                      float* mean, float* cov, float* reg, uint8_t* valid, const CovWeight& wt) {
    if (q == 0) return LKC_OK;
    // 64 queries a workgroup, or as many as leave room for four workgroups' LDS
    // on a CU (long weighted lists)
    const bool weighted = wt.kind != LKC_WEIGHT_NONE;
    const int row = 4 * cov_stride(k, weighted);
    const int nq = 64 * row <= 36 * 1024 ? 64 : 32;
    static_assert(32 * 4 * cov_stride(LKC_MAX_K, true) <= 36 * 1024, "k_cov's LDS");
    if (q >= (int64_t)1 << 32) return set_error(ctx, LKC_ERR_INVALID_ARG, "too many queries");
    // (a launch has fewer than 2^32 threads)
    for (int64_t q0 = 0; q0 < q; q0 += COV_SLICE * nq) {
        const int64_t here = std::min(COV_SLICE * nq, q - q0);
        const dim3 grid((unsigned)((here + nq - 1) / nq));
        const CovPtrs co{mean ? mean + 3 * q0 : nullptr, cov ? cov + 9 * q0 : nullptr,
                         reg ? reg + 9 * q0 : nullptr, valid + q0};
        const float* qs = queries ? queries + 3 * q0 : nullptr;
        if (weighted)
            hipLaunchKernelGGL(k_cov<true>, grid, dim3(256), (size_t)nq * row, ctx->stream, t->view,
                               qs, idx + q0 * k, count + q0, here, k, nq, eps, wt, co);
        else
            hipLaunchKernelGGL(k_cov<false>, grid, dim3(256), (size_t)nq * row, ctx->stream, t->view,
                               qs, idx + q0 * k, count + q0, here, k, nq, eps, wt, co);
    }
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return hip_error(ctx, e, "covariance launch");
    return LKC_OK;
}

lkc_status launch_batched(lkc_ctx* ctx, lkc_target_set* set, const float* queries,
                          int64_t total_q, int32_t k, float radius, float eps, int32_t* idx,
                          float* d2, int32_t* count, float* mean, float* cov, float* reg,
                          uint8_t* valid, const LaunchCfg& cfg) {
    lkc_status s = check_cfg(ctx, cfg);
    if (s != LKC_OK) return s;
    if (set->staged_total != total_q)
        return set_error(ctx, LKC_ERR_INVALID_ARG,
                         "the staged scans cover %lld queries but total_q is %lld",
                         (long long)set->staged_total, (long long)total_q);
    if (set->staged_scans == 0) return LKC_OK;
    SearchJob j{set->views_dev, set->host_views, set->n_targets, queries, total_q,
                set->scans_dev, set->header_dev, k, radius, eps, 1,
                KnnPtrs{idx, d2, count}, CovPtrs{mean, cov, reg, valid}};
    return run_search(ctx, j, cfg);
}

}  // namespace lkc
