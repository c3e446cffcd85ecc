// Exact polyhedral geodesics by whole-mesh propagation, one source per wave64:
// all pairs (no cutoff), and cutoff passes with many targets (near passes).
//
// Every other particle of the surface is a target, so a source's windows
// must cover the whole mesh (the paper's full-mesh sequence trees, Sec. 3.1
// and Sec. 4; the Thomson-like long-range case). Without a cutoff two things
// keep the unfolding finite, both exact:
//  - vertex domination (the window filter of Xin and Wang's improvement of
//    the Chen-Han algorithm, the method the paper uses): each source keeps a
//    table D(v) of path lengths that have reached every vertex. A child window
//    on an edge S-E whose distance function f(x) = sg + |p - x| exceeds
//    D(S) + x (the path through S, then along the edge) is dominated there;
//    since f(x) - x is non-increasing the dominated part is [x0, x*) and is
//    trimmed (likewise (x**, x1] for the path through E). A window dominated
//    everywhere is dropped. Shortest paths to points beyond the edge are
//    never dominated this way, so no pair is lost.
//  - processing in rounds of increasing key: children whose key reaches the
//    round's threshold wait for the next round, so the search cannot run
//    ahead along one branch; once every target has been reached, windows
//    whose key exceeds the largest target distance (widened by the tie gap)
//    are dropped.
// A third filter, one angle, one split (one_split), halves the windows of
// surfaces with saddle or boundary vertices.
// Bend vertices are launched by the rules of the cutoff kernel, from a table
// that can hold every saddle and boundary vertex of the surface.
//
// Near passes take a cutoff instead: windows are dropped at it, a row holds the
// targets within it (gathered as they are reached, sorted by particle), and
// no table is cleared per source: vertex and half-edge entries carry the
// source's epoch, the states of the targets reached are reset one by one. A
// face's several targets are offered to all lanes' windows side by side
// (offer_pairs). On surfaces without bend vertices and cutoffs that stay on one
// side of them (kDom false), the domination tests, the rounds that order them
// and all that serves bend vertices are left out: there is next to nothing to
// dominate (the rule and its times stand where the pass is prepared). With hundreds of targets the cutoff kernel's per-target
// pruning keeps nearly every window; domination keeps 700 of its 2670 a
// source on the benchmark torus at 232 targets: 8192 sources 5.95 -> 1.34 ms
// a pass, at 58 targets 0.94 -> 0.47 ms.
//
// Mapping: the state of all n targets (best distance, best distance of
// another direction, tangent; 32 bytes each), the vertex table, the
// bend-vertex table and the window overflow in per-wavefront global areas
// (the overflow is two-ended: the current round grows from one end, the next
// round from the other); targets are found through the surface's
// particles-by-face index.
//
// What bounds it: the latency of one iteration of a wavefront (64 windows),
// at two wavefronts per SIMD: two dependent rounds of loads (about 1.3k and
// 1.5k cycles on the icosphere of 81,920 faces, mostly L2 misses) and about
// 5k cycles of arithmetic and stack work. The domination tests therefore run
// in squares (no square roots) and without branches, one body makes the
// children of both sides, the interval is cut while the second round's loads
// are on their way, a child takes its edge's vertex distances from its
// parent, and global stack traffic goes a wavefront's worth at a time.
// Together with records read in whole rounds: 2000 sources on that sphere
// 0.953 -> 0.652 s a pass (23 -> 33 G windows/s), 100 sources on an aspect-3
// torus of 3456 faces 18.7 -> 11.2 ms (and 18.8 -> 11.3 M windows). Fetching
// the next half-edge record straight into LDS an iteration ahead was slower
// (0.84 s, and 0.98 s with lanes sharing the loads): every later LDS access
// of the iteration waits for such a fetch.
#include <cmath>
#include <type_traits>

#include <hip/hip_ext.h>

#include "gsim_internal.h"
#include "window.h"

namespace gsim {
namespace {

using namespace wnd;

constexpr int kChunks = 8;
static_assert(kChunks == kWorkChunks, "one work counter per chunk");

// One target of a source: best distance, best distance of another direction,
// tangent of the best path. One 32-byte record, read as a whole.
struct alignas(16) TgtState {
    double d1 = INFINITY, d2 = INFINITY, tx = 0.0, ty = 0.0;
};

struct AllArgs {
    const SurfDesc *sd;
    BatchIdx bi;
    GeoParams gp;
    void *stack;     // per wavefront: stack_cap records of 64 bytes
    unsigned long long *vdist;  // per wavefront: vstride vertex distances
    int64_t vstride;
    char *roots;     // per wavefront: a bend-vertex table (rstride bytes, rcap vertices)
    int64_t rstride;
    int rcap;
    int32_t *work;
    Counters *ctr;
    unsigned long long *split;  // per wavefront: hstride half-edge entries (null: no surface has bend vertices)
    int64_t hstride;
    unsigned long long *best;  // teams: per team, tcap best distances
    TgtState *ttab;  // per wavefront: the state of tcap targets
    int64_t tstride; // bytes between two wavefronts' ttab (and, in near passes, touch, sort) areas
    int32_t *touch;  // near passes, per wavefront: the targets reached (tcap entries)
    unsigned long long *sort;  // near passes, per wavefront: kBigCandMax sort keys
    uint32_t *epoch; // near passes, per wavefront: the epoch of its last source
    uint32_t epoch_max;  // the first source's
    int tcap;
    int grab;
};

struct AllLds {
    BendLds B;
    int32_t unfound;  // targets not reached yet (near passes: targets reached)
    double maxb;      // windows with a larger key cannot improve any target
    unsigned long long starts;  // near passes: offer_pairs
    long long clk[6];           // per-source profile: start, loop, launches' time, iterations, results, launches before
    int32_t owner[kWave];
};

// Near passes: sort keys (particle, place in the by-face index) of a row;
// rows longer than kSortLds are sorted in global memory.
constexpr int kSortLds = 512;
struct SortLds {
    unsigned long long key[kSortLds];
};
struct NoSort {};

// A team's wavefronts (one source each workgroup): the source taken, what any
// of them met, and whether any has windows left for the next round (by the
// round's parity).
struct TeamLds {
    int32_t idx, overflow, more[2];
};
template <bool kNear>
struct SortOf {
    using T = typename std::conditional<kNear, SortLds, NoSort>::type;
};

// Per-source constants.
struct ACtx {
    double tol, tie_rel, tie_dir, root_keep, dom_rel, bucket;
    double cutoff;  // infinity for all pairs
    double split_rel;  // one_split: relative gap of the two distances
    RootCfg rc;
};

struct SrcStats {
    unsigned long long windows, launches, guards;
    int stale, pruned, depth;  // (stale and pruned: per lane)
    bool overflow;
};

// Window stack of the round-by-round order: LDS first, then one end of the
// wavefront's global area for the current round; the next round's windows
// grow from the other end, gathered in an LDS buffer and written out a
// wavefront's worth at a time (a store in flight would hold up the next
// iteration's wait for its loads).
template <typename R>
struct RoundStack {
    using Rec = typename RecOf<R>::T;
    int kL;
    Rec *lds;
    Rec *glb;
    int gcap;
    int lsp, gsp, dsp;
    int dir;
    Rec *ldd;  // kWave records waiting to go to the next round's end
    int dl;

    __device__ Rec &cur(int k) { return dir == 0 ? glb[k] : glb[gcap - 1 - k]; }
    __device__ Rec &def(int k) { return dir == 0 ? glb[gcap - 1 - k] : glb[k]; }

    __device__ void push(bool want, bool later, const Win<R> &w, bool &overflow) {
        const bool now = want && !later;
        uint64_t m = __ballot(now);
        int cnt = __popcll(m);
        if (cnt) {
            const int r = __popcll(m & lanemask_lt());
            const int space = kL - lsp;
            if (now) {
                if (r < space) {
                    store_rec(lds[lsp + r], w);
                } else {
                    const int pos = gsp + (r - space);
                    if (pos + dsp < gcap) store_rec(cur(pos), w);
                    else overflow = true;
                }
            }
            const int to_l = min(cnt, space);
            lsp += to_l;
            gsp = min(gsp + (cnt - to_l), gcap - dsp);
        }
        const bool lat = want && later;
        m = __ballot(lat);
        cnt = __popcll(m);
        if (cnt) {
            const int r = __popcll(m & lanemask_lt());
            if (dl + cnt > kWave) flush(overflow);
            if (lat) store_rec(ldd[dl + r], w);
            dl += cnt;
        }
    }
    // the buffered windows of the next round into its end of the global area
    __device__ void flush(bool &overflow) {
        wave_sync();
        const int l = lane_id();
        if (l < dl) {
            if (dsp + l + gsp < gcap) def(dsp + l) = ldd[l];
            else overflow = true;
        }
        dsp = min(dsp + dl, gcap - gsp);
        dl = 0;
        wave_sync();
    }
    // A wavefront's windows mostly arrive from the global area (a round's
    // windows wait there), a few lanes' worth an iteration. They are taken
    // over into the LDS stack a wavefront's worth at a time, so that one
    // iteration in many, not each, waits for that memory.
    __device__ bool refill(bool &have, Win<R> &w) {
        const uint64_t need = __ballot(!have);
        const int nneed = __popcll(need);
        if (lsp < nneed && gsp > 0) {
            wave_sync();  // make earlier global pushes of other lanes visible
            const int take = min(min(kL - lsp, kWave), gsp);
            if (lane_id() < take) lds[lsp + lane_id()] = cur(gsp - take + lane_id());
            lsp += take;
            gsp -= take;
            wave_sync();
        }
        const int r = __popcll(need & lanemask_lt());
        const int take_l = min(nneed, lsp);
        if (!have && r < take_l) {
            load_rec(lds[lsp - 1 - r], w);
            have = true;
        }
        lsp -= take_l;
        return __ballot(have) != 0;
    }
    // the next round's windows become the current ones (the current round is empty)
    __device__ void next_round(bool &overflow) {
        flush(overflow);
        dir ^= 1;
        gsp = dsp;
        dsp = 0;
    }
};

// Path lengths that have reached the vertices, updated by 64-bit minima. In
// whole-mesh passes the table holds doubles (positive doubles order like
// their bit patterns) and is cleared for every source. In near passes, whose
// sources reach a small part of the mesh, nothing is cleared: an entry is the
// source's epoch (20 bits, falling from source to source, so that a newer
// source's entries win every minimum), then the length as a float rounded up
// (a longer path through the vertex dominates less: exact, only the pruning
// is weaker by the rounding, 6e-8).
constexpr int kEpochShift = 44;
static_assert(kEpochMax < (1u << 20) - 1, "all ones marks an entry never written");
template <bool kNear>
struct VertexTable {
    unsigned long long *p;
    unsigned long long epoch;
    __device__ double operator[](int v) const {
        const unsigned long long x = p[v];
        if constexpr (!kNear) return __longlong_as_double((long long)x);
        return x >> kEpochShift == epoch ? (double)__uint_as_float((unsigned)(x >> 12)) : INFINITY;
    }
    __device__ void put(int v, double d) const {
        if constexpr (!kNear) atomicMin(p + v, (unsigned long long)__double_as_longlong(d));
        else atomicMin(p + v, epoch << kEpochShift | (unsigned long long)__float_as_uint(__double2float_ru(d)) << 12);
    }
    // is a path of squared length r (from the root image) plus sg worth a put?
    __device__ bool shorter(double r, double D, double sg) const;
};

// The state of a wavefront's targets by their place in the by-face index,
// and, in near passes, the list of the targets reached so far (their states
// are reset when the source is done).
template <bool kNear>
struct TargetTable {
    TgtState *st;
    int32_t *touch;
    unsigned long long *best;  // teams: every target's best distance over the team's wavefronts (else null)
    __device__ TgtState &operator[](int q) const { return st[q]; }
};

// Target update (j: the target's place in the by-face index): best distance,
// its tangent, and the best distance among candidates whose direction differs
// (tie gap); `alt` is the distance of an another-direction path that comes
// with the candidate. The lanes load their targets together (or hand in the
// entries `c` loaded earlier, with no other update in between) and leave when
// their candidate cannot change anything (the stored distances only
// decrease); the others are applied in registers, lanes with the same target
// one after another (in rounds).
template <bool kNear>
__device__ inline void target_update_loaded(AllLds &L, const TargetTable<kNear> &td, const ACtx &C, bool ok, int j, double d,
                                            double tx, double ty, double alt, const TgtState &c) {
    double c1 = INFINITY, c2 = INFINITY;
    if (ok) {
        c1 = c.d1;
        c2 = c.d2;
        if (d >= c1 && d >= c2 && alt >= c2) ok = false;
    }
    uint64_t m = __ballot(ok);
    if (!m) return;
    double ax = c.tx, ay = c.ty;
    int reached = 0;  // targets found for the first time
    for (bool todo = ok; m;) {
        const int wl = m & (m - 1) ? claim(L.B.win, todo, j) : lane_id();
        const bool mine = todo && wl == lane_id();
        int first = 0;
        if (mine) {
            const double c1_in = c1, c2_in = c2;
            const bool found = c1 < INFINITY;
            const bool differ = !found || fabs(ax * ty - ay * tx) > C.tie_dir || ax * tx + ay * ty < 0.0;
            if (d < c1) {
                if (differ) c2 = fmin(c2, c1);
                c1 = d;
                ax = tx;
                ay = ty;
                first = !found;
            } else if (differ) {
                c2 = fmin(c2, d);
            }
            c2 = fmin(c2, alt);
            if (c1 < c1_in || c2 < c2_in) td[j] = TgtState{c1, c2, ax, ay};
            if (!kNear && td.best && c1 < c1_in) atomicMin(td.best + j, (unsigned long long)__double_as_longlong(c1));
        }
        const uint64_t mfirst = __ballot(first);
        if (kNear && first) td.touch[L.unfound + reached + __popcll(mfirst & lanemask_lt())] = j;
        reached += __popcll(mfirst);
        todo = todo && !mine;
        m = __ballot(todo);
        if (m) {
            const double w1 = __shfl(c1, wl), w2 = __shfl(c2, wl), wx = __shfl(ax, wl), wy = __shfl(ay, wl);
            const int wj = __shfl(j, wl);
            if (todo && wj == j) {
                c1 = w1;
                c2 = w2;
                ax = wx;
                ay = wy;
            }
        }
    }
    if (lane_id() == 0 && reached) L.unfound += kNear ? reached : -reached;
    lane_step_barrier();
}

template <bool kNear>
__device__ inline void target_update(AllLds &L, const TargetTable<kNear> &td, const ACtx &C, bool ok, int j, double d, double tx,
                                     double ty, double alt) {
    TgtState c;
    if (ok) c = td[j];
    target_update_loaded(L, td, C, ok, j, d, tx, ty, alt, c);
}

// The domination tests below compare a window's distance f(x) = sg + |p - X|
// at a point X of the child edge with the length of a path through a vertex,
// in squares: with r = |p - X|^2, f(x) > d exactly when d < sg or
// r > (d - sg)^2. No square root is taken, and the rounding stays at that of
// the distances themselves, far inside the widening by rel.
__device__ inline bool longer(double r, double d_sg) { return d_sg < 0.0 || r > d_sg * d_sg; }

template <bool kNear>
__device__ inline bool VertexTable<kNear>::shorter(double r, double D, double sg) const {
    // the float entry exceeds the length it stands for: equal paths are not put again
    return !longer(r, (kNear ? D * (1.0 - 1.2e-7) : D) - sg);
}

// Trim a child interval [x0, x1] on an edge S -> E (length Lc, child frame
// origin S, root image (px, py)) against the paths through S and through E;
// returns false when nothing is left. The path through S and then along the
// edge has length DS + x; it is shorter than the window where
// g(x) = f(x) - x - DS > 0, and g is non-increasing, so the dominated part
// is [x0, x*). Likewise h(x) = f(x) - (Lc - x) - DE is non-decreasing and
// the part dominated by the path through E is (x**, x1]. The vertex path
// lengths are widened by the factor 1 + rel first, so only parts dominated
// beyond the rounding error of the working precision are cut. r0 and r1: the
// squared distances from p at the ends, updated with them.
__device__ inline bool vertex_trim(double px, double py, double sg, double Lc, double DS, double DE, double rel,
                                   double &x0, double &x1, double &r0, double &r1) {
    // the vertex paths count as shorter only by more than `rel` of their length
    const double dl = DS * (1.0 + rel) - sg;       // through S: dl + x
    const double mm = DE * (1.0 + rel) + Lc - sg;  // through E: mm - x
    const double eps_x = 1e-9 * Lc, h2 = py * py;
    // the far end of S's part, or the near end of E's, dominated: nothing is
    // left. Most windows pass all four tests, so they run without a branch
    // and the trims share one.
    const bool s0 = longer(r0, dl + x0), s1 = longer(r1, dl + x1);
    const bool e0 = longer(r0, mm - x0), e1 = longer(r1, mm - x1);
    bool left = x1 - x0 > 1e-12 * Lc && !s1 && !e0;
    if (left && (s0 || e1)) {
        if (s0) {
            // g(x*) = 0: sqrt((x - px)^2 + py^2) = dl + x
            const double den = 2.0 * (px + dl);
            const double xs = (px * px + h2 - dl * dl) / den;
            if (den > 0.0 && xs - eps_x > x0) {
                x0 = fmin(x1, xs - eps_x);
                r0 = (x0 - px) * (x0 - px) + h2;
                if (longer(r0, mm - x0)) left = false;
            }
        }
        if (e1) {
            // h(x**) = 0: sqrt((x - px)^2 + py^2) = mm - x
            const double den = 2.0 * (px - mm);
            const double xs = (px * px + h2 - mm * mm) / den;
            if (den < 0.0 && xs + eps_x < x1) {
                x1 = fmax(x0, xs + eps_x);
                r1 = (x1 - px) * (x1 - px) + h2;
            }
        }
        left = left && x1 - x0 > 1e-12 * Lc;
    }
    return left;
}

// Is the whole child interval [x0, x1] dominated by the path through the
// face's third vertex O (at (ox, oy) in the child frame, on the near side of
// the edge), i.e. DO + |O - X| < f(X)? The points of the edge line where that
// holds are the line's intersection with one branch region of a hyperbola
// with foci p and O, which is convex: domination at both ends means
// domination everywhere in between. With e = DO - sg, A = |O - X|^2 and
// r = |p - X|^2 the test e + sqrt(A) < sqrt(r) is squared twice.
__device__ inline bool opposite_dominates(double ox, double oy, double DO, double sg, double rel, double x0, double x1,
                                          double r0, double r1) {
    const double e = DO * (1.0 + rel) - sg, e2 = e * e;
    auto dom = [&](double x, double r) {
        const double A = (x - ox) * (x - ox) + oy * oy;
        // e >= 0: sqrt(r) > e + sqrt(A); e < 0: not sqrt(A) >= |e| + sqrt(r)
        const double P = e >= 0.0 ? A : r, Q = e >= 0.0 ? r : A;
        const double t = Q - P - e2, tt = t * t, pp = 4.0 * e2 * P;
        return e >= 0.0 ? t > 0.0 && tt > pp : !(t >= 0.0 && tt >= pp);
    };
    return dom(x0, r0) && dom(x1, r1);
}

// One angle, one split (Chen and Han, SoCG 1990): when another window of the
// same half-edge has reached the face's third vertex C by a shorter path, the
// rays of this window on that path's side of C are longer than it. Their
// paths cross the other's in the wedge between this window's ray to C and
// themselves (both windows leave the wedge's faces unfolded the same way), and
// are longer there: at most one child is left, the left one when the other
// ray crosses the half-edge to the right of this window's ray, else the right
// one. Hv keeps per half-edge the shortest such path and its crossing, packed
// with the source's epoch so that one 64-bit minimum updates both: 24 bits of
// the distance as a float rounded up, 20 bits of the crossing as a fraction
// of the edge. The distances must differ by rel beyond that rounding, far
// more than any tie band carried on to the targets; crossings closer than a
// thousandth of the edge decide nothing.
// Returns the sides still open: bit 0 the left child, bit 1 the right one.
__device__ inline int one_split(unsigned long long *Hv, unsigned long long epoch, int he, unsigned long long hw, double d,
                                double x, double len, double rel) {
    constexpr double kOne = (double)((1 << 20) - 1);
    const float hd = __uint_as_float((unsigned)((hw >> 20) & 0xffffff) << 7);
    const double hx = (double)(unsigned)(hw & 0xfffff) * (1.0 / kOne) * len;
    const bool other = hw >> kEpochShift == epoch && (double)hd * (1.0 + rel) < d;
    const int sides = other && hx > x + 1e-3 * len ? 1 : other && hx < x - 1e-3 * len ? 2 : 3;
    const unsigned db = (__float_as_uint(__double2float_ru(d)) + 127u) >> 7;
    const unsigned xb = (unsigned)(fmin(fmax(x / len, 0.0), 1.0) * kOne);
    const unsigned long long mine = epoch << kEpochShift | (unsigned long long)db << 20 | xb;
    if (mine < hw) atomicMin(Hv + he, mine);
    return sides;
}

// Where the rays through the ends of a window's interval leave through the
// far edge A -> C (left) or C -> B, in FP64 in both precisions; the side is
// selected per lane.
template <typename R>
__device__ inline void far_ends(const He<R> &h, const Win<R> &w, double txc, bool left, double &x0, double &x1) {
    const double px = w.px, py = w.py, b0 = w.b0, b1 = w.b1, cx = h.cx, cy = h.cy, L = h.L;
    const double Lc = left ? (double)h.Lp : (double)h.Ln;
    auto cut = [&](double b) {
        const double db = b - px;
        const double num = left ? py * b : (px - cx) * (-py) - (py - cy) * db;
        const double den = left ? py * cx + cy * db : (L - cx) * (-py) + cy * db;
        return Lc * num / den;
    };
    const double c0 = cut(b0), c1 = cut(b1);
    x0 = b0 <= (left ? 0.0 : txc) ? 0.0 : c0;
    x1 = b1 >= (left ? txc : L) ? Lc : c1;
    x0 = fmin(fmax(x0, 0.0), Lc);
    x1 = fmin(fmax(x1, 0.0), Lc);
}

// Offers every target of a lane's face: those of the by-face index from q on
// (-1: none). cand(t, d) tells whether the lane reaches target t and at what
// distance, dir(t, d, tx, ty, alt) its direction there and the distance of
// the other direction; t0 and c0 are the first target's record and state,
// loaded by the caller.
template <class Cand, class Dir>
__device__ inline void offer_targets(const FaceTarget *ftgt, AllLds &L, const TargetTable<false> &td, const ACtx &C, int q,
                                     int src, FaceTarget t0, TgtState c0, const Cand &cand, const Dir &dir) {
    while (__ballot(q >= 0)) {
        bool ok = false;
        double d = 0, tx = 0, ty = 0, alt = INFINITY;
        if (q >= 0 && t0.j != src) {
            ok = cand(t0, d);
            if (ok) dir(t0, d, tx, ty, alt);
        }
        target_update_loaded(L, td, C, ok, q, d, tx, ty, alt, c0);
        q = q >= 0 && t0.more ? q + 1 : -1;
        if (q >= 0) {
            t0 = ftgt[q];
            c0 = td[q];
        }
    }
}

// Near passes, whose faces hold several targets each: the (lane, target)
// pairs of all lanes side by side, 64 at a time, instead of each lane's
// targets one after another. A lane has cnt targets from place q0 on. cand
// is called by every lane with the pair's owner lane (whose values it fetches
// by shuffles), the target and whether there is a pair; it returns whether
// the owner reaches the target, with distance, direction and other-direction
// distance. On the benchmark torus with 1.8 targets a face, about six rounds
// an iteration become one.
template <class Cand>
__device__ inline void offer_pairs(const FaceTarget *ftgt, AllLds &L, const TargetTable<true> &td, const ACtx &C, int cnt,
                                   int q0, int src, const Cand &cand) {
    const int lane = lane_id();
    const uint64_t any = __ballot(cnt > 0);
    if (!any) return;
    // places of the pairs: a scan, which a count of lanes replaces where no
    // face has more than one target
    int inc = cnt;
    if (__ballot(cnt > 1)) {
        for (int o = 1; o < kWave; o <<= 1) {
            const int y = __shfl_up(inc, o);
            if (lane >= o) inc += y;
        }
    } else {
        inc = __popcll(any & (lanemask_lt() << 1 | 1));
    }
    const int excl = inc - cnt, total = __builtin_amdgcn_readlane(inc, kWave - 1);
    for (int base = 0; base < total; base += kWave) {
        // the lanes with pairs in this batch, in order, and a bit at the
        // place where each one's pairs begin
        const bool in = cnt > 0 && excl < base + kWave && inc > base;
        const uint64_t mi = __ballot(in);
        if (lane == 0) L.starts = 0;
        wave_sync();
        if (in) {
            L.owner[__popcll(mi & lanemask_lt())] = lane;
            atomicOr(&L.starts, 1ull << max(excl - base, 0));
        }
        wave_sync();
        const bool act = base + lane < total;
        const int own = L.owner[__popcll(L.starts & (lanemask_lt() << 1 | 1)) - 1];
        const int q = __shfl(q0, own) + (base + lane - __shfl(excl, own));
        FaceTarget t{{0.0, 0.0, 0.0}, -1, 0};
        TgtState c;
        if (act) {
            t = ftgt[q];
            c = td[q];
        }
        double d = 0, tx = 0, ty = 0, alt = INFINITY;
        bool ok = cand(own, t, d, tx, ty, alt);
        ok = ok && act && t.j != src && d < L.maxb;
        target_update_loaded(L, td, C, ok, q, d, tx, ty, alt, c);
    }
}

// Barycentrics of a target in the order of the half-edge in slot k of its
// face: that of its head and of the opposite vertex (selects: a lane's index
// into the record would put it in scratch).
__device__ inline double head_bary(const FaceTarget &t, int k) { return k == 0 ? t.b[1] : k == 1 ? t.b[2] : t.b[0]; }
__device__ inline double opp_bary(const FaceTarget &t, int k) { return k == 0 ? t.b[2] : k == 1 ? t.b[0] : t.b[1]; }

// Targets from q on in the face with entry half-edge slot k, seen through
// window w whose root has the tangent (rtx, rty) and other-direction distance
// rD2 (bend vertices).
template <typename R>
__device__ inline void query_face(const FaceTarget *ftgt, AllLds &L, const TargetTable<false> &td, const ACtx &C, int q,
                                  int src, int k, const He<R> &H, const Win<R> &w, double rtx, double rty, double rD2,
                                  const FaceTarget &t0, const TgtState &c0) {
    R dx = 0, dy = 0, l = 0;
    offer_targets(
        ftgt, L, td, C, q, src, t0, c0,
        [&](const FaceTarget &t, double &d) {
            const double bh = head_bary(t, k), bo = opp_bary(t, k);
            const R qx = (R)bh * H.L + (R)bo * H.cx;
            const R qy = (R)bo * H.cy;
            const R xq = w.px + (qx - w.px) * (-w.py) / (qy - w.py);
            const R sl = (R)C.tol * H.L;
            dx = qx - w.px;
            dy = qy - w.py;
            l = sqrt(dx * dx + dy * dy);
            d = (double)w.sg + (double)l;
            return xq >= w.b0 - sl && xq <= w.b1 + sl;
        },
        [&](const FaceTarget &, double, double &tx, double &ty, double &alt) {
            if (w.root < 0) {
                dx /= l;
                dy /= l;
                tx = (double)(w.c * dx - w.s * dy);
                ty = (double)(w.s * dx + w.c * dy);
            } else {
                tx = rtx;
                ty = rty;
                alt = rD2 + (double)l;
            }
        });
}

// The same in near passes, cnt targets from place q on.
template <bool kRoots, typename R>
__device__ inline void query_pairs(const FaceTarget *ftgt, AllLds &L, const TargetTable<true> &td, const ACtx &C, int cnt,
                                   int q, int src, int k, const He<R> &H, const Win<R> &w, double rtx, double rty,
                                   double rD2) {
    offer_pairs(ftgt, L, td, C, cnt, q, src,
                [&](int own, const FaceTarget &t, double &d, double &tx, double &ty, double &alt) {
                    const int ok_ = __shfl(k, own), root = kRoots ? __shfl(w.root, own) : -1;
                    const R hL = __shfl(H.L, own), hcx = __shfl(H.cx, own), hcy = __shfl(H.cy, own);
                    const R px = __shfl(w.px, own), py = __shfl(w.py, own);
                    const R b0 = __shfl(w.b0, own), b1 = __shfl(w.b1, own);
                    const double bh = head_bary(t, ok_), bo = opp_bary(t, ok_);
                    const R qx = (R)bh * hL + (R)bo * hcx, qy = (R)bo * hcy;
                    const R xq = px + (qx - px) * (-py) / (qy - py), sl = (R)C.tol * hL;
                    const R dx = qx - px, dy = qy - py, l = sqrt(dx * dx + dy * dy);
                    const R c = __shfl(w.c, own), s = __shfl(w.s, own);
                    double ux = 0.0, uy = 0.0, u2 = INFINITY;
                    if constexpr (kRoots) {
                        ux = __shfl(rtx, own);
                        uy = __shfl(rty, own);
                        u2 = __shfl(rD2, own);
                    }
                    d = (double)__shfl(w.sg, own) + (double)l;
                    const R ex = dx / l, ey = dy / l;
                    tx = root < 0 ? (double)(c * ex - s * ey) : ux;
                    ty = root < 0 ? (double)(s * ex + c * ey) : uy;
                    alt = root < 0 ? INFINITY : u2 + (double)l;
                    return xq >= b0 - sl && xq <= b1 + sl;
                });
}

// Launch the pending bend vertices (their distance improved, or their best
// direction changed, or a tie appeared), their fans flattened over the lanes
// a chunk of vertices at a time. Returns whether a window found no room (the
// caller ends the source).
template <typename R, bool kNear, int kTeam>
__device__ bool launch_roots(const SurfDesc &sd, AllLds &L, const BendTable &G, const TargetTable<kNear> &td,
                             const VertexTable<kNear> &Dv, const ACtx &C, RoundStack<R> &S, double T, int src,
                             SrcStats &st) {
    const int lane = lane_id();
    const DevMesh &M = sd.m;
    const HeRec *const he = uniform(M.he);
    const PseudoRec *const prec = uniform(M.prec);
    const int32_t *const fan = uniform(M.fan), *const pidx = uniform(M.pidx), *const ffirst = uniform(sd.ffirst),
                  *const fstart = uniform(sd.fstart);
    const FaceTarget *const ftgt = uniform(sd.ftgt);
    // take the pending list (its vertices may be queued again while they launch)
    const int npend = L.B.npend;
    const double maxb = L.maxb;
    bool lost = false;
    int nsel = 0;
    for (int base = 0; base < npend; base += kWave) {
        const int k = base + lane;
        int e = 0;
        bool sel = false;
        double D = 0.0;
        if (k < npend) {
            e = G.pend[k];
            D = G.rD[e];
            sel = D < G.rL[e] * C.rc.keep && D < maxb;
            // a wavefront of the team that reached the vertex by a shorter
            // path launches it (paths within the tie band both are)
            if (kTeam > 1) sel = sel && D <= Dv[prec[e].v] * (1.0 + 4.0 * C.tie_rel);
            G.queued[e] = 0;
        }
        const uint64_t mk = __ballot(sel);
        if (sel) {
            const int pos = nsel + __popcll(mk & lanemask_lt());
            G.sel[pos] = e;
            if (pos < kLaunchChunk) L.B.sel[pos] = e;  // the first chunk also through LDS
            G.rL[e] = D;
        }
        nsel += __popcll(mk);
    }
    if (lane == 0) L.B.npend = 0;
    wave_sync();
    for (int c0 = 0; c0 < nsel; c0 += kLaunchChunk) {
        const int cn = min(kLaunchChunk, nsel - c0);
        int carry = 0;
        for (int base = 0; base < cn; base += kWave) {
            const int k = base + lane;
            int deg = 0;
            if (k < cn) {
                if (c0 > 0) L.B.sel[k] = G.sel[c0 + k];
                deg = prec[L.B.sel[k]].fan_deg;
            }
            int inc = deg;
            for (int o = 1; o < kWave; o <<= 1) {
                const int y = __shfl_up(inc, o);
                if (lane >= o) inc += y;
            }
            if (k < cn) L.B.pref[k + 1] = carry + inc;
            st.launches += (unsigned long long)__popcll(__ballot(deg > 0));
            carry += __builtin_amdgcn_readlane(inc, kWave - 1);
        }
        if (lane == 0) L.B.pref[0] = 0;
        wave_sync();
        const int total = carry;
        for (int base = 0; base < total; base += kWave) {
            const int idx = base + lane;
            const bool act = idx < total;
            int k = 0;
            if (act) {
                int lo = 0, hi = cn - 1;
                while (lo < hi) {
                    const int mid = (lo + hi + 1) >> 1;
                    if (L.B.pref[mid] <= idx) lo = mid;
                    else hi = mid - 1;
                }
                k = lo;
            }
            const int el = act ? L.B.sel[k] : 0;
            const int fb = act ? prec[el].fan_beg : 0;
            const double D = act ? G.rD[el] : 0.0;
            const double vtx = act ? G.rtx[el] : 0.0, vty = act ? G.rty[el] : 0.0;
            const double D2 = act ? G.rD2[el] : INFINITY;
            const int h = act ? fan[fb + (idx - L.B.pref[k])] : 0;
            const int g = h / 3, hk = h - 3 * g;
            const int hn = 3 * g + (hk == 2 ? 0 : hk + 1);
            const HeRec Rh = he[h], Rn = he[hn];
            int q = -1, cnt = 0;
            if constexpr (kNear) {
                q = act ? fstart[g] : 0;
                cnt = act ? fstart[g + 1] - q : 0;
            } else {
                q = act ? ffirst[g] : -1;
            }
            // the two other vertices of face(h): reached along its edges
            const int u1 = Rh.head, u2 = Rh.opp_flags >> 1;
            FaceTarget t0{{0.0, 0.0, 0.0}, -1, 0};
            TgtState c0s;
            double D1 = INFINITY, D3 = INFINITY;
            int e1 = -1, e2 = -1;
            if (act) {
                if (!kNear && q >= 0) {
                    t0 = ftgt[q];
                    c0s = td[q];
                }
                D1 = Dv[u1];
                D3 = Dv[u2];
                e1 = pidx[u1];
                e2 = pidx[u2];
                if (D + Rh.L < D1) Dv.put(u1, D + Rh.L);
                if (D + Rh.Lp < D3) Dv.put(u2, D + Rh.Lp);
                D1 = fmin(D1, D + Rh.L);
                D3 = fmin(D3, D + Rh.Lp);
            }
            Win<R> nw;
            bool want = false, later = false;
            if (act && Rn.twin >= 0) {
                // window across the edge opposite v: twin(next(h)) runs u2 ->
                // u1; the parts that the paths along those vertices' edges
                // dominate are cut at once
                const double px = Rn.L - Rn.cx, py = -Rn.cy;
                double x0 = 0.0, x1 = Rn.L, r0 = px * px + py * py, r1 = (Rn.L - px) * (Rn.L - px) + py * py;
                if (vertex_trim(px, py, D, Rn.L, D3, D1, C.dom_rel, x0, x1, r0, r1)) {
                    nw.px = (R)px;
                    nw.py = (R)py;
                    nw.b0 = (R)x0;
                    nw.b1 = (R)x1;
                    nw.sg = (R)D;
                    nw.c = R(1);
                    nw.s = R(0);
                    nw.he = Rn.twin;
                    nw.root = el;
                    const double rk = px < x0 ? r0 : px > x1 ? r1 : py * py;
                    want = !longer(rk, maxb - D);
                    later = T <= D || rk >= (T - D) * (T - D);
                }
            }
            // direct targets in face(h): straight segments inside the face
            if constexpr (kNear)
                offer_pairs(ftgt, L, td, C, cnt, q, src,
                            [&](int own, const FaceTarget &t, double &d, double &tx, double &ty, double &alt) {
                                const int ko = __shfl(hk, own);
                                const double bh = head_bary(t, ko), bo = opp_bary(t, ko);
                                const double x = bh * __shfl(Rh.L, own) + bo * __shfl(Rh.cx, own);
                                const double y = bo * __shfl(Rh.cy, own), Do = __shfl(D, own);
                                d = Do + sqrt(x * x + y * y);
                                tx = __shfl(vtx, own);
                                ty = __shfl(vty, own);
                                alt = __shfl(D2, own) + (d - Do);
                                return true;
                            });
            else offer_targets(
                ftgt, L, td, C, q, src, t0, c0s,
                [&](const FaceTarget &t, double &d) {
                    const double bh = head_bary(t, hk), bo = opp_bary(t, hk);
                    const double x = bh * Rh.L + bo * Rh.cx, y = bo * Rh.cy;
                    d = D + sqrt(x * x + y * y);
                    return true;
                },
                [&](const FaceTarget &, double d, double &tx, double &ty, double &alt) {
                    tx = vtx;
                    ty = vty;
                    alt = D2 + (d - D);
                });
            bend_update(G, L.B, C.rc, e1 >= 0, e1, D + Rh.L, vtx, vty, D2 + Rh.L);
            bend_update(G, L.B, C.rc, e2 >= 0, e2, D + Rh.Lp, vtx, vty, D2 + Rh.Lp);
            S.push(want, later, nw, lost);
        }
        wave_sync();  // the chunk arrays are rewritten by the next chunk
    }
    return __ballot(lost) != 0;
}

// Windows with a larger key than the farthest target's distance (dist(q) of n
// targets; widened by the tie gap) cannot improve any.
template <class Dist>
__device__ inline void key_bound(AllLds &L, const ACtx &C, int n, const Dist &dist) {
    double mx = 0.0;
    for (int q = lane_id(); q < n; q += kWave) mx = fmax(mx, dist(q));
    for (int o = 32; o > 0; o >>= 1) mx = fmax(mx, __shfl_xor(mx, o));
    if (lane_id() == 0) L.maxb = fmin(L.maxb, mx * (1.0 + C.tie_rel) + 1e-12 * mx);
}

// An entry that other wavefronts of the team have updated by atomics, read
// where those act (not from this compute unit's vector cache).
__device__ inline unsigned long long team_load(const unsigned long long *p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// The smallest of the members' entries into all of them: tab, the first
// member's table of n entries, the others' stride entries apart.
template <int kTeam>
__device__ inline void team_merge(unsigned long long *tab, int64_t stride, int n) {
    for (int i = threadIdx.x; i < n; i += kWave * kTeam) {
        unsigned long long x[kTeam], m = ~0ull;
#pragma unroll
        for (int k = 0; k < kTeam; ++k) x[k] = team_load(tab + k * stride + i);
#pragma unroll
        for (int k = 0; k < kTeam; ++k) m = x[k] < m ? x[k] : m;
#pragma unroll
        for (int k = 0; k < kTeam; ++k)
            if (x[k] != m) tab[k * stride + i] = m;
    }
}

// One source's whole-mesh propagation and its row of results. With a
// finite cutoff, windows whose key reaches it are dropped (in FP32 a little
// beyond it, by the acceptance slack) and the row keeps every target; the
// pairs at or beyond the cutoff are left out downstream. Returns whether an
// FP32 result lies within the guard band around the cutoff (the caller then
// recomputes the source in FP64; `guard` marks that recompute). Inlined:
// as a call, the FP32 kernel spills around it and holds one wave per SIMD.
template <typename R, bool kNear, int kTeam, bool kDom>
__device__ __attribute__((always_inline)) inline bool run_all(const AllArgs &a, const SurfDesc &sd, AllLds &L,
                                                              const TargetTable<kNear> &td, unsigned char *stk,
                                                              int stk_bytes, unsigned char *later, SortLds *sl, TeamLds &team, int member, int src, bool guard,
                                                              uint32_t &epoch,
                                                              SrcStats &st) {
    const int lane = lane_id();
    const int slot = kTeam == 1 ? (int)blockIdx.x : (int)blockIdx.x * kTeam + member;
    const bool fp32 = sizeof(R) == 4;
    const int n = sd.n;
    // the mesh and the target index through local pointers: read from the
    // descriptor where they are used, each would be loaded again after every
    // store (and the loads that need it wait for that one)
    const DevMesh &M = sd.m;
    const HeRec *const he = uniform(M.he);
    const HeRecF *const hef = uniform(M.hef);
    const int32_t *const pidx = uniform(M.pidx), *const ffirst = uniform(sd.ffirst), *const fstart = uniform(sd.fstart);
    const FaceTarget *const ftgt = uniform(sd.ftgt);
    ACtx C;
    C.tol = fp32 ? a.gp.cone_tol32 : a.gp.cone_tol;
    C.tie_rel = fp32 ? a.gp.tie_rel32 : a.gp.tie_rel;
    C.tie_dir = fp32 ? a.gp.tie_dir32 : a.gp.tie_dir;
    C.root_keep = fp32 ? 1.0 - a.gp.root_rel32 : 1.0;
    C.rc = {C.root_keep, C.tie_dir, C.tie_rel};
    C.dom_rel = fp32 ? a.gp.dom_rel32 : a.gp.dom_rel;
    // rounds: wide ones mean fewer round changes, but on a surface with bend
    // vertices they launch vertices before their distances settle. A team
    // launches at round changes only and shares its distances there, so its
    // rounds are narrow: half an edge, three quarters, an edge, two and four
    // give 100 sources on the aspect-3 torus of 3456 faces 11.1, 11.5, 12.0, 13.7
    // and 16.1 M windows in 4.3, 4.3, 5.0, 6.9 and 8.3 ms (alone 11.3 M, 11.2 ms);
    // 100 on a flat grid of 3200, where half an edge is less than the smallest
    // step between vertices, 10.4, 6.0 and 5.9 ms for the first three (18.6).
    const double width = M.n_pseudo == 0 ? 16.0 : kTeam > 1 ? 0.75 : 4.0;
    C.bucket = uniform(!kDom ? INFINITY : a.gp.bucket > 0.0 ? a.gp.bucket : width * M.max_edge);
    C.cutoff = uniform(sd.cutoff);
    if constexpr (kNear) {
        // every entry of earlier sources is void; once the epochs are used
        // up, the tables are cleared and start over
        if (--epoch == 0) {
            for (int v = lane; v < (int)a.vstride; v += kWave) a.vdist[(int64_t)slot * a.vstride + v] = ~0ull;
            for (int h = lane; h < (int)a.hstride; h += kWave) a.split[(int64_t)slot * a.hstride + h] = ~0ull;
            epoch = a.epoch_max;
            wave_sync();
        }
    }
    const unsigned long long ep = kNear ? epoch : 0;
    const VertexTable<kNear> Dv{a.vdist + (int64_t)slot * a.vstride, ep};
    // one_split: FP64 passes (the FP32 pass's tie band is as wide as its
    // distances' errors) on surfaces with bend vertices, whose windows split
    // often (an aspect-3 torus of 3456 faces: 188k windows a source without
    // it, 112k with it); on a convex sphere one window in a hundred covers a
    // vertex, and the entries would cost more than the 1 % of windows they
    // save
    unsigned long long *Hv = kDom && !fp32 && M.n_pseudo > 0 && a.split ? a.split + (int64_t)slot * a.hstride : nullptr;
    C.split_rel = fmax(1e-6, 64.0 * C.tie_rel);
    const BendTable G = bend_table(a.roots, a.rstride, slot, a.rcap);
    RoundStack<R> S;
    S.lds = reinterpret_cast<typename RecOf<R>::T *>(stk);
    S.kL = stk_bytes / (int)sizeof(typename RecOf<R>::T);
    S.glb = reinterpret_cast<typename RecOf<R>::T *>(reinterpret_cast<Rec64 *>(a.stack) + (size_t)slot * a.gp.stack_cap);
    S.gcap = fp32 ? 2 * a.gp.stack_cap : a.gp.stack_cap;
    S.lsp = S.gsp = S.dsp = S.dl = 0;
    S.dir = 0;
    S.ldd = reinterpret_cast<typename RecOf<R>::T *>(later);

    // the profile's marks live in LDS, not in registers
    const bool prof = sd.prof != nullptr && lane == 0;
    if (prof) {
        L.clk[0] = clock64();
        L.clk[2] = L.clk[3] = 0;
        L.clk[5] = (long long)st.launches;
    }
    // ---- tables
    if constexpr (!kNear) {
        for (int v = lane; v < M.nv; v += kWave) Dv.p[v] = (unsigned long long)__double_as_longlong(INFINITY);
        if (Hv)
            for (int h = lane; h < 3 * M.nf; h += kWave) Hv[h] = ~0ull;
        if (kTeam > 1)
            for (int q = threadIdx.x; q < n; q += kWave * kTeam)
                td.best[q] = (unsigned long long)__double_as_longlong(INFINITY);
        if (kTeam > 1 && threadIdx.x == 0) team.overflow = team.more[0] = team.more[1] = 0;
        for (int j = lane; j < n; j += kWave) td[j] = TgtState{};
    }
    if (lane == 0) {
        L.B.npend = 0;
        L.B.ntouched = 0;
        L.unfound = kNear ? 0 : n - 1;
        L.maxb = C.cutoff < INFINITY ? C.cutoff * (fp32 ? 1.0 + fmax(a.gp.slack32, a.gp.guard_rel) : 1.0)
                                     : INFINITY;
    }
    if (kTeam > 1) __syncthreads();  // the shared state is ready
    else wave_sync();
    bool overflow = false;
    double T = C.bucket;

    // ---- seed from the source (root -1, sg = 0), in FP64
    const int fs = sd.face[src];
    const double sb[3] = {sd.bary[3 * (int64_t)src], sd.bary[3 * (int64_t)src + 1], sd.bary[3 * (int64_t)src + 2]};
    const HeRec R0 = he[3 * fs];
    const double P[3][2] = {{0.0, 0.0}, {R0.L, 0.0}, {R0.cx, R0.cy}};
    const double sx = sb[1] * P[1][0] + sb[2] * P[2][0], sy = sb[1] * P[1][1] + sb[2] * P[2][1];
    {
        // targets in the source's face: straight segments
        const bool mine = lane == 0 && member == 0;
        int q = mine ? sd.fstart[fs] : 0, q1 = mine ? sd.fstart[fs + 1] : 0;
        while (__ballot(q < q1)) {
            bool ok = false;
            int j = 0;
            double d = 0, tx = 0, ty = 0;
            if (q < q1) {
                const FaceTarget t = sd.ftgt[q];
                j = q;
                if (t.j != src) {
                    const double *b = t.b;
                    const double qx = b[1] * P[1][0] + b[2] * P[2][0], qy = b[1] * P[1][1] + b[2] * P[2][1];
                    const double dx = qx - sx, dy = qy - sy;
                    d = sqrt(dx * dx + dy * dy);
                    if (d > 0.0) {
                        tx = dx / d;
                        ty = dy / d;
                    }
                    ok = !kNear || d < L.maxb;
                }
                ++q;
            }
            target_update(L, td, C, ok, j, d, tx, ty, INFINITY);
        }
    }
    {
        Win<R> w, wa, wb;
        bool want = false, wantA = false, wantB = false;
        int rv = -1;
        double rd = 0, rtx = 0, rty = 0;
        double ka = 0, kb = 0;
        // a team's members take the source's angles in turn, four shares of each
        // edge a member (equal angles, so that on a smooth surface each has
        // its part of the windows; their ends are the same numbers on both
        // sides)
        constexpr int kShares = kTeam > 1 ? 4 : 1;
        if (lane < 3 * kShares) {
            const int k = lane % 3, share = lane / 3 * kTeam + member, h = 3 * fs + k;
            const HeRec Rh = he[h];
            const double ex = (P[(k + 1) % 3][0] - P[k][0]) / Rh.L, ey = (P[(k + 1) % 3][1] - P[k][1]) / Rh.L;
            const int v = M.T[h];
            {
                const double dx = P[k][0] - sx, dy = P[k][1] - sy;
                rd = sqrt(dx * dx + dy * dy);
                Dv.put(v, rd);
                rv = M.pidx[v];
                if (kTeam > 1 && (lane >= 3 || k % kTeam != member)) rv = -1;
                if (rv >= 0) {
                    rtx = rd > 0 ? dx / rd : 0.0;
                    rty = rd > 0 ? dy / rd : 0.0;
                }
            }
            const double hx = sb[(k + 1) % 3] * Rh.L + sb[(k + 2) % 3] * Rh.cx, hy = sb[(k + 2) % 3] * Rh.cy;
            if (Rh.twin >= 0) {
                w.px = (R)(Rh.L - hx);
                w.py = (R)(-hy);
                w.b0 = R(0);
                w.b1 = (R)Rh.L;
                if (kTeam > 1) {
                    // directions to the edge's ends and half way between them;
                    // within a half, steps along the chord are nearly equal angles
                    const double px = Rh.L - hx, qx = Rh.L - px;
                    const double n0 = 1.0 / sqrt(px * px + hy * hy), n1 = 1.0 / sqrt(qx * qx + hy * hy);
                    const double ux = -px * n0, uy = hy * n0, vx = qx * n1, vy = hy * n1;
                    const double nm = 1.0 / sqrt((ux + vx) * (ux + vx) + (uy + vy) * (uy + vy));
                    const double mx = (ux + vx) * nm, my = (uy + vy) * nm;
                    auto end = [&](int i) {
                        const double t = 2.0 * (double)i / (kShares * kTeam);
                        const double dx = t < 1.0 ? ux + t * (mx - ux) : mx + (t - 1.0) * (vx - mx);
                        const double dy = t < 1.0 ? uy + t * (my - uy) : my + (t - 1.0) * (vy - my);
                        const double x = px + hy * dx / dy;
                        return i <= 0 ? 0.0 : i >= kShares * kTeam ? (double)Rh.L : fmin(fmax(x, 0.0), (double)Rh.L);
                    };
                    if (sb[(k + 2) % 3] > 0.0) {
                        w.b0 = (R)end(share);
                        w.b1 = (R)end(share + 1);
                    }
                }
                w.sg = R(0);
                w.c = (R)(-ex);
                w.s = (R)(-ey);
                w.he = Rh.twin;
                w.root = -1;
                if (sb[(k + 2) % 3] > 0.0) {
                    want = w.b1 > w.b0;
                } else if (share == 0) {
                    // source on this edge: the face across contains it as well
                    const He<R> Ht = load_he(M, Rh.twin, R(0));
                    w.py = R(0);
                    if (Ht.tp >= 0) {
                        make_left(Ht, w, 0.0, (double)Ht.Lp, wa);
                        wantA = true;
                        ka = (double)seg_dist(wa.px, wa.py, wa.b0, wa.b1);
                    }
                    if (Ht.tn >= 0) {
                        make_right(Ht, w, 0.0, (double)Ht.Ln, wb);
                        wantB = true;
                        kb = (double)seg_dist(wb.px, wb.py, wb.b0, wb.b1);
                    }
                }
            }
        }
        if constexpr (kDom) bend_update(G, L.B, C.rc, rv >= 0, rv, rd, rtx, rty, INFINITY);
        // on-edge sources: targets and third vertex of the face across
        for (int k = 0; k < 3; ++k) {
            const bool on = sb[(k + 2) % 3] <= 0.0 && he[3 * fs + k].twin >= 0;
            if (!on || member != 0) continue;  // wave-uniform
            const HeRec Rh = he[3 * fs + k];
            const int t = Rh.twin, g = t / 3, m = t % 3;
            const HeRec Rt = he[t];
            const double ex = (P[(k + 1) % 3][0] - P[k][0]) / Rh.L, ey = (P[(k + 1) % 3][1] - P[k][1]) / Rh.L;
            const double c = -ex, s = -ey;
            const double ptx = Rh.L - (sb[(k + 1) % 3] * Rh.L + sb[(k + 2) % 3] * Rh.cx);
            int q = lane == 0 ? sd.fstart[g] : 0, q1 = lane == 0 ? sd.fstart[g + 1] : 0;
            while (__ballot(q < q1)) {
                bool ok = false;
                int j = 0;
                double d = 0, tx = 0, ty = 0;
                if (q < q1) {
                    const FaceTarget tg = sd.ftgt[q];
                    j = q;
                    if (tg.j != src) {
                        const double *b = sd.bary + 3 * (int64_t)tg.j;
                        const double qx = b[(m + 1) % 3] * Rt.L + b[(m + 2) % 3] * Rt.cx;
                        const double qy = b[(m + 2) % 3] * Rt.cy;
                        double dx = qx - ptx, dy = qy;
                        d = sqrt(dx * dx + dy * dy);
                        if (d > 0) {
                            dx /= d;
                            dy /= d;
                            tx = c * dx - s * dy;
                            ty = s * dx + c * dy;
                        }
                        ok = !kNear || d < L.maxb;
                    }
                    ++q;
                }
                target_update(L, td, C, ok, j, d, tx, ty, INFINITY);
            }
            const double dx = Rt.cx - ptx, dy = Rt.cy;
            const double d = sqrt(dx * dx + dy * dy);
            const int opp = Rt.opp_flags >> 1;
            if (lane == 0) Dv.put(opp, d);
            const int eo = lane == 0 ? M.pidx[opp] : -1;
            if constexpr (kDom) bend_update(G, L.B, C.rc, eo >= 0, eo, d, (c * dx - s * dy) / d, (s * dx + c * dy) / d, INFINITY);
        }
        S.push(want, false, w, overflow);
        S.push(wantA, ka >= T, wa, overflow);
        S.push(wantB, kb >= T, wb, overflow);
    }

    // ---- propagation, round by round
    if (prof) L.clk[1] = clock64();
    bool have = false;
    Win<R> w;
    double DA = INFINITY, DB = INFINITY;  // vertex distances of the window's half-edge (infinite: not read yet)
    unsigned long long nwin = 0;
    int pruned = 0, depth = 0;
    int round = 0;
    for (;;) {
        if (__ballot(overflow)) overflow = true;
        if (overflow) {
            if (kTeam == 1) break;
            // the others learn of it at the end of the round
            S.lsp = S.gsp = S.dsp = S.dl = 0;
            L.B.npend = 0;
            have = false;
        }
        depth = max(depth, S.lsp + S.gsp + S.dsp + S.dl);
        bool busy = S.refill(have, w);
        if (kDom && kTeam == 1 && !busy && L.B.npend > 0) {
            if (prof) L.clk[2] -= clock64();
            if (launch_roots<R, kNear, kTeam>(sd, L, G, td, Dv, C, S, T, src, st)) overflow = true;
            if (prof) L.clk[2] += clock64();
            // no lane holds a window here: nothing of one has to live through the launch
            w = Win<R>{};
            DA = DB = INFINITY;
            busy = S.refill(have, w);
        }
        if (kTeam > 1 && !busy) {
            // the end of the round, for the whole team: what each member has
            // learned on its own becomes common, then the bend vertices that
            // the round reached are launched, and the next one begins
            S.next_round(overflow);
            const bool lost = __ballot(overflow) != 0;
            if (lane == 0) {
                if (lost) team.overflow = 1;
                if (L.B.npend > 0 || S.gsp > 0) team.more[round & 1] = 1;
            }
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // this member's entries have arrived
            __syncthreads();
            const bool more = !team.overflow && team.more[round & 1];
            team_merge<kTeam>(a.vdist + (int64_t)blockIdx.x * kTeam * a.vstride, a.vstride, M.nv);
            key_bound(L, C, n, [&](int q) {
                return sd.ftgt[q].j == src ? 0.0 : __longlong_as_double((long long)team_load(td.best + q));
            });
            if (threadIdx.x == 0) team.more[~round & 1] = 0;
            __syncthreads();
            if (!more) break;
            T += C.bucket;
            if (L.B.npend > 0) {
                if (launch_roots<R, kNear, kTeam>(sd, L, G, td, Dv, C, S, T, src, st)) overflow = true;
                w = Win<R>{};
                DA = DB = INFINITY;
            }
            ++round;
            continue;
        }
        if (!busy) {
            if (S.dsp + S.dl == 0 && L.B.npend == 0) break;
            // next round; once every target is reached, bound the keys
            S.next_round(overflow);
            T += C.bucket;
            if (!kNear && L.unfound == 0) {
                wave_sync();  // every lane's target stores are visible
                key_bound(L, C, n, [&](int q) { return sd.ftgt[q].j == src ? 0.0 : td[q].d1; });
            }
            wave_sync();
            continue;
        }
        nwin += (unsigned long long)__popcll(__ballot(have));
        if (nwin > (unsigned long long)a.gp.max_windows) {
            overflow = true;
            if (kTeam == 1) break;
            continue;
        }
        if (prof) ++L.clk[3];
        // Three rounds of loads an iteration, each issued as a whole: the
        // records that the window names (half-edge and its entry, the face's
        // first target, the root's entry), then what those name (vertex
        // distances, the target, the third vertex's number), then the third
        // vertex's bend entry, which the children's arithmetic covers.
        He<R> H;
        int vA = 0, vB = 0, q0 = -1, qcnt = 0;
        bool act = have;
        double txc = 0.0;
        int k = 0;
        double wtx = 0.0, wty = 0.0, wD2 = INFINITY;  // the root's tangent and other-direction distance
        unsigned long long hw = ~0ull;
        if (act) {
            const int f = w.he / 3;
            k = w.he - 3 * f;
            H = load_he(he, hef, w.he, R(0));
            vA = he[w.he].tail;
            vB = he[w.he].head;
            if constexpr (kNear) {
                q0 = fstart[f];
                qcnt = fstart[f + 1] - q0;
            } else {
                q0 = ffirst[f];
            }
            if (Hv) hw = Hv[w.he];
            double rD = 0.0, rL = INFINITY;
            if (kDom && w.root >= 0) {
                rD = G.rD[w.root];
                rL = G.rL[w.root];
                wtx = G.rtx[w.root];
                wty = G.rty[w.root];
                wD2 = G.rD2[w.root];
                // stale: from an earlier launch of its root, or a new launch is due
                if (bend_stale(rD, rL, w, C.rc)) {
                    act = have = false;
                    ++st.stale;
                }
            }
            if (!act) {
                q0 = -1;
                qcnt = 0;
                DA = DB = INFINITY;
            }
        }
        double DC = INFINITY;
        bool cin = false, go_l = false, go_r = false;
        double dcv = 0.0, xa = 0.0, xb = 0.0;
        int eo = -1;
        FaceTarget t0{{0.0, 0.0, 0.0}, -1, 0};  // none
        TgtState c0;
        if (act) {
            // a lane that goes on with a child has the distances of the
            // half-edge's ends from the parent's face
            if constexpr (kDom) {
                if (!(DA < INFINITY)) DA = Dv[vA];
                if (!(DB < INFINITY)) DB = Dv[vB];
                DC = Dv[H.opp];
            }
            if (!kNear && q0 >= 0) {
                t0 = ftgt[q0];
                c0 = td[q0];
            }
            if (kDom && H.pseudo) eo = pidx[H.opp];
            const double px = w.px, py = w.py, sg = w.sg;
            txc = px + ((double)H.cx - px) * (-py) / ((double)H.cy - py);
            const double sl = C.tol * (double)H.L;
            cin = txc >= (double)w.b0 - sl && txc <= (double)w.b1 + sl;
            go_l = H.tp >= 0 && (double)w.b0 < txc;
            go_r = H.tn >= 0 && (double)w.b1 > txc;
            // the first child's interval, while the loads above are on their way
            if (Hv && cin) {
                const double dx = (double)H.cx - px, dy = (double)H.cy - py;
                dcv = sg + sqrt(dx * dx + dy * dy);
                const int sides = one_split(Hv, ep, w.he, hw, dcv, txc, (double)H.L, C.split_rel);
                go_l = go_l && (sides & 1);
                go_r = go_r && (sides & 2);
            }
            far_ends(H, w, txc, go_l, xa, xb);
            // vertices of the face reached through this window: the table's
            // values are combined with this window's own paths, which then go
            // to the table (compared in squares first: few are shorter)
            if constexpr (kDom) {
                const double rA = px * px + py * py, rB = ((double)H.L - px) * ((double)H.L - px) + py * py;
                if ((double)w.b0 <= 0.0 && Dv.shorter(rA, DA, sg)) {
                    DA = fmin(DA, sg + sqrt(rA));
                    Dv.put(vA, DA);
                }
                if ((double)w.b1 >= (double)H.L && Dv.shorter(rB, DB, sg)) {
                    DB = fmin(DB, sg + sqrt(rB));
                    Dv.put(vB, DB);
                }
                if (cin) {
                    const double dx = (double)H.cx - px, dy = (double)H.cy - py;
                    const double rC = dx * dx + dy * dy;
                    if (!Hv) dcv = sg + sqrt(rC);
                    if (Dv.shorter(rC, DC, sg)) {
                        DC = fmin(DC, dcv);
                        Dv.put(H.opp, DC);
                    }
                }
            }
        }
        if constexpr (kNear) query_pairs<kDom>(ftgt, L, td, C, qcnt, q0, src, k, H, w, wtx, wty, wD2);
        else query_face(ftgt, L, td, C, q0, src, k, H, w, wtx, wty, wD2, t0, c0);
        // third vertex as a bend vertex: its entry is loaded here and updated
        // after the children
        const bool ok3 = eo >= 0 && cin;
        BendEntry e3;
        if (ok3) e3 = bend_load(G, eo);
        // children, trimmed against the vertex paths and bounded by maxb. One
        // body serves both sides, its constants selected per lane: nearly
        // every window has one child, on either side, and the few with two
        // (the third vertex in their cone) run it again for the right one.
        Win<R> c1, c2;
        bool h1 = false, h2 = false;
        bool l1 = false, l2 = false;  // left for the next round
        const double maxb = L.maxb;
        auto child = [&](bool left, double x0, double x1, Win<R> &c, bool &hc, bool &lc) {
            const double hcx = H.cx, hcy = H.cy, hL = H.L;
            const double Lc = left ? (double)H.Lp : (double)H.Ln;
            // the child frame: axis (ax, ay), origin A (left: edge A -> C, S =
            // A, E = C) or C (right: edge C -> B, S = C, E = B)
            const R ax = left ? H.ex : H.ux, ay = left ? H.ey : H.uy;
            const R qx = left ? w.px : w.px - H.cx, qy = left ? w.py : w.py - H.cy;
            c.px = ax * qx + ay * qy;
            c.py = ax * qy - ay * qx;
            c.sg = w.sg;
            c.c = w.c * ax - w.s * ay;
            c.s = w.s * ax + w.c * ay;
            c.he = left ? H.tp : H.tn;
            c.root = w.root;
            const double DS = left ? DA : DC, DE = left ? DC : DB, DO = left ? DB : DA;
            // the face's remaining vertex (B or A) in the child frame
            const double rx = left ? hL : -hcx, ry = left ? 0.0 : -hcy;
            const double ox = (double)ax * rx + (double)ay * ry, oy = (double)ax * ry - (double)ay * rx;
            const double cpx = c.px, cpy = c.py, sg = c.sg;
            double r0 = (x0 - cpx) * (x0 - cpx) + cpy * cpy, r1 = (x1 - cpx) * (x1 - cpx) + cpy * cpy;
            if (kDom ? vertex_trim(cpx, cpy, sg, Lc, DS, DE, C.dom_rel, x0, x1, r0, r1) &&
                           !opposite_dominates(ox, oy, DO, sg, C.dom_rel, x0, x1, r0, r1)
                     : x1 - x0 > 1e-12 * Lc) {
                c.b0 = (R)x0;
                c.b1 = (R)x1;
                // the child's key (its smallest distance) against the bound
                // and the round's threshold
                const double rk = cpx < x0 ? r0 : cpx > x1 ? r1 : cpy * cpy;
                hc = !longer(rk, maxb - sg);
                lc = T <= sg || rk >= (T - sg) * (T - sg);
            }
            if (!hc) ++pruned;
        };
        if (go_l || go_r) child(go_l, xa, xb, c1, h1, l1);
        if (go_l && go_r) {
            far_ends(H, w, txc, false, xa, xb);
            child(false, xa, xb, c2, h2, l2);
        }
        if constexpr (kDom) {
            double tx = wtx, ty = wty, alt = INFINITY;
            if (ok3) {
                if (w.root < 0) {
                    R dx = H.cx - w.px, dy = H.cy - w.py;
                    const R l = sqrt(dx * dx + dy * dy);
                    tx = (double)(w.c * (dx / l) - w.s * (dy / l));
                    ty = (double)(w.s * (dx / l) + w.c * (dy / l));
                } else {
                    alt = wD2 + (dcv - (double)w.sg);
                }
            }
            bend_update_loaded(G, L.B, C.rc, ok3, eo, dcv, tx, ty, alt, e3);
        }
        // children of the next round wait; of the two of this round, the lane keeps one
        const bool keep1 = h1 && !l1, keep2 = h2 && !l2;
        S.push(h1 && !keep1, true, c1, overflow);
        S.push(h2 && (keep1 || !keep2), l2, c2, overflow);
        if (act) {
            // the kept child's half-edge runs A -> C (left) or C -> B
            DA = keep1 && go_l ? DA : keep1 || keep2 ? DC : INFINITY;
            DB = keep1 && go_l ? DC : keep1 || keep2 ? DB : INFINITY;
            if (keep1) w = c1;
            else if (keep2) w = c2;
            else have = false;
        }
    }

    // ---- results: row src, entry j for target j
    if (prof) L.clk[4] = clock64();
    const int32_t *Tt = M.T;
    const double *p0 = M.V + 3 * (int64_t)Tt[3 * fs], *p1 = M.V + 3 * (int64_t)Tt[3 * fs + 1];
    const double *nn = M.fnrm + 3 * (int64_t)fs;
    double ex3[3] = {p1[0] - p0[0], p1[1] - p0[1], p1[2] - p0[2]};
    const double el = sqrt(ex3[0] * ex3[0] + ex3[1] * ex3[1] + ex3[2] * ex3[2]);
    ex3[0] /= el;
    ex3[1] /= el;
    ex3[2] /= el;
    const double ey3[3] = {nn[1] * ex3[2] - nn[2] * ex3[1], nn[2] * ex3[0] - nn[0] * ex3[2],
                           nn[0] * ex3[1] - nn[1] * ex3[0]};
    bool ovf = __ballot(overflow) != 0;
    const int64_t c0 = (int64_t)src * sd.cap;
    bool near_cut = false;
    if (kTeam > 1) {
        if (ovf && lane == 0) team.overflow = 1;
        __syncthreads();  // every wavefront's targets are final
        ovf = team.overflow != 0;
    } else {
        wave_sync();  // every lane's tangent stores are visible
    }
    // one result: place s of the row, target at place q of the by-face index
    auto result = [&](int64_t o, int q, int j) {
        TgtState t = td[q];
        if constexpr (kTeam > 1) {
            // the team's wavefronts each hold their own paths' best: the
            // shortest wins, and the next of another direction
            const char *base = reinterpret_cast<const char *>(td.st) - member * a.tstride;
            t = *(reinterpret_cast<const TgtState *>(base) + q);
            for (int m = 1; m < kTeam; ++m) {
                const TgtState u = *(reinterpret_cast<const TgtState *>(base + m * a.tstride) + q);
                const bool differ = !(t.d1 < INFINITY) || !(u.d1 < INFINITY) ||
                                    fabs(t.tx * u.ty - t.ty * u.tx) > C.tie_dir || t.tx * u.tx + t.ty * u.ty < 0.0;
                const double worse = differ ? fmax(t.d1, u.d1) : INFINITY, d2 = fmin(fmin(t.d2, u.d2), worse);
                if (u.d1 < t.d1) t = u;
                t.d2 = d2;
            }
        }
        double d = t.d1;
        uint8_t fl = guard ? GSIM_PAIR_GUARD_BIT : 0;
        if (j == src) d = INFINITY;
        else if (ovf) d = NAN;
        if (j != src && t.d2 - d <= C.tie_rel * d) fl |= GSIM_PAIR_TIE_BIT;
        if (d == 0.0) fl |= GSIM_PAIR_ZERO_BIT;
        near_cut |= C.cutoff < INFINITY && fabs(d - C.cutoff) <= a.gp.guard_rel * C.cutoff;
        sd.cdist[o] = d;
        sd.cflags[o] = fl;
        for (int qd = 0; qd < 3; ++qd) sd.ctan[3 * o + qd] = t.tx * ex3[qd] + t.ty * ey3[qd];
    };
    if constexpr (!kNear) {
        // row src, entry j for target j
        for (int q = threadIdx.x; q < n; q += kWave * kTeam) {
            const int j = sd.ftgt[q].j;
            result(c0 + j, q, j);
        }
    } else {
        // the targets reached, in ascending particle order
        const int nt = L.unfound, cap = min(sd.cap, kBigCandMax);
        if (lane == 0) sd.cand_cnt[src] = nt;
        if (nt > cap) {
            st.overflow = true;  // more targets than the row holds
        } else {
            int P = 1;
            while (P < nt) P <<= 1;
            unsigned long long *key = P <= kSortLds ? sl->key : reinterpret_cast<unsigned long long *>(
                reinterpret_cast<char *>(a.sort) + (int64_t)slot * a.tstride);
            for (int s = lane; s < P; s += kWave) {
                unsigned long long x = ~0ull;
                if (s < nt) {
                    const int q = td.touch[s];
                    x = (unsigned long long)(unsigned)sd.ftgt[q].j << 32 | (unsigned)q;
                }
                key[s] = x;
            }
            wave_sync();
            // bitonic sort of key[0, P) ascending
            for (int kk = 2; kk <= P; kk <<= 1)
                for (int jj = kk >> 1; jj > 0; jj >>= 1) {
                    for (int s = lane; s < P; s += kWave) {
                        const int t = s ^ jj;
                        if (t > s) {
                            const unsigned long long x = key[s], y = key[t];
                            if ((x > y) == ((s & kk) == 0)) {
                                key[s] = y;
                                key[t] = x;
                            }
                        }
                    }
                    wave_sync();
                }
            for (int s = lane; s < nt; s += kWave) {
                const int j = (int)(key[s] >> 32);
                sd.cand[c0 + s] = j;
                result(c0 + s, (int)(unsigned)key[s], j);
            }
        }
        for (int s = lane; s < nt; s += kWave) td[td.touch[s]] = TgtState{};
        wave_sync();
    }
    if (prof) {
        long long *qp = sd.prof + 8 * (int64_t)src;
        const long long t_end = clock64();
        qp[0] += t_end - L.clk[0];
        qp[1] += L.clk[3];
        qp[2] += (long long)nwin;
        qp[3] += (long long)st.launches - L.clk[5];
        qp[4] += L.clk[1] - L.clk[0];
        qp[5] += L.clk[4] - L.clk[1] - L.clk[2];
        qp[6] += L.clk[2];
        qp[7] += t_end - L.clk[4];
    }
    st.windows += nwin;
    st.pruned += pruned;
    st.overflow |= ovf;
    st.depth = max(st.depth, depth);
    if constexpr (kDom) bend_reset(G, L.B);
    if constexpr (kTeam > 1) {
        __syncthreads();  // the row is written, and the tables are free again
    }
    return fp32 && !ovf && __ballot(near_cut) != 0;
}

// kNear: a pass with a cutoff whose rows hold only the targets within it
// (whole-mesh passes: a row holds every particle).
// kDom: with domination tests and bend vertices (false: near passes over
// surfaces without bend vertices).
// kTeam wavefronts per workgroup share one source (whole-mesh passes with few
// sources, whose one wavefront each would leave most of the device idle): each
// starts from its share of the source's angles and propagates a round on its
// own, with its own stack and tables. At the end of a round the team meets: the
// smallest vertex distance of any member becomes everyone's, the targets' best
// distances bound everyone's keys, and each member launches the bend vertices
// that it reached first by length. The target states are merged when all are
// done. Nothing that a member reads changes between two meetings, and minima
// do not depend on their order, so results repeat bit for bit. (Sharing the
// half-edge entries as well saves one window in a hundred and costs a sixth of
// the time.) 100 sources on the aspect-3 torus of 3456 faces take 11.2 ms alone
// and 4.3 ms in teams of eight, 200 on the sphere of 5120 faces 9.8 and 2.1.
// FP64 only: in FP32-mixed mode another order of paths could move a flag.
template <bool kMixed, int kStk, bool kNear, int kTeam, bool kDom>
__global__ __launch_bounds__(kWave *kTeam, 2) void k_geodesic_all(AllArgs a) {
    static_assert(kDom || kNear, "without domination: near passes only");
    static_assert(kTeam == 1 || (!kNear && !kMixed), "teams: whole-mesh passes, FP64");
    __shared__ AllLds Ls[kTeam];
    __shared__ typename SortOf<kNear>::T sorted;
    __shared__ alignas(16) unsigned char stks[kTeam][kStk];
    __shared__ alignas(16) unsigned char laters[kTeam][kWave * sizeof(Rec64)];
    __shared__ TeamLds team;
    const int member = kTeam == 1 ? 0 : __builtin_amdgcn_readfirstlane((int)threadIdx.x / kWave);
    AllLds &L = Ls[member];
    unsigned char *stk = stks[member], *later = laters[member];
    const int64_t off = ((int64_t)blockIdx.x * kTeam + member) * a.tstride;
    const TargetTable<kNear> td{reinterpret_cast<TgtState *>(reinterpret_cast<char *>(a.ttab) + off),
                                kNear ? reinterpret_cast<int32_t *>(reinterpret_cast<char *>(a.touch) + off) : nullptr,
                                kTeam > 1 ? a.best + (int64_t)blockIdx.x * a.tcap : nullptr};
    uint32_t epoch = kNear ? __builtin_amdgcn_readfirstlane(a.epoch[blockIdx.x]) : 0;
    SortLds *sl = kNear ? reinterpret_cast<SortLds *>(&sorted) : nullptr;
    const int lane = lane_id();
    const int total = a.bi.begin[a.bi.nsurf];
    int chunk = blockIdx.x % kChunks, chunks_left = kChunks;
    SrcStats st;
    st.windows = st.launches = st.guards = 0;
    st.stale = st.pruned = 0;
    st.depth = 0;
    st.overflow = false;
    unsigned long long c_limited = 0;
    int next = 0, left = 0;
    for (;;) {
        if (left == 0) {
            while (chunks_left > 0) {
                const int lo = (int)(((int64_t)total * chunk) / kChunks);
                const int hi = (int)(((int64_t)total * (chunk + 1)) / kChunks);
                int t = 0;
                if (lane == 0 && member == 0) t = atomicAdd(&a.work[chunk * kWorkStride], a.grab);
                t = __shfl(t, 0);
                if (kTeam > 1) {
                    // the first member claims for all
                    if (threadIdx.x == 0) team.idx = t;
                    __syncthreads();
                    t = team.idx;
                    __syncthreads();
                }
                if (lo + t < hi) {
                    next = lo + t;
                    left = min(a.grab, hi - next);
                    break;
                }
                chunk = (chunk + 1) % kChunks;
                --chunks_left;
            }
            if (left == 0) break;
        }
        const int idx = next++;
        --left;
        const int si = __builtin_amdgcn_readfirstlane(batch_surface(a.bi, idx));
        const SurfDesc &sd = a.sd[si];
        const int src = sd.ftgt[idx - a.bi.begin[si]].j;  // in the faces' order: neighbours run together
        if (!kNear && threadIdx.x == 0) sd.cand_cnt[src] = sd.n;
        st.overflow = false;
        bool again = !kMixed;
        if (kMixed) again = run_all<float, kNear, kTeam, kDom>(a, sd, L, td, stk, kStk, later, sl, team, member, src, false, epoch, st);
        if (again) {
            // FP64 (the plain path, or the recompute of an FP32 source whose
            // results come too close to the cutoff to decide in FP32)
            run_all<double, kNear, kTeam, kDom>(a, sd, L, td, stk, kStk, later, sl, team, member, src, kMixed, epoch, st);
            st.guards += kMixed && member == 0 ? 1 : 0;
        }
        if (st.overflow && member == 0) ++c_limited;
    }
    if (kNear && lane == 0) a.epoch[blockIdx.x] = epoch;
    unsigned long long pr = (unsigned long long)st.pruned, stale = (unsigned long long)st.stale;
    for (int o = 32; o > 0; o >>= 1) {
        pr += __shfl_xor(pr, o);
        stale += __shfl_xor(stale, o);
    }
    if (lane == 0) {
        // only the counts that are not zero, in one of several slots
        Counters *ctr = a.ctr + ((int)blockIdx.x % kCtrSlots) * kCtrStride;
        if (st.windows) atomicAdd(&ctr->windows, st.windows);
        if (pr) atomicAdd(&ctr->pruned, pr);
        if (st.launches) atomicAdd(&ctr->launches, st.launches);
        if (stale) atomicAdd(&ctr->stale, stale);
        if (st.guards) atomicAdd(&ctr->guards, st.guards);
        if (c_limited) atomicAdd(&ctr->limited, c_limited);
        if (st.depth) atomicMax(&ctr->max_depth, (unsigned long long)st.depth);
    }
}

using AllKernel = void (*)(AllArgs);
template <bool kMixed, bool kNear, bool kDom>
AllKernel kernel_of(int kb, int team) {
    if constexpr (!kNear && !kMixed) {
        if (team == 8) return &k_geodesic_all<kMixed, 4096, kNear, 8, kDom>;
        if (team == 4) return &k_geodesic_all<kMixed, 4096, kNear, 4, kDom>;
        if (team == 2) return &k_geodesic_all<kMixed, 4096, kNear, 2, kDom>;
    }
    if (kb <= 4) return &k_geodesic_all<kMixed, 4096, kNear, 1, kDom>;
    if (kb <= 8) return &k_geodesic_all<kMixed, 8192, kNear, 1, kDom>;
    return &k_geodesic_all<kMixed, 16384, kNear, 1, kDom>;
}
AllKernel kernel_for(int kb, bool fp32, AllPass pass, int team) {
    if (pass == kNearPlain) return fp32 ? kernel_of<true, true, false>(kb, team) : kernel_of<false, true, false>(kb, team);
    if (pass == kNearPass) return fp32 ? kernel_of<true, true, true>(kb, team) : kernel_of<false, true, true>(kb, team);
    return fp32 ? kernel_of<true, false, true>(kb, team) : kernel_of<false, false, true>(kb, team);
}

static_assert(sizeof(TgtState) == 32, "a NearArea's target state");

}  // namespace

hipError_t launch_near_init(char *area, int first, int nslots, int tcap, unsigned long long *vdist, int64_t vstride,
                            unsigned long long *split, int64_t hstride, uint32_t *epoch, uint32_t epoch_max, hipStream_t s) {
    // every target unreached, every vertex and half-edge entry void. (A
    // double of all-ones bits would be a NaN: the states get infinities.)
    const int64_t n = nslots - first, bytes = NearArea(tcap).bytes;
    hipError_t e = launch_fill_u64(reinterpret_cast<unsigned long long *>(area + first * bytes), n * bytes / 8,
                                   0x7ff0000000000000ull, s);
    if (e == hipSuccess) e = launch_fill_u64(vdist + first * vstride, n * vstride, ~0ull, s);
    if (e == hipSuccess && hstride) e = launch_fill_u64(split + first * hstride, n * hstride, ~0ull, s);
    if (e == hipSuccess) e = launch_fill_u32(epoch + first, n, epoch_max, s);
    return e;
}

hipError_t launch_geodesic_all(const SurfDesc *desc, const BatchIdx &bi, const GeoParams &gp, const GeoShape &shape,
                               char *stack_mem, unsigned long long *vdist, int64_t vstride, char *roots, int64_t rstride,
                               int rcap, void *ttab, int tcap, unsigned long long *split, int64_t hstride,
                               uint32_t *epoch, uint32_t epoch_max, AllPass pass, int team, unsigned long long *best,
                               int32_t *work_ctr, Counters *ctr, bool fp32, hipStream_t s, hipEvent_t ev0, hipEvent_t ev1) {
    const bool near = pass != kWholeMesh;
    if (near && !epoch) return hipErrorInvalidValue;
    AllArgs a;
    a.sd = desc;
    a.bi = bi;
    a.gp = gp;
    a.stack = stack_mem;
    a.vdist = vdist;
    a.vstride = vstride;
    a.split = split;
    a.hstride = hstride;
    a.roots = roots;
    a.rstride = rstride;
    a.rcap = rcap;
    a.work = work_ctr;
    a.ctr = ctr;
    a.ttab = static_cast<TgtState *>(ttab);
    a.tcap = tcap;
    const NearArea na(tcap);
    a.tstride = near ? na.bytes : (int64_t)tcap * sizeof(TgtState);
    a.touch = near ? reinterpret_cast<int32_t *>(static_cast<char *>(ttab) + na.touch) : nullptr;
    a.sort = near ? reinterpret_cast<unsigned long long *>(static_cast<char *>(ttab) + na.sort) : nullptr;
    a.epoch = epoch;
    a.epoch_max = epoch_max;
    a.grab = shape.grab < 1 ? 1 : shape.grab;
    if (shape.nslots < 1 || bi.begin[bi.nsurf] < 1) return hipSuccess;
    if (team < 1 || shape.nslots % team || (team > 1 && (near || fp32 || !best))) return hipErrorInvalidValue;
    a.best = best;
    const AllKernel f = kernel_for(shape.lds_stack_kb, fp32, pass, team);
    const dim3 grid(shape.nslots / team), block(kWave * team);
    const uint32_t pad = shape.pad_lds > 0 ? (uint32_t)shape.pad_lds : 0;
    if (ev0 || ev1) hipExtLaunchKernelGGL(f, grid, block, pad, s, ev0, ev1, 0, a);
    else hipLaunchKernelGGL(f, grid, block, pad, s, a);
    return hipGetLastError();
}

size_t geodesic_all_lds_bytes(int lds_stack_kb, bool fp32, AllPass pass) {
    hipFuncAttributes at{};
    if (hipFuncGetAttributes(&at, (const void *)kernel_for(lds_stack_kb, fp32, pass, 1)) != hipSuccess) return 65536;
    return at.sharedSizeBytes;
}

int geodesic_all_waves_per_cu(int lds_stack_kb, bool fp32, AllPass pass, int team) {
    int nb = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, (const void *)kernel_for(lds_stack_kb, fp32, pass, team),
                                                     kWave * team, 0) != hipSuccess)
        return 0;
    return nb * team;
}

}  // namespace gsim
