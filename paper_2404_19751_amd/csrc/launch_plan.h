// Host arithmetic of launches and scratch memory, free of HIP.
#pragma once
#include <stdint.h>

#include <algorithm>

namespace gsim {

// Blocks of a kernel that strides over n items (fills of tables that may hold
// billions of entries): a launch takes fewer than 2^32 threads, and 2^20
// blocks keep every compute unit busy to the end.
constexpr int64_t kFillBlocksMax = 1 << 20;
inline int fill_blocks(int64_t n, int block) {
    return (int)std::min<int64_t>((n + block - 1) / block, kFillBlocksMax);
}

// Byte offsets of one wavefront's near-pass area for tcap particles: target
// states (32 bytes each), the list of targets reached, sort keys.
constexpr int kBigCandMax = 4096;  // the most targets of a source
struct NearArea {
    int64_t touch, sort, bytes;
    explicit NearArea(int64_t tcap)
        : touch(32 * tcap), sort((touch + 4 * tcap + 15) / 16 * 16),
          bytes((sort + 8 * (int64_t)kBigCandMax + 255) / 256 * 256) {}
};

// The tables of one wavefront of a near pass: target area of tcap particles,
// vertex and half-edge entries.
struct NearLayout {
    int64_t tcap = 0, vstride = 0, hstride = 0;
    bool operator==(const NearLayout &o) const { return tcap == o.tcap && vstride == o.vstride && hstride == o.hstride; }
};
// Records (of 64 bytes) of a near pass's window stack. Near passes go round by
// round: what waits at once is a front around the source, not a depth-first
// path. The deepest measured hold 3.6 records for each face within the cutoff
// (a flat disc's share of nf faces) in FP64 and 3.3 in FP32-mixed (tori, bumpy
// spheres, height fields, flat and corrugated sheets, 5 to 55 % of the surface;
// whole-mesh passes, which go the same way, have `all` records). At least
// `cap` records, the depth of depth-first passes, and in powers of two so that
// cutoffs next to each other ask for the same.
inline int near_stack_records(double nf, double disc_share, int cap, int all) {
    const double want = 8.0 * nf * std::min(1.0, disc_share);
    int64_t n = 1024;
    while ((double)n < want && n < all) n *= 2;
    return (int)std::max<int64_t>(cap, std::min<int64_t>(n, all));
}

// What a near pass asks for: its layout, bytes of a bend-vertex table and of a
// window stack, and the wavefronts that could run at once.
struct NearNeed {
    NearLayout lay;
    int64_t roots = 0, stack = 0;
    int64_t waves = 1;
};
// Bytes of a wavefront's buffers, in this order: stack, bend-vertex table,
// target area, vertex entries, half-edge entries, epoch.
constexpr int kNearBufs = 6;
inline void near_wave_bytes(const NearNeed &w, double b[kNearBufs]) {
    b[0] = (double)w.stack;
    b[1] = (double)w.roots;
    b[2] = (double)NearArea(w.lay.tcap).bytes;
    b[3] = 8.0 * (double)w.lay.vstride;
    b[4] = 8.0 * (double)w.lay.hstride;
    b[5] = 4.0;
}
// Bytes that the buffers (holding `held`) must grow by for `waves` wavefronts:
// a buffer too small is freed and allocated anew with a quarter more.
inline double near_growth(const NearNeed &w, int64_t waves, const double held[kNearBufs]) {
    double b[kNearBufs], g = 0.0;
    near_wave_bytes(w, b);
    for (int k = 0; k < kNearBufs; ++k)
        if ((double)waves * b[k] > held[k]) g += 1.25 * (double)waves * b[k] - held[k];
    return g;
}
// The wavefronts of a near pass: as many as could run, within the scratch
// budget and with room left on the device (nine tenths of what is free).
inline int64_t near_waves(const NearNeed &w, double budget, double free_bytes, const double held[kNearBufs]) {
    double b[kNearBufs], all = 0.0;
    near_wave_bytes(w, b);
    for (double x : b) all += x;
    int64_t lo = 1, hi = std::max<int64_t>(1, std::min<int64_t>(w.waves, (int64_t)(budget / all)));
    while (lo < hi) {
        const int64_t mid = (lo + hi + 1) / 2;
        if (near_growth(w, mid, held) <= 0.9 * free_bytes) lo = mid;
        else hi = mid - 1;
    }
    return lo;
}

// Does a near pass of n particles have room for half the wavefronts that could
// run (`resident` on the device)? Every wavefront keeps a state for each of the
// surface's particles, so with a million the budget holds a thousand of them,
// and a pass whose targets fit the cutoff kernel's table is better off there.
inline bool near_fills_device(const NearNeed &w, int64_t resident, double budget) {
    double b[kNearBufs], all = 0.0;
    near_wave_bytes(w, b);
    for (double x : b) all += x;
    return 2.0 * budget / all >= (double)std::min(resident, w.lay.tcap);
}

// The layout to run a pass in that needs `need` where the tables are prepared
// for `cur`: one that holds both, so that surfaces and particle counts used in
// turn settle on one layout (tables of another are prepared anew, which costs
// a fill of all of them), with a quarter to spare where the particles have
// outgrown it.
inline NearLayout near_joint(const NearLayout &cur, const NearLayout &need) {
    if (cur.tcap == 0) return need;
    NearLayout j;
    j.tcap = need.tcap > cur.tcap ? std::max(need.tcap, cur.tcap + cur.tcap / 4) : cur.tcap;
    j.vstride = std::max(cur.vstride, need.vstride);
    j.hstride = std::max(cur.hstride, need.hstride);
    return j;
}

}  // namespace gsim
