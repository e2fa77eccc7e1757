// Initial placement on the device: random sequential addition in rounds
// (App. A starts from a dilute, non-overlapping configuration placed with a
// cell list; the algorithm is our reading, stated in include/rcp.h).
//
// Spheres are ranked largest first and placed class by class (size class
// floor(log2(D0 / D0_min)), largest class first).  A round takes a window of
// consecutive ranks of one class; every unplaced sphere of the window
// proposes the position of its next attempt, from the SplitMix64 counter
// stream of the host placement; a proposal is valid when it overlaps no
// placed sphere, and a valid proposal is accepted unless a valid proposal of
// a lower rank in the same round overlaps it.  Accepted spheres are placed,
// the others move on to their next attempt.  The result depends on the
// window but not on timing: every decision is a function of the proposals
// and of the spheres placed before the round.
//
// Placed spheres are binned per class on a grid of cells at least as wide
// as kappa0 times the class's largest diameter (a sphere meets only spheres
// of its own class or larger ones, so the 27 cells around it in each
// larger-or-equal class's grid hold every sphere it can overlap), kept as an
// open-addressing hash of occupied cells with a linked list per cell.  The
// proposals of a round are binned the same way in a table of their own.
//
// Ranks, rounds and classes advance on the device (PlaceState): a round is
// three launches, the host queues several and reads the state back once for
// them.
//
// Compiled without floating-point contraction: the overlap test rounds
// exactly as the host placement's.
#include "rcp_kernels.hpp"

namespace rcp {

constexpr uint64_t kPlaceEmpty = ~0ull;

__device__ __forceinline__ uint64_t sm64(uint64_t seed, uint64_t k)
{
    // SplitMix64 output function (Steele, Lea and Flood 2014) at counter k
    uint64_t z = seed + (k + 1u) * 0x9E3779B97F4A7C15ull;
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    return z ^ (z >> 31);
}

__device__ __forceinline__ double place_u01(uint64_t seed, uint64_t i, uint64_t attempt, int axis)
{
    const uint64_t k = ((i << 24) | attempt) * 4u + (uint64_t)axis;
    return (double)(sm64(seed, k) >> 11) * 0x1p-53;
}

__device__ __forceinline__ double place_mi(double d, double L, double hL)
{
    return d > hL ? d - L : (d < -hL ? d + L : d);
}

__device__ __forceinline__ int64_t place_cell(double v, double inv_w, int64_t nc)
{
    int64_t c = (int64_t)(v * inv_w);
    return c < 0 ? 0 : (c >= nc ? nc - 1 : c);
}

__device__ __forceinline__ uint64_t place_mix(uint64_t k)
{
    k ^= k >> 33;
    k *= 0xff51afd7ed558ccdull;
    k ^= k >> 33;
    return k;
}

// Head of the list of cell `key` (or -1).
__device__ __forceinline__ int32_t place_find(const PlaceSlot *tab, uint64_t mask, uint64_t key)
{
    for (uint64_t s = place_mix(key) & mask;; s = (s + 1) & mask) {
        const uint64_t k = tab[s].key;
        if (k == key) return tab[s].head;
        if (k == kPlaceEmpty) return -1;
    }
}

// Push item v on the list of cell `key`; returns the previous head.
__device__ __forceinline__ int32_t place_push(PlaceSlot *tab, uint64_t mask, uint64_t key, int32_t v)
{
    for (uint64_t s = place_mix(key) & mask;; s = (s + 1) & mask) {
        const unsigned long long prev =
            atomicCAS((unsigned long long *)&tab[s].key, (unsigned long long)kPlaceEmpty,
                      (unsigned long long)key);
        if (prev == kPlaceEmpty || prev == key) return atomicExch(&tab[s].head, v);
    }
}

// hLa[ax] = L / 2, or +inf on an axis bounded by walls (no image).
__device__ __forceinline__ bool place_overlap(double xj, double yj, double zj, const double *p,
                                              double dj, double di, double kappa0, double L,
                                              const double *hLa)
{
#pragma clang fp contract(off)
    const double dx = place_mi(xj - p[0], L, hLa[0]);
    const double dy = place_mi(yj - p[1], L, hLa[1]);
    const double dz = place_mi(zj - p[2], L, hLa[2]);
    const double r2 = (dx * dx + dy * dy) + dz * dz;
    const double dd = kappa0 * (0.5 * (di + dj));
    return r2 < dd * dd;
}

// Lanes that look at the cells around one proposal: one per cell of the
// 27-cell stencil (the lookups are chains of dependent reads; a thread per
// proposal walking 27 cells of every class took 168 us a round on average on 2e5
// spheres of size ratio 1e3, 27 lanes 21).
constexpr int kPlaceLanes = 32;
constexpr int kPlacePer = kBlock / kPlaceLanes;

// Cell of stencil lane l around p in grid g, for partners within reach (the
// largest centre distance at which they can overlap): false when the lane has
// no cell or no point of its cell is that near.  Fewer than three cells per
// axis: every cell once.
__device__ __forceinline__ bool place_lane_cell(const PlaceGrid &g, const double *p, double reach,
                                                int l, uint64_t &key)
{
    if (l >= 27) return false;
    const int o[3] = {l / 9, (l / 3) % 3, l % 3};
    const int64_t nc = g.nc;
    // cell units, with a margin far above the rounding of p * inv_w
    const double rc = reach * g.inv_w * (1.0 + 1e-9) + 1e-8;
    double d2 = 0.0;
    int64_t a[3];
#pragma unroll
    for (int ax = 0; ax < 3; ++ax) {
        if (nc < 3) {
            if (o[ax] >= nc) return false;
            a[ax] = o[ax];
            continue;
        }
        const int64_t c = place_cell(p[ax], g.inv_w, nc);
        const double f = p[ax] * g.inv_w - (double)c;
        const double d = o[ax] == 0 ? f : (o[ax] == 2 ? 1.0 - f : 0.0);
        if (d > 0.0) d2 += d * d;
        a[ax] = c + o[ax] - 1;
        a[ax] = a[ax] < 0 ? a[ax] + nc : (a[ax] >= nc ? a[ax] - nc : a[ax]);
    }
    key = ((uint64_t)a[0] * (uint64_t)nc + (uint64_t)a[1]) * (uint64_t)nc + (uint64_t)a[2];
    return d2 <= rc * rc;
}

// Whether any lane of this proposal's group sees a hit.
__device__ __forceinline__ bool group_any(bool hit)
{
    const uint64_t m = __ballot(hit);
    return ((m >> (threadIdx.x & kPlaceLanes)) & 0xffffffffull) != 0;
}

// Sort keys of the ranks (largest first, ties by index: the sort is stable)
// and the diameters by sphere, from the records.
__global__ __launch_bounds__(kBlock) void k_place_keys(const P4 *Q, const int32_t *orig, int64_t n,
                                                      double *__restrict__ d0)
{
    const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (i < n) d0[orig[i]] = fabs(Q[i].d);
}

__global__ __launch_bounds__(kBlock) void k_place_init(PlaceArgs a, int64_t tcap,
                                                      uint64_t *__restrict__ keys,
                                                      uint32_t *__restrict__ vals)
{
    const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (i < tcap) {
        a.tab[i].key = kPlaceEmpty;
        a.tab[i].head = -1;
    }
    if (i < a.n) {
        a.att[i] = 0;
        a.placed[i] = 0;
        keys[i] = ~(uint64_t)__double_as_longlong(a.d0[i]);
        vals[i] = (uint32_t)i;
    }
    if (i == 0) {
        PlaceState st;
        st.lo = st.hi = 0;
        st.first = 0;
        st.rounds = 0;
        st.cls = a.ncls;
        st.fail = 0;
        st.done = 0;
        st.pad = 0;
        *a.st = st;
    }
}

// Start of a round: the proposal table cleared; the window moved to the
// lowest rank still unplaced, or to the next smaller class.
__global__ __launch_bounds__(kBlock) void k_place_begin(PlaceArgs a)
{
    const int64_t s = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (s < a.pcap) {
        a.ptab[s].key = kPlaceEmpty;
        a.ptab[s].head = -1;
    }
    if (s != 0) return;
    PlaceState st = *a.st;
    if (st.done) return;
    if (st.fail) {
        st.lo = st.hi = a.n;
        st.done = 1;
        *a.st = st;
        return;
    }
    int64_t lo = (int64_t)st.first;
    while (st.cls == a.ncls || lo >= a.grid[st.cls].end) {
        if (st.cls == 0) {
            st.done = 1;
            break;
        }
        --st.cls;
    }
    if (st.done) {
        st.lo = st.hi = a.n;
    } else {
        const int64_t e = a.grid[st.cls].end;
        st.lo = lo;
        st.hi = lo + a.window < e ? lo + a.window : e;
        st.first = (unsigned long long)st.hi;
        ++st.rounds;
    }
    *a.st = st;
}

// Proposals of the window's unplaced ranks: position of the next attempt,
// validity (clear of the walls, if any, and of the placed spheres of this
// class and larger ones), and the valid ones binned in the proposal table.
__global__ __launch_bounds__(kBlock) void k_place_propose(PlaceArgs a)
{
    const int64_t lo = a.st->lo, hi = a.st->hi;
    const int c = a.st->cls;
    const int l = (int)(threadIdx.x & (kPlaceLanes - 1));
    const int64_t s = (int64_t)blockIdx.x * kPlacePer + threadIdx.x / kPlaceLanes;
    const int64_t k = lo + s;
    if (k >= hi || a.placed[k]) {
        if (k < hi && l == 0) a.valid[s] = 0;
        return;
    }
    const int32_t i = a.ord[k];
    const double di = a.d0[i];
    double p[3];
    for (int ax = 0; ax < 3; ++ax) {
        // in two dimensions z = 0 (axis 2 of the stream is not drawn)
        double v = ax < a.dim ? place_u01(a.seed, (uint64_t)i, (uint64_t)a.att[k], ax) * a.L : 0.0;
        if (v >= a.L) v -= a.L;
        p[ax] = v;
    }
    const int32_t bounded = a.walls | a.round;
    const double hLa[3] = {(bounded & 1) ? INFINITY : a.hL, (bounded & 2) ? INFINITY : a.hL,
                           (bounded & 4) ? INFINITY : a.hL};
    bool ok = !bounded || inside_walls(p, a.kappa0 * di, a.L, a.walls, a.round);
    for (int cc = c; cc < a.ncls && ok; ++cc) {
        const PlaceGrid &g = a.grid[cc];
        if (!g.any) continue;
        uint64_t key = 0;
        bool hit = false;
        if (place_lane_cell(g, p, a.kappa0 * (0.5 * (di + g.dmax)), l, key))
            for (int32_t j = place_find(a.tab + g.off, g.mask, key); j >= 0 && !hit; j = a.next[j])
                hit = place_overlap(a.x[3 * j], a.x[3 * j + 1], a.x[3 * j + 2], p, a.d0[j], di,
                                    a.kappa0, a.L, hLa);
        ok = !group_any(hit);
    }
    if (l != 0) return;
    for (int ax = 0; ax < 3; ++ax) a.prop[3 * s + ax] = p[ax];
    a.valid[s] = ok ? 1 : 0;
    if (!ok) return;
    const PlaceGrid &g = a.grid[c];
    const uint64_t key = ((uint64_t)place_cell(p[0], g.inv_w, g.nc) * (uint64_t)g.nc +
                          (uint64_t)place_cell(p[1], g.inv_w, g.nc)) * (uint64_t)g.nc +
                         (uint64_t)place_cell(p[2], g.inv_w, g.nc);
    a.pnext[s] = place_push(a.ptab, a.pmask, key, (int32_t)s);
}

// Conflicts among the round's valid proposals (the lower rank wins), then
// the accepted spheres are placed and the others move on to their next
// attempt; st->first receives the lowest rank of the window still unplaced.
__global__ __launch_bounds__(kBlock) void k_place_commit(PlaceArgs a)
{
    const int64_t lo = a.st->lo, hi = a.st->hi;
    const int c = a.st->cls;
    const int l = (int)(threadIdx.x & (kPlaceLanes - 1));
    const int64_t s = (int64_t)blockIdx.x * kPlacePer + threadIdx.x / kPlaceLanes;
    const int64_t k = lo + s;
    if (k >= hi || a.placed[k]) return;
    const int32_t i = a.ord[k];
    const double di = a.d0[i];
    const double p[3] = {a.prop[3 * s], a.prop[3 * s + 1], a.prop[3 * s + 2]};
    const int32_t bounded = a.walls | a.round;
    const double hLa[3] = {(bounded & 1) ? INFINITY : a.hL, (bounded & 2) ? INFINITY : a.hL,
                           (bounded & 4) ? INFINITY : a.hL};
    const PlaceGrid &g = a.grid[c];
    bool acc = a.valid[s] != 0;
    if (acc) {
        uint64_t key = 0;
        bool hit = false;
        if (place_lane_cell(g, p, a.kappa0 * (0.5 * (di + g.dmax)), l, key))
            for (int32_t s2 = place_find(a.ptab, a.pmask, key); s2 >= 0 && !hit; s2 = a.pnext[s2])
                hit = s2 < s && place_overlap(a.prop[3 * s2], a.prop[3 * s2 + 1],
                                              a.prop[3 * s2 + 2], p, a.d0[a.ord[lo + s2]], di,
                                              a.kappa0, a.L, hLa);
        acc = !group_any(hit);
    }
    if (l != 0) return;
    if (acc) {
        a.x[3 * i] = p[0];
        a.x[3 * i + 1] = p[1];
        a.x[3 * i + 2] = p[2];
        a.placed[k] = 1;
        const uint64_t key = ((uint64_t)place_cell(p[0], g.inv_w, g.nc) * (uint64_t)g.nc +
                              (uint64_t)place_cell(p[1], g.inv_w, g.nc)) * (uint64_t)g.nc +
                             (uint64_t)place_cell(p[2], g.inv_w, g.nc);
        a.next[i] = place_push(a.tab + g.off, g.mask, key, i);
    } else {
        if (++a.att[k] >= a.max_attempts) atomicOr(&a.st->fail, 1);
        atomicMin(&a.st->first, (unsigned long long)k);
    }
}

// Seating (a cascade stage, Sec. 4: the finer class is seated in the voids
// of the coarser ones): each sphere on its own, its first proposal of the
// placement counter stream that overlaps no frozen sphere, r^2 < dd^2 with
// dd = (D_j + kappa0 D0_i) / 2 and the separation x_j - p (minimum image).
__global__ __launch_bounds__(kBlock) void k_seat(SeatArgs a, int64_t ng)
{
#pragma clang fp contract(off)
    const int64_t t = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (t >= ng) return;
    const int32_t i = a.gidx[t];
    const double di = a.gd[t];
    const int64_t nc = a.nc;
    // fewer than three cells per axis: every cell once
    const bool wrap = nc >= 3;
    const int64_t m = wrap ? 3 : nc;
    for (int64_t att = 0; att < a.max_attempts; ++att) {
        double p[3];
        for (int ax = 0; ax < 3; ++ax) {
            double v = ax < a.dim ? place_u01(a.seed, (uint64_t)i, (uint64_t)att, ax) * a.L : 0.0;
            if (v >= a.L) v -= a.L;
            p[ax] = v;
        }
        const int64_t cx = place_cell(p[0], a.inv_w, nc), cy = place_cell(p[1], a.inv_w, nc),
                      cz = place_cell(p[2], a.inv_w, nc);
        bool ok = true;
        for (int64_t ox = 0; ox < m && ok; ++ox)
            for (int64_t oy = 0; oy < m && ok; ++oy)
                for (int64_t oz = 0; oz < m && ok; ++oz) {
                    int64_t ax = ox, ay = oy, az = oz;
                    if (wrap) {
                        ax += cx - 1, ay += cy - 1, az += cz - 1;
                        ax = ax < 0 ? ax + nc : (ax >= nc ? ax - nc : ax);
                        ay = ay < 0 ? ay + nc : (ay >= nc ? ay - nc : ay);
                        az = az < 0 ? az + nc : (az >= nc ? az - nc : az);
                    }
                    const int64_t q = (ax * nc + ay) * nc + az;
                    for (int32_t o = a.start[q]; o < a.start[q + 1]; ++o) {
                        const double dx = place_mi(a.fxd[4 * o] - p[0], a.L, a.hL);
                        const double dy = place_mi(a.fxd[4 * o + 1] - p[1], a.L, a.hL);
                        const double dz = place_mi(a.fxd[4 * o + 2] - p[2], a.L, a.hL);
                        const double r2 = (dx * dx + dy * dy) + dz * dz;
                        const double dd = 0.5 * (a.fxd[4 * o + 3] + a.kappa0 * di);
                        if (r2 < dd * dd) {
                            ok = false;
                            break;
                        }
                    }
                }
        if (ok) {
            a.x[3 * (int64_t)i] = p[0];
            a.x[3 * (int64_t)i + 1] = p[1];
            a.x[3 * (int64_t)i + 2] = p[2];
            return;
        }
    }
    atomicOr(a.fail, 1);
}

void launch_seat(const SeatArgs &a, int64_t ng, hipStream_t st)
{
    if (ng <= 0) return;
    hipLaunchKernelGGL(k_seat, dim3((unsigned)((ng + kBlock - 1) / kBlock)), dim3(kBlock), 0, st,
                       a, ng);
}

void launch_place_init(const PlaceArgs &a, const P4 *Q, const int32_t *orig, double *d0,
                       int64_t tcap, uint64_t *keys, uint32_t *vals, hipStream_t st)
{
    const unsigned gn = (unsigned)((a.n + kBlock - 1) / kBlock);
    hipLaunchKernelGGL(k_place_keys, dim3(gn), dim3(kBlock), 0, st, Q, orig, a.n, d0);
    const int64_t m = a.n > tcap ? a.n : tcap;
    hipLaunchKernelGGL(k_place_init, dim3((unsigned)((m + kBlock - 1) / kBlock)), dim3(kBlock), 0,
                       st, a, tcap, keys, vals);
}

void launch_place_round(const PlaceArgs &a, hipStream_t st)
{
    const unsigned gc = (unsigned)((a.pcap + kBlock - 1) / kBlock);
    hipLaunchKernelGGL(k_place_begin, dim3(gc), dim3(kBlock), 0, st, a);
    const unsigned g = (unsigned)((a.window + kPlacePer - 1) / kPlacePer);
    hipLaunchKernelGGL(k_place_propose, dim3(g), dim3(kBlock), 0, st, a);
    hipLaunchKernelGGL(k_place_commit, dim3(g), dim3(kBlock), 0, st, a);
}

}  // namespace rcp
