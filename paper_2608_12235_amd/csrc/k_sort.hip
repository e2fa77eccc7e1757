// Stable LSD radix sort of (u64 key, u32 value) pairs and of u64 keys, for
// the neighbour-list build (Morton ordering, entry sort), of several arrays
// at once.
//
// Sort: the fewest passes with digits of at most nine bits, all as narrow as
// that allows; tiles of 2048 keys (256 threads x 8 rounds).  Per pass:
// per-tile digit histogram -> per digit, an exclusive scan over the tiles
// and the digit's total (one block per digit) -> stable scatter, which adds
// the totals of the smaller digits and ranks each key among equal digits of
// its wave's 512 with ballots and a counter row of the wave's own in LDS:
// no barrier between the rounds.
// A pass over a few tiles is bound by latency: the scatter of four tiles
// took 8.5 us with eight-bit digits and four barriers a round, 7.1 now.
// Nine-bit digits save a pass at 17 and 18, 25 to 27, 33 to 36, ... bits.
// The keys of a tile go through LDS in digit order, so that a wave's stores
// are runs of several keys.  The whole build of 1e5 spheres (5.2e5 entries):
// 244 -> 227 us; of 1.2e5 with 3.9e6 entries: 561 -> 505; of 512: 174 -> 155.
#include "rcp_kernels.hpp"

namespace rcp {

constexpr int kTile = kBlock * 8;   // 2048 items per tile
constexpr int kMaxDigits = 512;     // two a thread
static_assert(kTile == kSortTile && kMaxDigits == kSortDigits && kMaxDigits == 2 * kBlock, "");

// ---------------------------------------------------------------- scan
// Scans of one value per thread across the block: the exclusive prefix, and
// the block total in *total.
__device__ __forceinline__ uint32_t block_exclusive(uint32_t v, uint32_t *total)
{
    __shared__ uint32_t ws[kWavesPerBlock];
    const int lane = threadIdx.x & (kWave - 1), w = threadIdx.x / kWave;
    uint32_t inc = v;
#pragma unroll
    for (int o = 1; o < kWave; o <<= 1) {
        uint32_t u = __shfl_up(inc, o, kWave);
        if (lane >= o) inc += u;
    }
    if (lane == kWave - 1) ws[w] = inc;
    __syncthreads();
    uint32_t off = 0, tot = 0;
    for (int k = 0; k < kWavesPerBlock; ++k) {
        if (k < w) off += ws[k];
        tot += ws[k];
    }
    __syncthreads();
    *total = tot;
    return off + inc - v;
}

__device__ __forceinline__ uint64_t block_exclusive(uint64_t v)
{
    __shared__ uint64_t ws[kWavesPerBlock];
    const int lane = threadIdx.x & (kWave - 1), w = threadIdx.x / kWave;
    uint64_t inc = v;
#pragma unroll
    for (int o = 1; o < kWave; o <<= 1) {
        const uint64_t u = __shfl_up(inc, o, kWave);
        if (lane >= o) inc += u;
    }
    if (lane == kWave - 1) ws[w] = inc;
    __syncthreads();
    uint64_t off = 0;
    for (int k = 0; k < w; ++k) off += ws[k];
    return off + inc - v;
}

// LDS accesses of the wave's lanes before and after stay in that order.
__device__ __forceinline__ void wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// ---------------------------------------------------------------- sort
// Several independent arrays (segments) are sorted by one sequence of
// launches: every launch covers the tiles of all segments, a block finding
// its segment by binary search over the segments' first tiles.  Histograms
// are laid out per segment, digit-major: hist[D t0 + d nt + t], D digits; or,
// where no segment has more than kFewTiles, tile by tile: hist[D (t0 + t) + d].
// Then each scatter block adds the tiles' counts itself and there is no scan
// in between, and with one tile a segment no histogram either.
enum { kScanned = 0, kFew = 1, kSingle = 2 };
// Whole builds, us, scanned / not: 512 spheres (1 tile of keys, 4 of
// entries) 90 / 80, 8784 spheres (5 and 11) 157 / 149; 6e4 spheres (30 of
// keys) the same, 172.  At 59 tiles a scatter takes 11.7 us instead of 7.3
// and saves a scan of 2.4 and its launch: no gain.
constexpr int64_t kFewTiles = 32;

// Segment of tile b: the last segment whose first tile is <= b.
__device__ __forceinline__ int seg_of_tile(const SortSeg *__restrict__ sg, int nseg, int64_t b)
{
    int lo = 0, hi = nseg - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (sg[mid].t0 <= b) lo = mid;
        else hi = mid - 1;
    }
    return lo;
}

__global__ __launch_bounds__(kBlock) void k_radix_hist(const SortSeg *__restrict__ sg, int nseg,
                                                      int par, int shift, int bits, int few,
                                                      uint32_t *__restrict__ hist)
{
    __shared__ uint32_t cnt[kMaxDigits];
    cnt[threadIdx.x] = 0;
    cnt[threadIdx.x + kBlock] = 0;
    const uint32_t D = 1u << bits;
    const int j = seg_of_tile(sg, nseg, blockIdx.x);
    const int64_t n = sg[j].n, t0 = sg[j].t0, nt = sg[j].nt;
    const int64_t t = (int64_t)blockIdx.x - t0;
    // pointers read from memory: global-address-space views keep the loads
    // off the flat path (which would also wait on the LDS atomics)
    const gptr<const uint64_t> keys = (gptr<const uint64_t>)(par ? sg[j].k[1] : sg[j].k[0]);
    // all eight loads in flight together (clamped indices: a tile holds at
    // least one key)
    const int64_t base = t * kTile;
    uint64_t kk[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) {
        const int64_t i = base + k * kBlock + threadIdx.x;
        kk[k] = keys[i < n ? i : n - 1];
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < 8; ++k) {
        const int64_t i = base + k * kBlock + threadIdx.x;
        if (i < n) atomicAdd(&cnt[(uint32_t)(kk[k] >> shift) & (D - 1u)], 1u);
    }
    __syncthreads();
    for (uint32_t d = threadIdx.x; d < D; d += kBlock)
        hist[(int64_t)D * t0 + (few ? (int64_t)D * t + d : (int64_t)d * nt + t)] = cnt[d];
}

// Block (j, d): exclusive scan, in place, of digit d's tile counts in
// segment j (tile order), and the digit's total to totals[D j + d].
__global__ __launch_bounds__(kBlock) void k_radix_rowscan(const SortSeg *__restrict__ sg, int bits,
                                                         uint32_t *__restrict__ hist,
                                                         uint32_t *__restrict__ totals)
{
    const int j = (int)(blockIdx.x >> bits), d = (int)(blockIdx.x & ((1u << bits) - 1u));
    const int64_t nt = sg[j].nt;
    uint32_t *row = hist + (sg[j].t0 << bits) + (int64_t)d * nt;
    uint32_t carry = 0;
    for (int64_t base = 0; base < nt; base += 4 * kBlock) {
        const int64_t i0 = base + (int64_t)threadIdx.x * 4;
        uint32_t v[4], sum = 0;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            v[k] = i0 + k < nt ? row[i0 + k] : 0u;
            sum += v[k];
        }
        uint32_t tot;
        uint32_t run = carry + block_exclusive(sum, &tot);
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            if (i0 + k < nt) row[i0 + k] = run;
            run += v[k];
        }
        carry += tot;
    }
    if (threadIdx.x == 0) totals[blockIdx.x] = carry;
}

template <bool kVals, int kMode>
__global__ __launch_bounds__(kBlock) void k_radix_scatter(const SortSeg *__restrict__ sg, int nseg,
                                                         int par, int shift, int bits,
                                                         const uint32_t *__restrict__ off,
                                                         const uint32_t *__restrict__ totals)
{
    constexpr int R = kTile / kBlock, kWaveTile = kTile / kWavesPerBlock;
    __shared__ uint32_t cnt[kWavesPerBlock][kMaxDigits];
    __shared__ uint32_t delta[kMaxDigits];
    __shared__ uint64_t sk[kTile];
    __shared__ uint32_t sv[kVals ? kTile : 1];
    const int tid = (int)threadIdx.x, lane = tid & (kWave - 1), w = tid / kWave;
    const int j = seg_of_tile(sg, nseg, blockIdx.x);
    const int64_t n = sg[j].n, t0 = sg[j].t0, nt = sg[j].nt;
    const int64_t t = (int64_t)blockIdx.x - t0, tile = t * kTile;
    const int m = (int)(n - tile < kTile ? n - tile : kTile);
    const gptr<const uint64_t> kin = (gptr<const uint64_t>)(par ? sg[j].k[1] : sg[j].k[0]) + tile;
    const gptr<uint64_t> kout = (gptr<uint64_t>)(par ? sg[j].k[0] : sg[j].k[1]);
    const gptr<const uint32_t> vin = (gptr<const uint32_t>)(par ? sg[j].v[1] : sg[j].v[0]) + tile;
    const gptr<uint32_t> vout = (gptr<uint32_t>)(par ? sg[j].v[0] : sg[j].v[1]);
    const uint32_t D = 1u << bits, mask = D - 1u;
    // the tile's keys (and values) are loaded up front, all in flight
    // together, 512 consecutive ones a wave (clamped indices: a tile holds at
    // least one key)
    uint64_t kk[R];
    uint32_t vv[R], pre[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int i = w * kWaveTile + r * kWave + lane, ic = i < m ? i : m - 1;
        kk[r] = kin[ic];
        vv[r] = kVals ? vin[ic] : 0u;
    }
    // this thread's two digits: totals in the segment, counts in earlier tiles
    const uint32_t d0 = 2u * (uint32_t)tid;
    uint32_t tot0 = 0, tot1 = 0, off0 = 0, off1 = 0;
    if (kMode == kFew && d0 < D) {
        const uint32_t *c = off + (int64_t)D * t0 + d0;
        const bool two = d0 + 1 < D;
#pragma unroll 8
        for (int64_t q = 0; q < nt; ++q) {
            const uint32_t a = gload(c, q * D), b = two ? gload(c, q * D + 1) : 0u;
            tot0 += a;
            tot1 += b;
            off0 += q < t ? a : 0u;
            off1 += q < t ? b : 0u;
        }
    }
    if (kMode == kScanned && d0 < D) {
        tot0 = totals[(uint64_t)j * D + d0];
        off0 = off[(int64_t)D * t0 + (int64_t)d0 * nt + t];
        if (d0 + 1 < D) {
            tot1 = totals[(uint64_t)j * D + d0 + 1];
            off1 = off[(int64_t)D * t0 + (int64_t)(d0 + 1) * nt + t];
        }
    }
    for (int k = tid; k < kWavesPerBlock * kMaxDigits; k += kBlock) (&cnt[0][0])[k] = 0;
    __syncthreads();
    // rank among the equal digits of the wave's keys: the rounds before (the
    // wave's own counters) and the lanes below
    const uint64_t lt = (1ull << lane) - 1ull;
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const bool valid = w * kWaveTile + r * kWave + lane < m;
        const uint32_t d = (uint32_t)(kk[r] >> shift) & mask;
        uint64_t peers = __ballot(valid);
        for (int b = 0; b < bits; ++b) {
            const bool bit = (d >> b) & 1u;
            const uint64_t bal = __ballot(bit);
            peers &= bit ? bal : ~bal;
        }
        const uint32_t rank = (uint32_t)__popcll(peers & lt);
        const uint32_t before = cnt[w][d];
        wave_sync();
        if (valid && rank == 0) cnt[w][d] = before + (uint32_t)__popcll(peers);
        wave_sync();
        pre[r] = before + rank;
    }
    __syncthreads();
    // where each digit's keys begin in the sorted tile (and each wave's among
    // them), and how far from there they go
    uint32_t c0[kWavesPerBlock], c1[kWavesPerBlock], n0 = 0, n1 = 0;
#pragma unroll
    for (int k = 0; k < kWavesPerBlock; ++k) {
        c0[k] = n0;
        c1[k] = n1;
        n0 += cnt[k][d0];
        n1 += cnt[k][d0 + 1];
    }
    if (kMode == kSingle) {
        tot0 = n0;
        tot1 = n1;
    }
    // one scan for both: tile counts above bit 40, segment totals below
    const uint64_t ex =
        block_exclusive(((uint64_t)(n0 + n1) << 40) | ((uint64_t)tot0 + tot1));
    const uint32_t l0 = (uint32_t)(ex >> 40), l1 = l0 + n0, g0 = (uint32_t)ex;
    delta[d0] = g0 + off0 - l0;
    delta[d0 + 1] = g0 + tot0 + off1 - l1;
#pragma unroll
    for (int k = 0; k < kWavesPerBlock; ++k) {
        cnt[k][d0] = l0 + c0[k];
        cnt[k][d0 + 1] = l1 + c1[k];
    }
    __syncthreads();
    // through LDS in digit order, so that lanes write runs
#pragma unroll
    for (int r = 0; r < R; ++r) {
        if (w * kWaveTile + r * kWave + lane < m) {
            const uint32_t p = cnt[w][(uint32_t)(kk[r] >> shift) & mask] + pre[r];
            sk[p] = kk[r];
            if (kVals) sv[p] = vv[r];
        }
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int i = r * kBlock + tid;
        if (i < m) {
            const uint64_t key = sk[i];
            const uint32_t pos = delta[(uint32_t)(key >> shift) & mask] + (uint32_t)i;
            kout[pos] = key;
            if (kVals) vout[pos] = sv[i];
        }
    }
}

// Segment descriptors travel as kernel arguments (no copy engine, no host
// staging that must outlive the call), kSegChunk per launch.
constexpr int kSegChunk = 32;
struct SegChunk {
    SortSeg s[kSegChunk];
};

__global__ void k_put_segs(SortSeg *__restrict__ dst, SegChunk c, int n)
{
    if ((int)threadIdx.x < n) dst[threadIdx.x] = c.s[threadIdx.x];
}

void launch_put_segs(SortSeg *dst, const SortSeg *src, int nseg, hipStream_t s)
{
    for (int b = 0; b < nseg; b += kSegChunk) {
        SegChunk c;
        const int n = nseg - b < kSegChunk ? nseg - b : kSegChunk;
        for (int q = 0; q < n; ++q) c.s[q] = src[b + q];
        hipLaunchKernelGGL(k_put_segs, dim3(1), dim3(kSegChunk), 0, s, dst + b, c, n);
    }
}

template <bool kVals>
static void launch_scatter(int mode, int64_t ntiles, hipStream_t s, const SortSeg *sg, int nseg,
                           int par, int shift, int bits, const uint32_t *hist,
                           const uint32_t *totals)
{
    const dim3 g((unsigned)ntiles), t(kBlock);
    if (mode == kSingle)
        hipLaunchKernelGGL((k_radix_scatter<kVals, kSingle>), g, t, 0, s, sg, nseg, par, shift,
                           bits, hist, totals);
    else if (mode == kFew)
        hipLaunchKernelGGL((k_radix_scatter<kVals, kFew>), g, t, 0, s, sg, nseg, par, shift, bits,
                           hist, totals);
    else
        hipLaunchKernelGGL((k_radix_scatter<kVals, kScanned>), g, t, 0, s, sg, nseg, par, shift,
                           bits, hist, totals);
}

int radix_sort_segs(const SortSeg *sg, int nseg, int64_t ntiles, int64_t most_tiles, int nbits,
                    bool vals, uint32_t *hist, uint32_t *totals, hipStream_t s)
{
    if (nseg <= 0 || ntiles <= 0) return 0;
    const int mode = most_tiles <= 1 ? kSingle : (most_tiles <= kFewTiles ? kFew : kScanned);
    int par = 0;
    const int passes = sort_passes(nbits);
    for (int q = 0, shift = 0; q < passes; ++q) {
        // as even as can be: the last passes take the odd bits
        const int bits = (nbits - shift) / (passes - q);
        if (mode != kSingle)
            hipLaunchKernelGGL(k_radix_hist, dim3((unsigned)ntiles), dim3(kBlock), 0, s, sg, nseg,
                               par, shift, bits, mode == kFew ? 1 : 0, hist);
        const int64_t some = packings_per_scan(bits);
        for (int64_t j = 0; mode == kScanned && j < nseg; j += some)
            hipLaunchKernelGGL(k_radix_rowscan, dim3((unsigned)std::min(some, nseg - j) << bits),
                               dim3(kBlock), 0, s, sg + j, bits, hist, totals + (j << bits));
        if (vals)
            launch_scatter<true>(mode, ntiles, s, sg, nseg, par, shift, bits, hist, totals);
        else
            launch_scatter<false>(mode, ntiles, s, sg, nseg, par, shift, bits, hist, totals);
        shift += bits;
        par ^= 1;
    }
    return par;
}

// ------------------------------------------------ positions out of list order
// Positions of packing seg from list order back into user order (xu:
// n x 3 row-major), the reverse of k_set_state; orig is a permutation
// of [0, n).
__global__ __launch_bounds__(kBlock) void k_get_positions(const SegPtrs *__restrict__ P,
                                                         const SegState *__restrict__ S, int seg,
                                                         int64_t n, double *__restrict__ xu)
{
    const P4 *Q = S[seg].cur ? P[seg].p[1] : P[seg].p[0];
    const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (i >= n) return;
    const int64_t u = P[seg].orig[i];
    const P4 q = Q[i];
    xu[3 * u] = q.x;
    xu[3 * u + 1] = q.y;
    xu[3 * u + 2] = q.z;
}

void launch_get_positions(const SegPtrs *P, const SegState *S, int seg, int64_t n, double *xu,
                          hipStream_t st)
{
    if (n <= 0) return;
    hipLaunchKernelGGL(k_get_positions, dim3((unsigned)((n + kBlock - 1) / kBlock)), dim3(kBlock),
                       0, st, P, S, seg, n, xu);
}

// ------------------------------------------------------ state and schedules
// Positions handed in by the host: in [-L, 2L) and finite, else *bad; wrapped
// into [0, L) on the axes that have images (bit a of bounded: axis a has
// none).
__global__ __launch_bounds__(kBlock) void k_check_positions(double *__restrict__ x, int64_t n3,
                                                           double L, int bounded,
                                                           uint32_t *__restrict__ bad)
{
    const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (i >= n3) return;
    double v = x[i];
    if (!(v >= -L && v < 2 * L)) {
        *bad = 1u;
        return;
    }
    if ((bounded >> (int)(i % 3)) & 1) return;
    if (v < 0) v += L;
    if (v >= L) v -= L;
    x[i] = v;
}

void launch_check_positions(double *x, int64_t n, double L, int bounded, uint32_t *bad,
                            hipStream_t st)
{
    launch_fill_u32(bad, 1, 0u, st);
    hipLaunchKernelGGL(k_check_positions, dim3((unsigned)((3 * n + kBlock - 1) / kBlock)),
                       dim3(kBlock), 0, st, x, 3 * n, L, bounded, bad);
}

// A state handed in (user order xu): positions into the current buffer, zero
// moments, kappa; the optimiser at its start, no list, on hold.  Nothing if
// *bad.
__global__ __launch_bounds__(kBlock) void k_set_state(const SegPtrs *__restrict__ P,
                                                     SegState *__restrict__ S, int seg, int64_t n,
                                                     const double *__restrict__ xu, double kappa,
                                                     const uint32_t *__restrict__ bad)
{
    if (bad && *bad) return;
    const SegPtrs &p = P[seg];
    SegState *s = S + seg;
    P4 *Q = s->cur ? p.p[1] : p.p[0];
    const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (i < n) {
        const int64_t u = p.orig[i];
        P4 q = Q[i];
        q.x = xu[3 * u];
        q.y = xu[3 * u + 1];
        q.z = xu[3 * u + 2];
        Q[i] = q;
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            p.m[a][i] = 0.0;
            p.v[a][i] = 0.0;
        }
    }
    if (i == 0) {
        s->kappa = kappa;
        s->t = 0;
        s->b1t = 1.0;
        s->b2t = 1.0;
        seg_bias_terms(*s);
        s->mk = 0.0;
        s->vk = 0.0;
        s->it_rung = 0;
        s->rung = 0;
        s->iters = 0;
        s->flags = F_STALE | F_HOLD;
    }
}

void launch_set_state(const SegPtrs *P, SegState *S, int seg, int64_t n, const double *xu,
                      double kappa, const uint32_t *bad, hipStream_t st)
{
    if (n <= 0) return;
    hipLaunchKernelGGL(k_set_state, dim3((unsigned)((n + kBlock - 1) / kBlock)), dim3(kBlock), 0,
                       st, P, S, seg, n, xu, kappa, bad);
}

}  // namespace rcp
