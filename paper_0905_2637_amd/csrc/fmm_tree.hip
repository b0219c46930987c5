// fmm_tree.hip -- tree build on the GPU: domain, z-order leaf keys, stable
// LSD radix sort of the particles by key, leaf ranges, sorted particle arrays.
//
// The uniform quadtree of Section 2.1 needs no pointer structure: box (a, b)
// at level l covers [x0 + a w_l, x0 + (a+1) w_l) x [...], its z-order number
// (Section 5.1) is the bit interleave of (a, b), and the particles of any box
// at any level form one contiguous range of the key-sorted particle array.
//
// Sort: least-significant-digit radix sort with 8-bit digits, ceil(2L/8)
// passes; single plans of few particles and leaves take one counting pass over
// the whole key instead (small sorts, below).  Each digit pass is a per-tile
// digit histogram, an exclusive scan of the digit-major histogram table, and a
// stable scatter in which every wavefront
// ranks its 64 keys by digit with 8 ballots (lanes sharing a digit are found
// by intersecting the ballots of the digit's bits).  Every pass is stable, so
// the final permutation is the unique one with ties in input order, and no
// global atomics are involved: the result is bit-for-bit reproducible.
//
// Several instances: the key of a particle of instance i is (i << 2 L_max) |
// (leaf key at depth L_i << 2 (L_max - L_i)), which orders instances first and
// leaves within each instance, so every instance's particles end up contiguous
// and in their own leaf order.  The input holds the instances one after the
// other, so plans with room for enough particles an instance sort them apart,
// by the leaf bits only (tile_of); the others sort together by the whole key.
//
// The particle record (key, input index, x, y, gamma) travels with the sort,
// so every pass reads and writes whole streams (the scatter writes runs of
// ~16 records per digit and tile) and no random gather follows: the last pass
// writes the sorted arrays the later stages read, plus the mixed-precision
// FP32 leaf-relative record.  The first histogram pass computes the keys.
#include <algorithm>

#include "fmm_device.h"

namespace fmm {
namespace {

// ---------------------------------------------------------------------------
// Domain
// ---------------------------------------------------------------------------

__global__ void __launch_bounds__(256)
k_bbox_partial(int n, const double* __restrict__ x, const double* __restrict__ y, double* __restrict__ part)
{
    double xmin = INFINITY, xmax = -INFINITY, ymin = INFINITY, ymax = -INFINITY;
    for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) {
        const double xv = x[i], yv = y[i];
        // fmin/fmax ignore a NaN operand: NaNs never move the box
        xmin = fmin(xmin, xv); xmax = fmax(xmax, xv);
        ymin = fmin(ymin, yv); ymax = fmax(ymax, yv);
    }
    __shared__ double sh[4][256];
    sh[0][threadIdx.x] = xmin; sh[1][threadIdx.x] = xmax;
    sh[2][threadIdx.x] = ymin; sh[3][threadIdx.x] = ymax;
    __syncthreads();
    for (int s = 128; s > 0; s >>= 1) {
        if (threadIdx.x < s) {
            sh[0][threadIdx.x] = fmin(sh[0][threadIdx.x], sh[0][threadIdx.x + s]);
            sh[1][threadIdx.x] = fmax(sh[1][threadIdx.x], sh[1][threadIdx.x + s]);
            sh[2][threadIdx.x] = fmin(sh[2][threadIdx.x], sh[2][threadIdx.x + s]);
            sh[3][threadIdx.x] = fmax(sh[3][threadIdx.x], sh[3][threadIdx.x + s]);
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        part[4 * blockIdx.x + 0] = sh[0][0];
        part[4 * blockIdx.x + 1] = sh[1][0];
        part[4 * blockIdx.x + 2] = sh[2][0];
        part[4 * blockIdx.x + 3] = sh[3][0];
    }
}

// Bounding square: x0 = min x, y0 = min y, W = the larger extent, 1 if the
// particles span nothing or the extent is not finite.  One workgroup, a
// partial box per thread: 4 us (39 us for one thread walking 256 of them).
__global__ void __launch_bounds__(256) k_bbox_final(int nblk, const double* __restrict__ part, int L, Domain* dom)
{
    double xmin = INFINITY, xmax = -INFINITY, ymin = INFINITY, ymax = -INFINITY;
    for (int b = threadIdx.x; b < nblk; b += 256) {
        xmin = fmin(xmin, part[4 * b + 0]); xmax = fmax(xmax, part[4 * b + 1]);
        ymin = fmin(ymin, part[4 * b + 2]); ymax = fmax(ymax, part[4 * b + 3]);
    }
#pragma unroll
    for (int d = 32; d > 0; d >>= 1) {
        xmin = fmin(xmin, __shfl_xor(xmin, d, 64)); xmax = fmax(xmax, __shfl_xor(xmax, d, 64));
        ymin = fmin(ymin, __shfl_xor(ymin, d, 64)); ymax = fmax(ymax, __shfl_xor(ymax, d, 64));
    }
    __shared__ double sh[4][4];
    if (__lane_id() == 0) {
        double* w = sh[threadIdx.x >> 6];
        w[0] = xmin; w[1] = xmax; w[2] = ymin; w[3] = ymax;
    }
    __syncthreads();
    if (threadIdx.x != 0) return;
    for (int k = 1; k < 4; ++k) {
        xmin = fmin(xmin, sh[k][0]); xmax = fmax(xmax, sh[k][1]);
        ymin = fmin(ymin, sh[k][2]); ymax = fmax(ymax, sh[k][3]);
    }
    double w = xmax - xmin;
    if (ymax - ymin > w) w = ymax - ymin;
    if (!(w > 0.0) || !isfinite(w)) w = 1.0;
    if (!isfinite(xmin)) xmin = 0.0;
    if (!isfinite(ymin)) ymin = 0.0;
    Domain d;
    d.x0 = xmin; d.y0 = ymin; d.W = w;
    d.s = ldexp(1.0, L) / w;
    *dom = d;
}

// ---------------------------------------------------------------------------
// Keys
// ---------------------------------------------------------------------------

// Box index along one axis: t = (v - o) * s, two correctly rounded FP64
// operations (an FMA cannot fuse a product of a difference).  Inside when
// 0 <= t <= 2^L; the far edge belongs to the last box; outside or NaN is
// clamped and flagged.
__device__ __forceinline__ int axis_box(double v, double o, double s, int side, bool& bad)
{
    const double t = (v - o) * s;
    if (!(t >= 0.0 && t <= double(side))) {
        bad = true;
        return t > double(side) ? side - 1 : 0;
    }
    const int b = int(floor(t));
    return b > side - 1 ? side - 1 : b;
}

// ---------------------------------------------------------------------------
// Exclusive scan (of the radix histogram table)
// ---------------------------------------------------------------------------

__device__ __forceinline__ int wave_incl_scan(int v)
{
    const int lane = __lane_id();
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const int t = __shfl_up(v, d, 64);
        if (lane >= d) v += t;
    }
    return v;
}

// Histogram table of a radix pass, digit-major [256][nblk]: one workgroup per
// digit scans its row into out (exclusive; out may be the table itself) and
// writes the digit's total; the scatter turns the 256 totals into the digits'
// starts itself.  A wavefront takes a run of the row, 64 tiles a round, four
// rounds' loads at once.  Latency-bound: 4.7 us a pass on 256 tiles and 14 us
// on 16,384, against 9.5 and 30 us for a two-level scan of the whole table by
// two kernels.
constexpr int kRowScanThreads = 1024;
constexpr int kRowScanWaves = kRowScanThreads / 64;

__global__ void __launch_bounds__(kRowScanThreads)
k_scan_rows(int nblk, const int32_t* in, int32_t* out, int32_t* __restrict__ total)
{
    __shared__ int wsum[kRowScanWaves];
    const int lane = __lane_id(), w = threadIdx.x >> 6;
    const int run_tiles = ((nblk + kRowScanThreads - 1) / kRowScanThreads) * 64;
    const int b0 = min(nblk, w * run_tiles), b1 = min(nblk, b0 + run_tiles);
    const int32_t* src = in + int64_t(blockIdx.x) * nblk;
    int32_t* dst = out + int64_t(blockIdx.x) * nblk;
    int s = 0;
#pragma unroll 8
    for (int b = b0 + lane; b < b1; b += 64) s += src[b];
    s = wave_incl_scan(s);
    if (lane == 63) wsum[w] = s;
    __syncthreads();
    int run = 0, all = 0;
#pragma unroll
    for (int k = 0; k < kRowScanWaves; ++k) {
        run += k < w ? wsum[k] : 0;
        all += wsum[k];
    }
    for (int c = b0; c < b1; c += 256) {
        int v[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int b = c + 64 * r + lane;
            v[r] = b < b1 ? src[b] : 0;
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            if (c + 64 * r >= b1) break;
            const int b = c + 64 * r + lane;
            const int inc = wave_incl_scan(v[r]);
            if (b < b1) dst[b] = run + inc - v[r];
            run += __builtin_amdgcn_readlane(inc, 63);
        }
    }
    if (threadIdx.x == 0) total[blockIdx.x] = all;
}

// ---------------------------------------------------------------------------
// Radix passes
// ---------------------------------------------------------------------------

constexpr int kRadixBins = 256;
constexpr int kRadixTile = 4096;   // keys per workgroup
constexpr int kSmallTiles = 64;
constexpr int kSmallKeyBits = 12;

// Instance owning input particle i (its particles are [part_off, next part_off)).
__device__ __forceinline__ int particle_inst(const Inst* __restrict__ inst, int n_inst, int64_t i)
{
    int lo = 0, hi = n_inst;
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (inst[mid].part_off <= i) lo = mid; else hi = mid;
    }
    return lo;
}

// The tiles of a radix pass.  One instance (or few particles an instance):
// tile b holds the positions from 4096 b, and the instance is the key's
// highest digits.  Segmented (kSegMinPer particles an instance and more): the
// input and every pass keep the instances apart, so their digits are never
// sorted.  Instance q owns the tiles from part_off[q] / 4096 + q on, at least
// as many as it needs; a tile's records go to places of its own instance.
// 512 instances of 2,048 to 65,536 particles, 10 leaf bits: two passes
// instead of three and no search for a particle's instance, tree 760 -> 529 us.
// Apart / by the whole key, evaluations (mixed, P = 8) in us: 64 instances of
// 16,384 445 / 467, 512 of 16,384 2,862 / 3,186; of 6,144 167 / 190 and 681 /
// 787, of 512 114 / 139 and 177 / 195 (mostly empty tiles, and the faster all
// the same).  The line is drawn for the workspace: a tile an instance more
// means a histogram row entry for each digit more, and plans need no more than
// the passes over the whole key did.
constexpr int kSegMinPer = 2 * kRadixTile;

__device__ __forceinline__ int64_t seg_tile(const Inst* __restrict__ inst, int q)
{
    return inst[q].part_off / kRadixTile + q;
}

struct Tile {
    int64_t base;      // first position
    int n;             // positions (0: none)
    int q;             // segmented: its instance,
    int64_t first;     // the instance's first position
    int t0, t1;        // and tiles [t0, t1)
};

template <bool SEG>
__device__ __forceinline__ Tile tile_of(int blk, int n, const Inst* __restrict__ inst, int n_inst, int nblk)
{
    Tile t{};
    if constexpr (!SEG) {
        t.base = int64_t(blk) * kRadixTile;
        t.n = int(max(int64_t(0), min(int64_t(kRadixTile), int64_t(n) - t.base)));
        return t;
    }
    // the last instance whose tiles begin at or before blk, 64 probes a round
    // (they ascend, and instance 0 begins at tile 0: lane 0 always says yes)
    int lo = 0, hi = n_inst;
    while (hi - lo > 1) {
        const int step = (hi - lo + 63) / 64, i = lo + int(__lane_id()) * step;
        const int below = __popcll(__ballot(i < hi && seg_tile(inst, i < hi ? i : lo) <= blk));
        lo += (below - 1) * step;
        hi = min(hi, lo + step);
    }
    t.q = __builtin_amdgcn_readfirstlane(lo);
    t.first = inst[t.q].part_off;
    t.t0 = int(seg_tile(inst, t.q));
    const bool last = t.q + 1 == n_inst;
    t.t1 = last ? nblk : int(seg_tile(inst, t.q + 1));
    const int64_t end = last ? int64_t(n) : inst[t.q + 1].part_off;
    t.base = t.first + int64_t(blk - t.t0) * kRadixTile;
    t.n = int(max(int64_t(0), min(int64_t(kRadixTile), end - t.base)));
    return t;
}

// The histogram kernels and the scatter take the same 4096-key tiles with
// TPB-thread workgroups, 4096 / TPB keys per thread.  Few tiles (small n)
// run with 1024 threads, so that every CU still holds many wavefronts to hide
// the memory latency of these passes; many tiles run with 256 threads and 16
// keys per thread, which measured faster there.

// First pass: the sort key of every particle (kept in input order for
// inspection), the out-of-domain count of the tile (every particle counts
// when the domain is wider than kMaxWidth), and the tile's histogram of the
// lowest digit.
template <int TPB, bool SEG>
__global__ void __launch_bounds__(TPB)
k_rhist_keys(int n, const double* __restrict__ x, const double* __restrict__ y, const Inst* __restrict__ inst,
             int n_inst, int key_shift, int nblk, uint32_t* __restrict__ key, int32_t* __restrict__ hist,
             int32_t* __restrict__ bad_blk, const int32_t* __restrict__ n_dev)
{
    if (n_dev) n = *n_dev;       // batched plans: the call's particle count, from the device
    constexpr int kTileRounds = kRadixTile / TPB;
    __shared__ int h[kRadixBins];
    __shared__ int nbad;
    const Tile tile = tile_of<SEG>(int(blockIdx.x), n, inst, n_inst, nblk);
    if (tile.n == 0) {           // a tile without particles (no input read)
        if (threadIdx.x < kRadixBins) hist[int64_t(threadIdx.x) * nblk + blockIdx.x] = 0;
        if (threadIdx.x == 0) bad_blk[blockIdx.x] = 0;
        return;
    }
    if (threadIdx.x == 0) nbad = 0;
    if (threadIdx.x < kRadixBins) h[threadIdx.x] = 0;
    int mybad = 0;
    // all coordinate loads first, then keys and counting
    double xv[kTileRounds], yv[kTileRounds];
#pragma unroll
    for (int r = 0; r < kTileRounds; ++r) {
        const int li = r * TPB + int(threadIdx.x);
        const int64_t ic = tile.base + (li < tile.n ? li : 0);
        xv[r] = x[ic];
        yv[r] = y[ic];
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < kTileRounds; ++r) {
        const int li = r * TPB + int(threadIdx.x);
        if (li < tile.n) {
            const int64_t i = tile.base + li;
            const int q = SEG ? tile.q : n_inst == 1 ? 0 : particle_inst(inst, n_inst, i);
            const int L = inst[q].L;
            const Domain d = inst[q].dom;
            const int side = 1 << L;
            bool bad = !(d.W <= kMaxWidth);    // a bounding square wider than the limit
            const int a = axis_box(xv[r], d.x0, d.s, side, bad);
            const int b = axis_box(yv[r], d.y0, d.s, side, bad);
            const uint32_t k = (uint32_t(q) << key_shift) | (morton(uint32_t(a), uint32_t(b)) << (key_shift - 2 * L));
            key[i] = k;
            atomicAdd(&h[k & (kRadixBins - 1)], 1);
            mybad += bad ? 1 : 0;
        }
    }
    if (mybad) atomicAdd(&nbad, mybad);
    __syncthreads();
    if (threadIdx.x < kRadixBins) hist[int64_t(threadIdx.x) * nblk + blockIdx.x] = h[threadIdx.x];
    if (threadIdx.x == 0) bad_blk[blockIdx.x] = nbad;
}

// Leaf (a, b), depth and domain of a sort key.
struct KeyLeaf {
    int q, L;
    uint32_t local;      // leaf key at depth L
};

__device__ __forceinline__ KeyLeaf key_leaf(uint32_t k, const Inst* __restrict__ inst, int key_shift)
{
    KeyLeaf r;
    r.q = key_shift >= 32 ? 0 : int(k >> key_shift);
    r.L = inst[r.q].L;
    const uint32_t mask = key_shift >= 32 ? 0xFFFFFFFFu : ((1u << key_shift) - 1u);
    r.local = (k & mask) >> (key_shift - 2 * r.L);
    return r;
}

// Digit histogram of one tile, written digit-major: hist[d * nblk + block].
template <int TPB, bool SEG>
__global__ void __launch_bounds__(TPB)
k_rhist(int n, const uint32_t* __restrict__ kin, int shift, int nblk, int32_t* __restrict__ hist,
        const Inst* __restrict__ inst, int n_inst, const int32_t* __restrict__ n_dev)
{
    if (n_dev) n = *n_dev;
    constexpr int kTileRounds = kRadixTile / TPB;
    __shared__ int h[kRadixBins];
    const Tile tile = tile_of<SEG>(int(blockIdx.x), n, inst, n_inst, nblk);
    if (tile.n == 0) {
        if (threadIdx.x < kRadixBins) hist[int64_t(threadIdx.x) * nblk + blockIdx.x] = 0;
        return;
    }
    if (threadIdx.x < kRadixBins) h[threadIdx.x] = 0;
    uint32_t kv[kTileRounds];
#pragma unroll
    for (int r = 0; r < kTileRounds; ++r) {
        const int li = r * TPB + int(threadIdx.x);
        kv[r] = kin[tile.base + (li < tile.n ? li : 0)];
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < kTileRounds; ++r) {
        if (r * TPB + int(threadIdx.x) < tile.n) atomicAdd(&h[(kv[r] >> shift) & (kRadixBins - 1)], 1);
    }
    __syncthreads();
    if (threadIdx.x < kRadixBins) hist[int64_t(threadIdx.x) * nblk + blockIdx.x] = h[threadIdx.x];
}

// Scatter tiles go to the XCDs in runs of this many from this many tiles on
// (below it the remapping measured no gain).
constexpr int kScatterXcdRun = 16;
constexpr int kScatterXcdMinTiles = 512;

// Where a sorted record goes, and what it carries.
struct Records {
    uint32_t* k;
    uint32_t* idx;
    double* x;
    double* y;
    double* g;
};

// Stable scatter of one tile, in two phases.
// Phase A ranks the tile: wavefront w owns input positions
// [4096 w / W, 4096 (w + 1) / W) of the W = TPB / 64 wavefronts and takes
// them 64 per round, in input order (loaded up front for 4 rounds, round by
// round for 16, which measured faster for each); it ranks
// its lanes by digit with 8 ballots, and the per-wavefront digit counts order
// the wavefronts, giving every record its position in the digit-sorted tile.
// Phase B stages each array through LDS in that order, so that consecutive
// threads write consecutive addresses of each digit's run (offs[d * nblk +
// block] is where the tile's run starts among digit d, total[d] the count of
// digit d; where segmented, both less those of the instances before): whole
// cache lines instead of scattered 8-byte writes.  hist == nullptr: the table
// was scanned in place, and a tile's count is the difference to the next entry
// (sorts apart and the 3D form have no room for a second table within the
// workspace that they always had; three passes of 16M records take 801 us with
// it, 803 to 819 without).
// iin == nullptr means the identity (first pass).  pk != nullptr (last pass,
// mixed precision) also writes the FP32 leaf-relative record
// (x - c, y - c) / w_L, gamma of the leaf centre c.
template <int TPB, bool SEG>
__global__ void __launch_bounds__(TPB)
k_rscatter(int n, const uint32_t* __restrict__ kin, const uint32_t* __restrict__ iin,
           const double* __restrict__ xin, const double* __restrict__ yin, const double* __restrict__ gin,
           int shift, int nblk, const int32_t* __restrict__ hist, const int32_t* __restrict__ offs,
           const int32_t* __restrict__ total, Records out, float4* __restrict__ pk, const Inst* __restrict__ inst, int n_inst,
           int key_shift, const int32_t* __restrict__ n_dev)
{
    if (n_dev) n = *n_dev;
    constexpr int kScatterThreads = TPB;
    constexpr int kScatterWaves = TPB / 64;
    constexpr int kPerThread = kRadixTile / TPB;
    constexpr bool kUpFront = kPerThread <= 4;
    __shared__ int gbase[kRadixBins];      // global start of this tile's run of digit d
    __shared__ int tstart[kRadixBins];     // start of digit d in the sorted tile
    __shared__ int wsum[2][4];
    __shared__ int whist[kScatterWaves][kRadixBins];   // per wavefront: records of digit d so far
    __shared__ uint32_t sk[kRadixTile];
    __shared__ double sv[kRadixTile];
    const int tid = threadIdx.x, lane = int(__lane_id()), w = tid >> 6;
    // large sorts: runs of kScatterXcdRun consecutive tiles per XCD, so that
    // the runs of one digit that neighbouring tiles write side by side meet
    // in one L2 (whole lines go out) instead of leaving partial lines in two
    const int blk = nblk >= kScatterXcdMinTiles ? xcd_runs(int(blockIdx.x), nblk, kScatterXcdRun) : int(blockIdx.x);
    const Tile seg = tile_of<SEG>(blk, n, inst, n_inst, nblk);
    const int64_t tile = seg.base;
    const int tile_n = seg.n;
    if (tile_n == 0) return;
    constexpr int kWaveKeys = kRadixTile / kScatterWaves;

    // the tile's histogram (one digit per thread of the first 256) scanned
    // into tstart, the digits' totals into their starts in the output; the
    // first four wavefronts hold both
    int hv = 0, hinc = 0, go = 0, tv = 0, tinc = 0;
    if (tid < kRadixBins) {
        const int32_t* row = offs + int64_t(tid) * nblk;
        go = row[blk];
        tv = total[tid];
        if (hist) {
            hv = hist[int64_t(tid) * nblk + blk];
        } else {
            const int next = row[min(blk + 1, nblk - 1)];
            hv = (blk + 1 < nblk ? next : tv) - go;
        }
        if constexpr (SEG) {     // the instance's share of the row
            const int before = row[seg.t0];
            tv = (seg.t1 < nblk ? row[seg.t1] : tv) - before;
            go -= before;
        }
        hinc = wave_incl_scan(hv);
        tinc = wave_incl_scan(tv);
        if (lane == 63) {
            wsum[0][w] = hinc;
            wsum[1][w] = tinc;
        }
    }
#pragma unroll
    for (int e = tid; e < kScatterWaves * kRadixBins; e += kScatterThreads) (&whist[0][0])[e] = 0;

    uint32_t kr[kPerThread], vr[kPerThread];
    double xr[kPerThread], yr[kPerThread], gr[kPerThread];
    bool valid[kPerThread];
    auto load = [&](int r) {
        const int li = w * kWaveKeys + r * 64 + lane;
        valid[r] = li < tile_n;
        const int64_t i = tile + (valid[r] ? li : 0);
        kr[r] = valid[r] ? kin[i] : 0u;
        vr[r] = iin ? iin[i] : uint32_t(i);
        xr[r] = xin[i];
        yr[r] = yin[i];
        gr[r] = gin ? gin[i] : 0.0;
    };
    if constexpr (kUpFront) {
#pragma unroll
        for (int r = 0; r < kPerThread; ++r) load(r);
    }
    __syncthreads();
    if (tid < kRadixBins) {
        int before = 0, start = 0;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            before += q < w ? wsum[0][q] : 0;
            start += q < w ? wsum[1][q] : 0;
        }
        tstart[tid] = before + hinc - hv;
        gbase[tid] = int(seg.first) + start + tinc - tv + go;
    }

    // rank within the wavefront, round after round (input order): equal
    // digits of one round are told apart by 8 ballots, earlier rounds by the
    // wavefront's running count of the digit
    const uint64_t lt_mask = (uint64_t(1) << lane) - 1;
    int lpos[kPerThread], dig[kPerThread];
#pragma unroll
    for (int r = 0; r < kPerThread; ++r) {
        if constexpr (!kUpFront) load(r);
        const int d = int((kr[r] >> shift) & (kRadixBins - 1));
        uint64_t same = __ballot(valid[r]);
#pragma unroll
        for (int b = 0; b < 8; ++b) {
            const bool bit = (d >> b) & 1;
            const uint64_t bb = __ballot(bit);
            same &= bit ? bb : ~bb;
        }
        const int rank = __popcll(same & lt_mask);
        const int before = whist[w][d];
        __builtin_amdgcn_wave_barrier();
        if (valid[r] && rank == 0) whist[w][d] = before + __popcll(same);
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        lpos[r] = valid[r] ? before + rank : -1;
        dig[r] = d;
    }
    __syncthreads();
    // exclusive prefix over the wavefronts, per digit
    if (tid < kRadixBins) {
        int acc = 0;
#pragma unroll
        for (int q = 0; q < kScatterWaves; ++q) {
            const int t = whist[q][tid];
            whist[q][tid] = acc;
            acc += t;
        }
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < kPerThread; ++r)
        if (lpos[r] >= 0) lpos[r] += tstart[dig[r]] + whist[w][dig[r]];

    // ---- phase B: stage each array in sorted order, write whole runs ----
    int dst[kPerThread];
    uint32_t ks_[kPerThread];
#pragma unroll
    for (int r = 0; r < kPerThread; ++r)
        if (lpos[r] >= 0) sk[lpos[r]] = kr[r];
    __syncthreads();
#pragma unroll
    for (int r = 0; r < kPerThread; ++r) {
        const int j = r * kScatterThreads + tid;
        dst[r] = -1;
        if (j < tile_n) {
            const uint32_t k = sk[j];
            const int d = int((k >> shift) & (kRadixBins - 1));
            ks_[r] = k;
            dst[r] = gbase[d] + (j - tstart[d]);
            out.k[dst[r]] = k;
        }
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < kPerThread; ++r)
        if (lpos[r] >= 0) sk[lpos[r]] = vr[r];
    __syncthreads();
#pragma unroll
    for (int r = 0; r < kPerThread; ++r)
        if (dst[r] >= 0) out.idx[dst[r]] = sk[r * kScatterThreads + tid];

    double xs_[kPerThread], ys_[kPerThread];
#pragma unroll
    for (int r = 0; r < kPerThread; ++r)
        if (lpos[r] >= 0) sv[lpos[r]] = xr[r];
    __syncthreads();
#pragma unroll
    for (int r = 0; r < kPerThread; ++r) {
        xs_[r] = sv[r * kScatterThreads + tid];
        if (dst[r] >= 0) out.x[dst[r]] = xs_[r];
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < kPerThread; ++r)
        if (lpos[r] >= 0) sv[lpos[r]] = yr[r];
    __syncthreads();
#pragma unroll
    for (int r = 0; r < kPerThread; ++r) {
        ys_[r] = sv[r * kScatterThreads + tid];
        if (dst[r] >= 0) out.y[dst[r]] = ys_[r];
    }
    if (!out.g) return;                    // point records (target points) carry no circulation
    __syncthreads();
#pragma unroll
    for (int r = 0; r < kPerThread; ++r)
        if (lpos[r] >= 0) sv[lpos[r]] = gr[r];
    __syncthreads();
#pragma unroll
    for (int r = 0; r < kPerThread; ++r) {
        if (dst[r] < 0) continue;
        const double gv = sv[r * kScatterThreads + tid];
        out.g[dst[r]] = gv;
        if (pk) {
            const KeyLeaf kl = key_leaf(ks_[r], inst, key_shift);
            const Domain dm = inst[kl.q].dom;
            const double wl = ldexp(dm.W, -kl.L);
            const double cx = dm.x0 + (double(morton_x(kl.local)) + 0.5) * wl;
            const double cy = dm.y0 + (double(morton_y(kl.local)) + 0.5) * wl;
            pk[dst[r]] = make_float4(float((xs_[r] - cx) * dm.s), float((ys_[r] - cy) * dm.s), float(gv), 0.0f);
        }
    }
}

// ---------------------------------------------------------------------------
// Small sorts: one pass over the whole key
// ---------------------------------------------------------------------------
//
// Up to kSmallTiles tiles of a single instance with at most kSmallKeyBits key
// bits sort by one counting pass over the whole key: a tile's counts per leaf
// are 16-bit (a tile has 4096 keys), one row per tile, and every scatter
// workgroup adds up the rows itself, which also gives the leaf ranges.  At
// these sizes a kernel costs its latency: three kernels (one for a single
// tile) replace four per digit and the leaf-range kernel.  Tree of 4,096 particles, 8 key bits: 11
// us instead of 23; 100,000, 10 bits: 22 instead of 56; 200,000, 12 bits: 32
// instead of 60.
constexpr int kSmallThreads = 1024;
constexpr int kSmallWaves = kSmallThreads / 64;
constexpr int kSmallPer = kRadixTile / kSmallThreads;

// Sort key of a particle of the only instance: its leaf.
__device__ __forceinline__ uint32_t leaf_key(double x, double y, const Domain& d, int L, bool& bad)
{
    const int side = 1 << L;
    bad = !(d.W <= kMaxWidth);             // a bounding square wider than the limit
    const int a = axis_box(x, d.x0, d.s, side, bad);
    const int b = axis_box(y, d.y0, d.s, side, bad);
    return morton(uint32_t(a), uint32_t(b));
}

// FP32 record (x - c, y - c) / w_L, gamma of leaf k's centre c.
__device__ __forceinline__ float4 leaf_record(uint32_t k, double x, double y, double g, const Domain& d, int L)
{
    const double w = ldexp(d.W, -L);
    const double cx = d.x0 + (double(morton_x(k)) + 0.5) * w;
    const double cy = d.y0 + (double(morton_y(k)) + 0.5) * w;
    return make_float4(float((x - cx) * d.s), float((y - cy) * d.s), float(g), 0.0f);
}

// Keys, out-of-domain count and leaf counts of every tile.
__global__ void __launch_bounds__(kSmallThreads)
k_small_keys(int n, const double* __restrict__ x, const double* __restrict__ y, const Inst* __restrict__ inst,
             uint32_t* __restrict__ key, uint16_t* __restrict__ hist, int32_t* __restrict__ bad_blk)
{
    extern __shared__ int h[];
    __shared__ int nbad;
    const int L = inst[0].L, bins = 1 << (2 * L), tid = threadIdx.x;
    const Domain d = inst[0].dom;
    const int base = int(blockIdx.x) * kRadixTile;
    if (tid == 0) nbad = 0;
    for (int e = tid; e < bins; e += kSmallThreads) h[e] = 0;
    double xv[kSmallPer], yv[kSmallPer];
#pragma unroll
    for (int r = 0; r < kSmallPer; ++r) {
        const int i = min(n - 1, base + r * kSmallThreads + tid);
        xv[r] = x[i];
        yv[r] = y[i];
    }
    __syncthreads();
    int mybad = 0;
#pragma unroll
    for (int r = 0; r < kSmallPer; ++r) {
        const int i = base + r * kSmallThreads + tid;
        if (i < n) {
            bool bad;
            const uint32_t k = leaf_key(xv[r], yv[r], d, L, bad);
            key[i] = k;
            atomicAdd(&h[k], 1);
            mybad += bad ? 1 : 0;
        }
    }
    if (mybad) atomicAdd(&nbad, mybad);
    __syncthreads();
    uint16_t* row = hist + int64_t(blockIdx.x) * bins;
    for (int e = tid; e < bins; e += kSmallThreads) row[e] = uint16_t(h[e]);
    if (tid == 0) bad_blk[blockIdx.x] = nbad;
}

// Leaf counts in LDS: 16 bits, kVec leaves a thread.
constexpr int kSmallVec = 4;
struct alignas(8) Counts {
    uint16_t v[kSmallVec];
};

// Places of one tile's records, and the leaf ranges (the first workgroup).
// Ranks as k_rscatter: wavefront w owns the input positions [256 w, 256 (w +
// 1)) of the tile, 64 a round.  ONE (the only tile): the keys are computed
// here, and the records are sorted in LDS and written out; else only the
// permutation is, and k_small_gather moves the records (scattered eight-byte
// stores take a cycle of the CU each: five a record from these few workgroups
// cost more than the whole sort).
template <bool ONE>
__global__ void __launch_bounds__(kSmallThreads)
k_small_sort(int n, int nblk, const uint32_t* __restrict__ kin, const double* __restrict__ x,
             const double* __restrict__ y, const double* __restrict__ g, const Inst* __restrict__ inst,
             uint32_t* __restrict__ key, const uint16_t* __restrict__ hist, int32_t* __restrict__ bad_blk, Records out,
             float4* __restrict__ pk, int32_t* __restrict__ leaf_start)
{
    extern __shared__ __attribute__((aligned(16))) char smem[];
    const int L = inst[0].L, bits = 2 * L, bins = 1 << bits;                 // at least kSmallVec
    int* gbase = reinterpret_cast<int*>(smem);                               // [bins] the tile's place in every leaf
    uint16_t* whist = reinterpret_cast<uint16_t*>(gbase + bins);             // [kSmallWaves][bins]
    __shared__ int wsum[kSmallWaves];
    __shared__ int nbad;
    const int tid = threadIdx.x, lane = int(__lane_id()), w = tid >> 6, blk = int(blockIdx.x);
    const Domain dm = inst[0].dom;
    const int base = blk * kRadixTile;
    const int first = base + w * (kRadixTile / kSmallWaves) + lane;          // the thread's records: first + 64 r
    if (ONE && tid == 0) nbad = 0;

    uint32_t kr[kSmallPer];
    double xr[kSmallPer], yr[kSmallPer], gr[kSmallPer];
    int mybad = 0;
#pragma unroll
    for (int r = 0; r < kSmallPer; ++r) {
        const int ic = min(first + 64 * r, n - 1);
        if constexpr (ONE) {
            xr[r] = x[ic];
            yr[r] = y[ic];
            gr[r] = g ? g[ic] : 0.0;
        } else {
            kr[r] = kin[ic];
        }
    }
    // this tile's part of every leaf: the counts of the tiles before it and of
    // all tiles, kSmallVec leaves a thread (at most 4096 leaves)
    const int d0 = tid * kSmallVec;
    const bool mine = d0 < bins;
    int pre[kSmallVec] = {0, 0, 0, 0}, tot[kSmallVec] = {0, 0, 0, 0};
    if constexpr (!ONE) {
        if (mine) {
            const Counts* row = reinterpret_cast<const Counts*>(hist + d0);
            const int stride = bins / kSmallVec;
#pragma unroll 8
            for (int b = 0; b < nblk; ++b) {
                const Counts c = row[int64_t(b) * stride];
#pragma unroll
                for (int q = 0; q < kSmallVec; ++q) {
                    tot[q] += c.v[q];
                    pre[q] += b < blk ? c.v[q] : 0;
                }
            }
        }
    }
    Counts* wz = reinterpret_cast<Counts*>(whist);
    for (int e = tid; e < kSmallWaves * bins / kSmallVec; e += kSmallThreads) wz[e] = Counts{{0, 0, 0, 0}};
    if constexpr (ONE) {
#pragma unroll
        for (int r = 0; r < kSmallPer; ++r) {
            bool bad;
            kr[r] = leaf_key(xr[r], yr[r], dm, L, bad);
            if (first + 64 * r < n) {
                key[first + 64 * r] = kr[r];
                mybad += bad ? 1 : 0;
            }
        }
    }
    __syncthreads();

    const uint64_t lt_mask = (uint64_t(1) << lane) - 1;
    int lpos[kSmallPer];
    uint16_t* wh = whist + w * bins;
#pragma unroll
    for (int r = 0; r < kSmallPer; ++r) {
        const bool valid = first + 64 * r < n;
        const uint32_t d = kr[r];
        uint64_t same = __ballot(valid);
        for (int b = 0; b < bits; ++b) {
            const bool bit = (d >> b) & 1;
            const uint64_t bb = __ballot(bit);
            same &= bit ? bb : ~bb;
        }
        const int rank = __popcll(same & lt_mask);
        const int before = wh[d];
        __builtin_amdgcn_wave_barrier();
        if (valid && rank == 0) wh[d] = uint16_t(before + __popcll(same));
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        lpos[r] = valid ? before + rank : -1;
    }
    if (ONE && mybad) atomicAdd(&nbad, mybad);
    __syncthreads();

    // the wavefronts' counts to their places within the tile's part of a leaf
    int s = 0;
    if (mine) {
        int acc[kSmallVec] = {0, 0, 0, 0};
#pragma unroll
        for (int k = 0; k < kSmallWaves; ++k) {
            Counts* c = reinterpret_cast<Counts*>(whist + k * bins + d0);
            const Counts t = *c;
            Counts o;
#pragma unroll
            for (int q = 0; q < kSmallVec; ++q) {
                o.v[q] = uint16_t(acc[q]);
                acc[q] += t.v[q];
            }
            *c = o;
        }
#pragma unroll
        for (int q = 0; q < kSmallVec; ++q) {
            if constexpr (ONE) tot[q] = acc[q];
            s += tot[q];
        }
    }
    const int inc = wave_incl_scan(s);
    if (lane == 63) wsum[w] = inc;
    __syncthreads();
    int start = inc - s;
#pragma unroll
    for (int k = 0; k < kSmallWaves; ++k) start += k < w ? wsum[k] : 0;
    if (mine) {
#pragma unroll
        for (int q = 0; q < kSmallVec; ++q) {
            gbase[d0 + q] = start + pre[q];
            if (blk == 0) leaf_start[d0 + q] = start;
            start += tot[q];
        }
        if (blk == 0 && d0 + kSmallVec == bins) leaf_start[bins] = start;
    }
    if (ONE && tid == 0) bad_blk[0] = nbad;
    __syncthreads();

#pragma unroll
    for (int r = 0; r < kSmallPer; ++r) {
        if (lpos[r] < 0) continue;
        lpos[r] += gbase[kr[r]] + wh[kr[r]];
        if constexpr (!ONE) out.idx[lpos[r]] = uint32_t(first + 64 * r);
    }
    if constexpr (!ONE) return;
    __syncthreads();
    // the sorted tile in LDS, over the counts
    double* sx = reinterpret_cast<double*>(smem);
    double* sy = sx + kRadixTile;
    double* sg = sy + kRadixTile;
    uint32_t* sk = reinterpret_cast<uint32_t*>(sg + kRadixTile);
    uint32_t* si = sk + kRadixTile;
#pragma unroll
    for (int r = 0; r < kSmallPer; ++r) {
        if (lpos[r] < 0) continue;
        sx[lpos[r]] = xr[r];
        sy[lpos[r]] = yr[r];
        sg[lpos[r]] = gr[r];
        sk[lpos[r]] = kr[r];
        si[lpos[r]] = uint32_t(first + 64 * r);
    }
    __syncthreads();
    for (int j = tid; j < n; j += kSmallThreads) {
        const uint32_t k = sk[j];
        out.k[j] = k;
        out.idx[j] = si[j];
        out.x[j] = sx[j];
        out.y[j] = sy[j];
        if (out.g) out.g[j] = sg[j];
        if (pk) pk[j] = leaf_record(k, sx[j], sy[j], sg[j], dm, L);
    }
}

// The records of a small sort to their places.
__global__ void __launch_bounds__(256)
k_small_gather(int n, const uint32_t* __restrict__ perm, const uint32_t* __restrict__ key, const double* __restrict__ x,
               const double* __restrict__ y, const double* __restrict__ g, const Inst* __restrict__ inst, Records out,
               float4* __restrict__ pk)
{
    const int j = int(blockIdx.x) * 256 + int(threadIdx.x);
    if (j >= n) return;
    const uint32_t i = perm[j], k = key[i];
    const double xv = x[i], yv = y[i], gv = g ? g[i] : 0.0;
    out.k[j] = k;
    out.x[j] = xv;
    out.y[j] = yv;
    if (out.g) out.g[j] = gv;
    if (pk) pk[j] = leaf_record(k, xv, yv, gv, inst[0].dom, inst[0].L);
}

// Depth 0: one leaf, nothing to sort.
__global__ void __launch_bounds__(256)
k_copy_one_leaf(int n, const double* __restrict__ x, const double* __restrict__ y, const double* __restrict__ g,
                Records out, float4* __restrict__ pk, const Inst* __restrict__ inst)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const double xv = x[i], yv = y[i], gv = g ? g[i] : 0.0;
    out.k[i] = 0u;
    out.idx[i] = uint32_t(i);
    out.x[i] = xv;
    out.y[i] = yv;
    if (out.g) out.g[i] = gv;
    if (pk) {
        const Domain dm = inst[0].dom;
        const double cx = dm.x0 + 0.5 * dm.W, cy = dm.y0 + 0.5 * dm.W;
        pk[i] = make_float4(float((xv - cx) * dm.s), float((yv - cy) * dm.s), float(gv), 0.0f);
    }
}

// Sorted position -> global leaf_start entry (instance segment + leaf).
__device__ __forceinline__ int64_t leaf_entry(uint32_t k, const Inst* __restrict__ inst, int key_shift)
{
    const KeyLeaf kl = key_leaf(k, inst, key_shift);
    return inst[kl.q].leaf_off + int64_t(kl.local);
}

// leaf_start[e] = first sorted position whose leaf entry is >= e, for every
// entry e < entries: position i owns the entries in (entry(i-1), entry(i)].
// Each instance's segment ends with one extra entry, which thereby receives
// the first position of the next instance (its particle count end).
// A workgroup takes kBoundsRounds x 256 consecutive positions, 256 per round
// (coalesced); all its key loads are issued before any range is written,
// and a single-instance plan reads its instance record once.
// A gap of more than kBoundsGap empty leaves is filled by the whole wavefront:
// one thread's loop over a clustered tree's gaps took longer than all the key
// loads (2^22 particles of 16 clusters, 2^18 leaves: 53 us, 14 here); below, a
// round of the wavefront for each of its gaps costs more than the loops side by
// side.  Tree stage with the line at 2 / 8 / 32 / never, us: 2^20 of 16
// clusters, 2^20 leaves 151 / 126 / 122 / 701; uniform, 2^20 leaves: 2^20
// particles 102 / 94 / 94 / 94, 2^18 123 / 90 / 85 / 86, 2^16 142 / 124 / 98 /
// 117, 4,096 249 / 249 / 256 / 819.
constexpr int kBoundsRounds = 16;
constexpr int kBoundsGap = 32;

__global__ void __launch_bounds__(256)
k_bounds(int n, int64_t entries, const uint32_t* __restrict__ ks, const Inst* __restrict__ inst, int n_inst,
         int key_shift, int32_t* __restrict__ leaf_start, const int32_t* __restrict__ n_dev)
{
    if (n_dev) {                 // batched plans: particles and leaf entries of the call
        n = n_dev[0];
        entries = n_dev[1];
    }
    const int64_t base = int64_t(blockIdx.x) * (256 * kBoundsRounds) + threadIdx.x;
    uint32_t kp[kBoundsRounds], kc[kBoundsRounds];      // keys of i - 1 and i
#pragma unroll
    for (int r = 0; r < kBoundsRounds; ++r) {
        const int64_t i = base + int64_t(r) * 256;
        const int64_t ip = i - 1 < 0 ? 0 : (i - 1 < n ? i - 1 : (n > 0 ? n - 1 : 0));
        const int64_t ic = i < n ? i : (n > 0 ? n - 1 : 0);
        kp[r] = ks[ip];
        kc[r] = ks[ic];
    }
    const int L0 = inst[0].L;
    const int64_t off0 = inst[0].leaf_off;
    auto entry = [&](uint32_t k) -> int64_t {
        if (n_inst == 1) return off0 + int64_t(k >> (key_shift - 2 * L0));
        return leaf_entry(k, inst, key_shift);
    };
#pragma unroll
    for (int r = 0; r < kBoundsRounds; ++r) {
        const int64_t i = base + int64_t(r) * 256;
        if (__ballot(i <= n) == 0) break;
        int lo = 0, hi = -1;                                // entries fit 31 bits
        if (i <= n) {
            lo = i == 0 ? 0 : int(entry(kp[r])) + 1;
            hi = i == n ? int(entries) - 1 : int(entry(kc[r]));
        }
        const bool wide = hi - lo >= kBoundsGap;
        if (!wide)
            for (int e = lo; e <= hi; ++e) leaf_start[e] = int32_t(i);
        for (uint64_t m = __ballot(wide); m != 0; m &= m - 1) {
            const int l = __builtin_ctzll(m);
            const int first = __builtin_amdgcn_readlane(lo, l), last = __builtin_amdgcn_readlane(hi, l);
            const int32_t at = int32_t(i) + (l - int(__lane_id()));
            for (int e = first + int(__lane_id()); e <= last; e += 64) leaf_start[e] = at;
        }
    }
}

inline unsigned blocks_for(int64_t n, int bs) { return unsigned((n + bs - 1) / bs); }

}  // namespace

hipError_t launch_domain(const Buffers& b, int n, const double* x, const double* y, int L, hipStream_t st,
                         int m, const double* tx, const double* ty)
{
    hipLaunchKernelGGL(k_bbox_partial, dim3(kBBoxBlocks), dim3(256), 0, st, n, x, y, b.bbox);
    if (m > 0)   // target points: their partial boxes follow the particles'
        hipLaunchKernelGGL(k_bbox_partial, dim3(kBBoxBlocks), dim3(256), 0, st, m, tx, ty, b.bbox + 4 * kBBoxBlocks);
    hipLaunchKernelGGL(k_bbox_final, dim3(1), dim3(256), 0, st, m > 0 ? 2 * kBBoxBlocks : kBBoxBlocks, b.bbox, L,
                       &b.inst[0].dom);
    return hipGetLastError();
}

int radix_passes(int key_bits) { return (key_bits + 7) / 8; }

int64_t radix_blocks(int64_t n) { return (n + kRadixTile - 1) / kRadixTile; }

bool small_sort(int64_t n_cap, int n_inst, int key_bits)
{
    return n_inst == 1 && key_bits >= 1 && key_bits <= kSmallKeyBits && radix_blocks(n_cap) <= kSmallTiles;
}

bool seg_sort(int64_t n_cap, int n_inst, int key_shift)
{
    return n_inst > 1 && key_shift > 0 && n_cap >= int64_t(kSegMinPer) * n_inst;
}

int64_t sort_tiles(int64_t n, int n_inst, bool segmented)
{
    return segmented ? n / kRadixTile + n_inst : radix_blocks(n);
}

namespace {

// Radix passes of at most this many tiles use the 1024-thread kernels: tree of
// 10M particles 580 us with them, 637 with 256 threads; 16M 991 and 1042; 32M
// 2002 and 1978; 64M 4316 and 3914.  (Batched evaluation of 9.7M, 2,880
// tiles: 3181 and 3260 us.)
constexpr int kWideTilesMax = 4096;

void scan_table(const Buffers& b, int nblk, hipStream_t st)
{
    hipLaunchKernelGGL(k_scan_rows, dim3(kRadixBins), dim3(kRowScanThreads), 0, st, nblk, b.hist, b.hist_scan,
                       b.scan_part);
}

}  // namespace

namespace {

// The passes of a sort over the keys' lowest 8 npass bits.  first: whether the
// first digit's histogram is there.
void radix_sort(const Buffers& b, int n, int nblk, bool wide, bool seg, int npass, bool first, const uint32_t* kin,
                const double* xin, const double* yin, const double* gin, const Records& fin, const Records& tmp,
                float4* pk, hipStream_t st, const int32_t* n_dev)
{
    const int threads = wide ? 1024 : 256;
    const auto count = seg ? (wide ? k_rhist<1024, true> : k_rhist<256, true>)
                           : (wide ? k_rhist<1024, false> : k_rhist<256, false>);
    const auto scatter = seg ? (wide ? k_rscatter<1024, true> : k_rscatter<256, true>)
                             : (wide ? k_rscatter<1024, false> : k_rscatter<256, false>);
    const int32_t* counts = b.hist_scan == b.hist ? nullptr : b.hist;
    const uint32_t* iin = nullptr;
    // the last pass writes the final arrays, the others alternate with tmp
    for (int pass = 0; pass < npass; ++pass) {
        const Records& out = ((npass - 1 - pass) & 1) ? tmp : fin;
        const int shift = 8 * pass;
        if (pass > 0 || !first)
            hipLaunchKernelGGL(count, dim3(nblk), dim3(threads), 0, st, n, kin, shift, nblk, b.hist, b.inst, b.n_inst,
                               n_dev);
        scan_table(b, nblk, st);
        hipLaunchKernelGGL(scatter, dim3(nblk), dim3(threads), 0, st, n, kin, iin, xin, yin, gin, shift, nblk, counts,
                           b.hist_scan, b.scan_part, out, pass == npass - 1 ? pk : nullptr, b.inst, b.n_inst,
                           b.key_shift, n_dev);
        kin = out.k;
        iin = out.idx;
        xin = out.x;
        yin = out.y;
        gin = out.g;
    }
}

// Keys, sort and leaf ranges of one point set: records (key, index, x, y and,
// when g != nullptr, gamma), final arrays in fin, leaf ranges in leaf_start.
void sort_points(const Buffers& b, int n, const double* x, const double* y, const double* g, uint32_t* key,
                 int32_t* bad_blk, const Records& fin, float4* pk, int32_t* leaf_start, int key_bits,
                 int64_t leaf_entries, hipStream_t st, const int32_t* n_dev = nullptr)
{
    const int nblk = int(sort_tiles(n, b.n_inst, b.seg_sort));
    if (b.small_sort) {
        // 16-bit counts of the wavefronts and a place per leaf in LDS, then (one tile) its records
        const size_t bins = size_t(1) << key_bits;
        const size_t counts_lds = bins * (sizeof(int) + kSmallWaves * sizeof(uint16_t));
        // the tiles' counts lie over the temporaries of the passes, 24 bytes a point for 2 bytes a
        // leaf and tile (at least 4097 points in two tiles and more)
        static_assert(24 * kRadixTile >= 2 * (sizeof(uint16_t) << kSmallKeyBits), "the counts fit");
        uint16_t* counts = reinterpret_cast<uint16_t*>(b.ktmp);
        if (nblk == 1) {
            const size_t lds = std::max(counts_lds, size_t(kRadixTile) * (3 * sizeof(double) + 2 * sizeof(uint32_t)));
            hipLaunchKernelGGL(k_small_sort<true>, dim3(1), dim3(kSmallThreads), lds, st, n, nblk, nullptr, x, y, g,
                               b.inst, key, counts, bad_blk, fin, pk, leaf_start);
        } else {
            hipLaunchKernelGGL(k_small_keys, dim3(nblk), dim3(kSmallThreads), bins * sizeof(int), st, n, x, y, b.inst,
                               key, counts, bad_blk);
            hipLaunchKernelGGL(k_small_sort<false>, dim3(nblk), dim3(kSmallThreads), counts_lds, st, n, nblk, key, x, y,
                               g, b.inst, key, counts, bad_blk, fin, pk, leaf_start);
            hipLaunchKernelGGL(k_small_gather, dim3(blocks_for(n, 256)), dim3(256), 0, st, n, fin.idx, key, x, y, g,
                               b.inst, fin, pk);
        }
        return;
    }
    const Records tmp{b.ktmp, b.itmp, b.xt, b.yt, g ? b.gt : nullptr};
    const bool wide = nblk <= kWideTilesMax;
    const int threads = wide ? 1024 : 256;
    const auto keys = b.seg_sort ? (wide ? k_rhist_keys<1024, true> : k_rhist_keys<256, true>)
                                 : (wide ? k_rhist_keys<1024, false> : k_rhist_keys<256, false>);
    hipLaunchKernelGGL(keys, dim3(nblk), dim3(threads), 0, st, n, x, y, b.inst, b.n_inst, b.key_shift, nblk, key, b.hist,
                       bad_blk, n_dev);
    const int npass = radix_passes(b.seg_sort ? b.key_shift : key_bits);
    if (npass == 0)
        hipLaunchKernelGGL(k_copy_one_leaf, dim3(blocks_for(n, 256)), dim3(256), 0, st, n, x, y, g, fin, pk, b.inst);
    else
        radix_sort(b, n, nblk, wide, b.seg_sort, npass, true, key, x, y, g, fin, tmp, pk, st, n_dev);
    hipLaunchKernelGGL(k_bounds, dim3(blocks_for(int64_t(n) + 1, 256 * kBoundsRounds)), dim3(256), 0, st, n,
                       leaf_entries, fin.k, b.inst, b.n_inst, b.key_shift, leaf_start, n_dev);
}

}  // namespace

hipError_t launch_tree(const Buffers& b, int n, const double* x, const double* y, const double* g,
                       int key_bits, int64_t leaf_entries, bool mixed, hipStream_t st, const int32_t* n_dev)
{
    const Records fin{b.ksorted, b.perm, b.xs, b.ys, b.gs};
    sort_points(b, n, x, y, g, b.key, b.bad_blk, fin, mixed ? b.pk : nullptr, b.leaf_start, key_bits,
                leaf_entries, st, n_dev);
    return hipGetLastError();
}

hipError_t launch_tree_points(const Buffers& b, int m, const double* tx, const double* ty, int key_bits,
                              int64_t leaf_entries, hipStream_t st)
{
    const Records fin{b.tks, b.tperm, b.txs, b.tys, nullptr};
    sort_points(b, m, tx, ty, nullptr, b.tkey, b.tbad, fin, nullptr, b.tleaf_start, key_bits, leaf_entries, st);
    return hipGetLastError();
}

hipError_t launch_sort_keys(const Buffers& b, int n, const uint32_t* key, const double* x, const double* y,
                            const double* g, uint32_t* ks, uint32_t* perm, double* xs, double* ys, double* gs,
                            int key_bits, hipStream_t st)
{
    const int npass = radix_passes(key_bits);
    if (n <= 0 || npass <= 0) return hipErrorInvalidValue;
    const int nblk = int(radix_blocks(n));
    const Records fin{ks, perm, xs, ys, gs};
    const Records tmp{b.ktmp, b.itmp, b.xt, b.yt, b.gt};
    radix_sort(b, n, nblk, nblk <= kWideTilesMax, false, npass, false, key, x, y, g, fin, tmp, nullptr, st, nullptr);
    return hipGetLastError();
}

}  // namespace fmm
