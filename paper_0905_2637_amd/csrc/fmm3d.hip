// fmm3d.hip -- the 3D form of the method on the GPU: the same tree and
// sweeps on a uniform octree (Section 8: the method carries over to 3D with
// a new kernel, its series expansions and translation operators), for the
// Laplace kernel 1/r with Cartesian Taylor expansions of total degree <= p.
//
// Per particle: potential phi(x) = sum_j q_j / |x - y_j| and its gradient,
// pairs at zero distance left out.  With w the box width of a level, c a
// box centre and everything scaled to unit boxes:
//   moments  Ms_k = sum_j q_j prod_i ((c_i - y_ji) / w)^k_i / k_i!
//   M2M      Ms_k(parent) = sum_{m <= k} Ms_m(child) 2^-|m| prod_i (s_i / 4)^(k_i - m_i) / (k_i - m_i)!,
//            s_i = +1 / -1 as the parent centre lies above / below the child's
//   M2L      Ls_n(t) = sum_k Ms_k(s) D_(k+n)((t - s) / w),   D_m = d^m (1/r)
//   L2L      Ls_n(child) += 2^-(1+|n|) sum_{m >= n} Ls_m(parent) 4^-(|m|-|n|) prod_i t_i^(m_i-n_i) / (m_i-n_i)!,
//            t_i = +1 / -1 as the child centre lies above / below the parent's
//   L2P      phi(x) = (1/w) sum_n Ls_n u^n / n!,  d phi / dx_i = (1/w^2) sum_n Ls_n u^(n-e_i) / (n-e_i)!,
//            u = (x - c) / w
// The scaling makes the M2L data level-independent: one operator D_(k+n) per
// integer offset of the interaction lists, from degree 5 on for non-negative x
// and y offsets only (the M2L reaches the others by reflection).
//
// Only the terms of degree <= 1 in z are kept: see fmm3d_internal.h.
//
// Layout: octree boxes in Morton order per level (children of box k at
// 8k .. 8k+7), levels one after another; coefficients of a box contiguous in
// the stored order of fmm3d_internal.h.  Tree build: keys, the library's
// stable radix sort (records carry x, y, q; z is gathered after), leaf
// ranges by binary search.
#include <type_traits>
#include <utility>

#include "fmm3d_internal.h"

namespace fmm3 {
namespace {

constexpr int kTpb = 256;
typedef double f64x4 __attribute__((ext_vector_type(4)));

__device__ inline uint32_t morton3(uint32_t a, uint32_t b, uint32_t c)
{
    uint32_t k = 0;
#pragma unroll
    for (int i = 0; i < 10; ++i)
        k |= (((a >> i) & 1u) << (3 * i)) | (((b >> i) & 1u) << (3 * i + 1)) | (((c >> i) & 1u) << (3 * i + 2));
    return k;
}

__device__ inline void unmorton3(uint32_t k, int& a, int& b, int& c)
{
    a = b = c = 0;
#pragma unroll
    for (int i = 0; i < 10; ++i) {
        a |= int((k >> (3 * i)) & 1u) << i;
        b |= int((k >> (3 * i + 1)) & 1u) << i;
        c |= int((k >> (3 * i + 2)) & 1u) << i;
    }
}

// multi-index (a, b, c) of graded position t
__device__ inline void decode3(int t, int& a, int& b, int& c)
{
    int d = 0;
    while (tet3(d + 1) <= t) ++d;
    int r = t - tet3(d), s = 0;
    while (tri3(s + 1) <= r) ++s;
    c = r - tri3(s);
    b = s - c;
    a = d - s;
}

// 4^-j / j! for j <= kP3Max (the shift coefficients of M2M and L2L)
__constant__ double kQuarterFact3[kP3Max + 1] = {1.0, 0.25, 1.0 / 32, 1.0 / 384, 1.0 / 6144, 1.0 / 122880,
                                                 1.0 / 2949120, 1.0 / 82575360, 1.0 / 2642411520.0,
                                                 1.0 / 95126814720.0};
// C(q, i), q <= 4
__constant__ double kBinom3[5][5] = {{1, 0, 0, 0, 0}, {1, 1, 0, 0, 0}, {1, 2, 1, 0, 0}, {1, 3, 3, 1, 0}, {1, 4, 6, 4, 1}};

__device__ inline double quarter_f(int j) { return kQuarterFact3[j]; }

// the lanes of a wavefront see each other's LDS writes past this point
__device__ __forceinline__ void wave_sync3()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// The kept moment (a, b, r), r <= 1, of a full set: every moment with c = 2 q
// + r folded into those of c = r, D_(.., c) = (-1)^q sum_i C(q, i) D_(a + 2 i,
// b + 2 (q - i), r).  full(a, b, c) reads the full set.
template <typename F>
__device__ inline double fold_moment3(int a, int b, int r, F&& full)
{
    double s = 0.0;
    for (int i = 0; 2 * i <= a; ++i)
        for (int j = 0; 2 * j <= b; ++j) {
            const double v = kBinom3[i + j][i] * full(a - 2 * i, b - 2 * j, 2 * (i + j) + r);
            s += ((i + j) & 1) ? -v : v;
        }
    return s;
}

// ---- tree -------------------------------------------------------------------

__global__ void __launch_bounds__(kTpb)
k3_keys(int n, const double* __restrict__ x, const double* __restrict__ y, const double* __restrict__ z, Geo3 g,
        uint32_t* __restrict__ key, unsigned long long* __restrict__ nbad)
{
    const int i = int(blockIdx.x) * kTpb + int(threadIdx.x);
    bool bad = false;
    if (i < n) {
        const double side = ldexp(1.0, g.L);
        const double u[3] = {(x[i] - g.x0) / g.W * side, (y[i] - g.y0) / g.W * side, (z[i] - g.z0) / g.W * side};
        uint32_t cc[3] = {0u, 0u, 0u};
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            if (!(u[d] >= 0.0 && u[d] < side)) bad = true;
            else cc[d] = uint32_t(floor(u[d]));
        }
        key[i] = bad ? (1u << (3 * g.L)) : morton3(cc[0], cc[1], cc[2]);
    }
    const uint64_t m = __ballot(bad);
    if (__lane_id() == 0 && m) atomicAdd(nbad, (unsigned long long)__popcll(m));
}

__global__ void __launch_bounds__(kTpb)
k3_gather(int n, const uint32_t* __restrict__ perm, const double* __restrict__ z, double* __restrict__ zs)
{
    const int i = int(blockIdx.x) * kTpb + int(threadIdx.x);
    if (i < n) zs[i] = z[perm[i]];
}

// leaf_start[b] = first sorted position with key >= b, b = 0 .. 8^L
__global__ void __launch_bounds__(kTpb)
k3_leaf_start(int64_t nleaf, int n, const uint32_t* __restrict__ ks, int32_t* __restrict__ leaf_start)
{
    const int64_t b = int64_t(blockIdx.x) * kTpb + threadIdx.x;
    if (b > nleaf) return;
    int lo = 0, hi = n;
    while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (int64_t(ks[mid]) < b) lo = mid + 1;
        else hi = mid;
    }
    leaf_start[b] = lo;
}

__global__ void k3_clear(unsigned long long* nbad) { *nbad = 0ull; }

// ---- upward sweep -------------------------------------------------------------

// P2M: one wavefront per leaf.  Ms_(a,b,c) = sum_j (X_a Y_b)_j (q Z_c)_j with
// X_a = ((c_x - x_j) / w)^a / a! and so on is a product over the particles of
// a (P+1)(P+2)/2 x 4 and a 4 x (P+1) matrix per four of them, so it runs on
// v_mfma_f64_16x16x4, 16 pairs (a, b) to a tile; 32 particles at a time leave
// their powers in LDS, one lane each.  The full set then folds into the kept
// terms.  2^20 particles in 32,768 leaves (p = 6): 59 us, against 288 us for
// one thread per coefficient raising its own powers.
template <int P>
__global__ void __launch_bounds__(kTpb, 2)
k3_p2m(Geo3 g, const int32_t* __restrict__ ls, const double* __restrict__ xs, const double* __restrict__ ys,
       const double* __restrict__ zs, const double* __restrict__ qs, const int32_t* __restrict__ term,
       double* __restrict__ me)
{
    constexpr int NP = (P + 1) * (P + 2) / 2, RT = (NP + 15) / 16, C = 32, S = C + 4, KP = stored3(P);
    constexpr int kShare = 3 * (P + 1) * S > NP * (P + 1) ? 3 * (P + 1) * S : NP * (P + 1);
    __shared__ double sh[kTpb / 64][kShare];
    const int lane = int(threadIdx.x) & 63;
    const int wave = __builtin_amdgcn_readfirstlane(int(threadIdx.x) >> 6);
    const uint32_t leaf = blockIdx.x * (kTpb / 64) + uint32_t(wave);
    if (leaf >= (1u << (3 * g.L))) return;
    int la, lb, lc;
    unmorton3(leaf, la, lb, lc);
    const double w = ldexp(g.W, -g.L), inv_w = 1.0 / w;
    const double cx = g.x0 + (la + 0.5) * w, cy = g.y0 + (lb + 0.5) * w, cz = g.z0 + (lc + 0.5) * w;
    double* sX = sh[wave];
    double* sY = sX + (P + 1) * S;
    double* sZ = sY + (P + 1) * S;
    const int col = lane & 15, k = lane >> 4;
    int ra[RT], rb[RT];      // (a, b) of the lane's row of every tile; rows past the last repeat (0, 0)
#pragma unroll
    for (int t = 0; t < RT; ++t) {
        int i = 16 * t + col, a = 0;
        while (a < P && i > P - a) i -= P - a + 1, ++a;
        const bool in = 16 * t + col < NP;
        ra[t] = (in ? a : 0) * S;
        rb[t] = (in ? i : 0) * S;
    }
    const int rc = (col <= P ? col : 0) * S;
    f64x4 acc[RT];
#pragma unroll
    for (int t = 0; t < RT; ++t) acc[t] = f64x4{0.0, 0.0, 0.0, 0.0};
    const int j1 = ls[leaf + 1];
    for (int jb = ls[leaf]; jb < j1; jb += C) {
        const int j = jb + lane;
        if (lane < C) {
            const bool in = j < j1;
            const double ux = in ? (cx - xs[j]) * inv_w : 0.0, uy = in ? (cy - ys[j]) * inv_w : 0.0;
            const double uz = in ? (cz - zs[j]) * inv_w : 0.0;
            double px = 1.0, py = 1.0, pz = in ? qs[j] : 0.0;
#pragma unroll
            for (int e = 0; e <= P; ++e) {
                sX[e * S + lane] = px;
                sY[e * S + lane] = py;
                sZ[e * S + lane] = pz;
                const double re = 1.0 / double(e + 1);
                px *= ux * re;
                py *= uy * re;
                pz *= uz * re;
            }
        }
        wave_sync3();
        const int steps = (min(C, j1 - jb) + 3) / 4;
        for (int st = 0; st < steps; ++st) {
            const int j4 = 4 * st + k;
            const double zv = sZ[rc + j4];
#pragma unroll
            for (int t = 0; t < RT; ++t)
                acc[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(sX[ra[t] + j4] * sY[rb[t] + j4], zv, acc[t], 0, 0, 0);
        }
        wave_sync3();
    }
    // lane l holds rows l / 16 + 4 r, column (c) l mod 16
    double* sT = sh[wave];
    if (col <= P)
#pragma unroll
        for (int t = 0; t < RT; ++t)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int row = 16 * t + k + 4 * r;
                if (row < NP) sT[row * (P + 1) + col] = acc[t][r];
            }
    wave_sync3();
    double* dst = me + (lvl_off3(g.L) + leaf) * KP;
    for (int e = lane; e < KP; e += 64) {
        const int id = term[e];
        dst[e] = id < 0 ? 0.0 : fold_moment3(id & 255, (id >> 8) & 255, id >> 16, [&](int a, int b, int c) {
            return sT[(a * (P + 1) - a * (a - 1) / 2 + b) * (P + 1) + c];
        });
    }
}

// parents at level l from their eight children; one workgroup per parent, one
// thread per term of the full set, which then folds into the kept terms (depth
// 5, p = 6: 32 us for the three launches, 81 us without the folding)
template <int P>
__global__ void __launch_bounds__(kTpb)
k3_m2m(int l, const int32_t* __restrict__ term, double* __restrict__ me)
{
    constexpr int KP = stored3(P), T = tet3(P + 1), Q = P + 1, D = 2 * Q * Q;
    __shared__ double sm[8][D];        // [signs][r][a][b]
    __shared__ double sT[T];
    __shared__ double sc[Q][Q];        // 2^-i 4^-(a-i) / (a-i)!
    const uint32_t par = blockIdx.x;
    const int t = int(threadIdx.x), nt = int(blockDim.x);
    const double* src = me + (lvl_off3(l + 1) + int64_t(8) * par) * KP;
    for (int e = t; e < Q * Q; e += nt) {
        const int a = e / Q, i = e % Q;
        sc[a][i] = i <= a ? ldexp(quarter_f(a - i), -i) : 0.0;
    }
    // A child's sign in the shift depends only on the parities of k - m: for
    // every term m the eight children's moments are replaced by their signed
    // sums H_pi(m) = sum_ch (-1)^popcount(ch & pi) Ms_m(ch) (a Walsh-Hadamard
    // transform over the children), so that each output sums over m once
    // instead of eight times.
    for (int e = t; e < KP; e += nt) {
        const int id = term[e];
        if (id < 0) continue;
        double v[8];
#pragma unroll
        for (int ch = 0; ch < 8; ++ch) v[ch] = src[ch * KP + e];
#pragma unroll
        for (int h = 1; h < 8; h <<= 1)
#pragma unroll
            for (int ch = 0; ch < 8; ++ch)
                if (!(ch & h)) {
                    const double u = v[ch], w = v[ch | h];
                    v[ch] = u + w;
                    v[ch | h] = u - w;
                }
        const int at = ((id >> 16) * Q + (id & 255)) * Q + ((id >> 8) & 255);
#pragma unroll
        for (int pi = 0; pi < 8; ++pi) sm[pi][at] = v[pi];
    }
    __syncthreads();
    for (int e = t; e < T; e += nt) {
        int a, b, c;
        decode3(e, a, b, c);
        double acc = 0.0;
        for (int k = 0; k <= c && k <= 1; ++k)
            for (int i = 0; i <= a; ++i) {
                const int pi = ((a - i) & 1) | (((c - k) & 1) << 2);
                double row = 0.0;
                for (int j = 0; j <= b; ++j) row += sm[pi | (((b - j) & 1) << 1)][(k * Q + i) * Q + j] * sc[b][j];
                acc += row * (sc[a][i] * sc[c][k]);
            }
        sT[e] = acc;
    }
    __syncthreads();
    double* dst = me + (lvl_off3(l) + par) * KP;
    for (int e = t; e < KP; e += nt) {
        const int id = term[e];
        dst[e] = id < 0 ? 0.0 : fold_moment3(id & 255, (id >> 8) & 255, id >> 16,
                                             [&](int a, int b, int c) { return sT[pos3(a, b, c)]; });
    }
}

// ---- downward sweep -------------------------------------------------------------

// The moments of levels 2 .. L as the M2L reads them (grid3): box-major in,
// term-major out, 64 grid points of one child position a workgroup.
struct Levels3 {
    int n_levels;
    int blk_begin[kDepth3Max + 1];   // first workgroup of each level from 2 up, then the total
};

// level of workgroup `blk`, which becomes its number within the level
__device__ __forceinline__ int level_of3(const Levels3& lv, int& blk)
{
    int li = 0;
    while (li + 1 < lv.n_levels && blk >= lv.blk_begin[li + 1]) ++li;
    blk -= lv.blk_begin[li];
    return 2 + li;
}

// x spread to every third bit (x < 2^10)
__device__ __forceinline__ uint32_t spread3(uint32_t x)
{
    x = (x | (x << 16)) & 0x030000FFu;
    x = (x | (x << 8)) & 0x0300F00Fu;
    x = (x | (x << 4)) & 0x030C30C3u;
    x = (x | (x << 2)) & 0x09249249u;
    return x;
}

template <int P>
__global__ void __launch_bounds__(kTpb)
k3_spread(Levels3 lv, const double* __restrict__ me, double* __restrict__ mt)
{
    constexpr int KP = stored3(P), S = KP + 1;
    __shared__ double sh[64 * S];
    __shared__ int sbox[64];
    int blk = int(blockIdx.x);
    const int l = level_of3(lv, blk);
    constexpr int B = fold3(P) ? 1 : 0;      // border
    const int cls = blk & 7, h = 1 << (l - 1), s = h + 2 * B, n = int(grid3(P, l)), i0 = (blk >> 3) * 64;
    const int t = int(threadIdx.x);
    if (t < 64) {
        const int i = i0 + t, x = i % s - B, y = i / s % s - B, z = i / (s * s) - B;
        const bool in = x >= 0 && y >= 0 && z >= 0 && x < h && y < h && z < h;
        sbox[t] = in ? int((spread3(uint32_t(x)) | spread3(uint32_t(y)) << 1 | spread3(uint32_t(z)) << 2) << 3 | uint32_t(cls))
                     : -1;
    }
    __syncthreads();
    const double* src = me + lvl_off3(l) * KP;
    for (int e = t; e < 64 * KP; e += kTpb) {
        const int i = e / KP, k = e % KP, box = sbox[i];
        sh[i * S + k] = box >= 0 ? src[int64_t(box) * KP + k] : 0.0;
    }
    __syncthreads();
    double* dst = mt + (grid_off3(P, l) + cls * int64_t(n)) * KP + i0;
    const int i = t & 63;
    if (i0 + i < n)
        for (int k = t >> 6; k < KP; k += kTpb / 64) dst[int64_t(k) * n + i] = sh[i * S + k];
}

// M2L of all levels in one launch, on v_mfma_f64_16x16x4: rows are output
// terms, columns 16 target boxes, four source terms a step.  A workgroup
// holds 32 boxes of one child position (two column groups), consecutive in
// the grid of their parents, so all of them walk the same offsets; its four
// wavefronts take every fourth operator and their sums meet in LDS.
// Folded (fold3): D_(k+n) at (sx ox, sy oy, oz) is sx^(a_k + a_n) sy^(b_k +
// b_n) times that at (ox, oy, oz), so one operator serves up to four sources
// v(sx, sy): with their signed sums h_pi = sum sx^pi_x sy^pi_y v(sx, sy), the
// outputs of parity class pi_n take h_(pi_n xor pi_k) from the source terms
// of class pi_k: 84 operators instead of 189 offsets, the rows of each class
// in tiles of their own.
// The operators come in lane order, the sources as 16 neighbouring boxes of
// one term (k3_spread; read box-major the four lane groups touched 64 lines a
// load, and the L1 lookups were the limit: 640 us), both straight from memory
// with the next step's in flight (a matrix instruction takes 64 cycles of its
// SIMD, more than the loads that feed it).
// 2^20 charges, depth 5, p = 6: 479 us, against 7,569 us for the full 84 x 84
// terms on the vector units, bound by an LDS read per multiply-add; the
// matrix cores alone need 270 us for the folded operators.

// f(integral_constant 0), ..., f(integral_constant N - 1)
template <typename F, int... I>
__device__ __forceinline__ void each3(std::integer_sequence<int, I...>, F&& f)
{
    (f(std::integral_constant<int, I>{}), ...);
}

__host__ __device__ constexpr int step_class3(int p, int st)
{
    int cl = 0;
    while (4 * st >= class_base3(p, cl + 1)) ++cl;
    return cl;
}

// Output classes [C0, C1) of CG column groups of 16 targets, the operators
// dealt to W wavefronts; sum: room for [W / 2][their tiles * CG][64].
template <int P, int CG, int W, int C0, int C1>
__device__ __forceinline__ void m2l3(const Levels3& lv, const double* __restrict__ mt, double* __restrict__ le,
                                     const double* __restrict__ op, f64x4* __restrict__ sum)
{
    constexpr bool FOLD = fold3(P);
    constexpr int KP = stored3(P), NS = steps3(P), RT = tiles3(P);
    constexpr int I0 = tile_base3(P, C0), NT = tile_base3(P, C1) - I0;       // its tiles
    constexpr int NV = FOLD ? 4 : 1;
    const int lane = int(threadIdx.x) & 63;
    const int wave = __builtin_amdgcn_readfirstlane(int(threadIdx.x) >> 6);
    const int G = int(gridDim.x);
    int blk = fmm::xcd_runs(int(blockIdx.x), G, G / fmm::kXcds);
    const int l = level_of3(lv, blk);
    const int cls = blk & 7, cx = cls & 1, cy = (cls >> 1) & 1, cz = cls >> 2;
    const int h = 1 << (l - 1), n = h * h * h, s = FOLD ? h + 2 : h, n_grid = int(grid3(P, l));
    const int col = lane & 15, grp = lane >> 4;
    const double* grid = mt + grid_off3(P, l) * KP;
    // not folded: terms of the last step; the lane's term of it and of the others
    constexpr int REST = KP - 4 * (NS - 1);
    const int grp_last = min(grp, REST - 1);
    // the lane's targets: places in the grid (folded: plus the lane's term of a step), and (not
    // folded) which of the 27 parents around the target's lie in the cube
    uint32_t box[CG], at[CG], inside[CG];
    bool valid[CG];
#pragma unroll
    for (int c = 0; c < CG; ++c) {
        const int t = (blk >> 3) * (16 * CG) + 16 * c + col;
        valid[c] = t < n;
        const int i = valid[c] ? t : 0, x = i & (h - 1), y = (i >> (l - 1)) & (h - 1), z = i >> (2 * (l - 1));
        box[c] = (spread3(uint32_t(x)) | spread3(uint32_t(y)) << 1 | spread3(uint32_t(z)) << 2) << 3 | uint32_t(cls);
        if constexpr (FOLD) {
            at[c] = uint32_t(grp * n_grid + ((z + 1) * s + y + 1) * s + x + 1);
            inside[c] = 0;
        } else {
            at[c] = uint32_t(i);
            const auto spread = [h](uint32_t m, int k, int by) {       // m at -1, 0, 1 along an axis
                return (k > 0 ? m : 0u) | m << by | (k < h - 1 ? m << 2 * by : 0u);
            };
            inside[c] = spread(spread(spread(1u, x, 1), y, 3), z, 9);
        }
    }
    f64x4 acc[NT][CG];
#pragma unroll
    for (int i = 0; i < NT; ++i)
#pragma unroll
        for (int c = 0; c < CG; ++c) acc[i][c] = f64x4{0.0, 0.0, 0.0, 0.0};

    // The wavefront's next operator from number u on (every W-th of those
    // outside the near block; NU: none left) and its sources.  Source (sx, sy)
    // of a box at offset (ox, oy, oz) is the box minus (sx ox, sy oy, oz): its
    // child position and the shift of its parent are the same for all boxes.
    constexpr int NU = FOLD ? 96 : 216;
    struct Operator {
        const double* a;          // the operator (folded: the lane's values)
        const double* src[NV];    // the sources' terms, from the place of the box; null: not in the list
        uint32_t at[CG];          // not folded: the lane's sources' places
    };
    int turn = 0;
    const auto next = [&](int u, Operator& o) {
        int ox = 0, oy = 0, oz = 0;
        for (; u < NU; ++u) {
            ox = FOLD ? (u & 3) : cx - 3 + u % 6;
            oy = FOLD ? ((u >> 2) & 3) : cy - 3 + (u / 6) % 6;
            oz = cz - 3 + (FOLD ? (u >> 4) : u / 36);
            if (abs(ox) <= 1 && abs(oy) <= 1 && abs(oz) <= 1) continue;
            if ((turn++ & (W - 1)) == wave) break;
        }
        if (u >= NU) return NU;   // the last operator's values are read once more, not used
        o.a = op + int64_t(operator3(P, ox, oy, oz)) * operator_size3(P) + (FOLD ? lane : 0);
        if constexpr (!FOLD) {
            const int sx = cx - ox, sy = cy - oy, sz = cz - oz, dx = sx >> 1, dy = sy >> 1, dz = sz >> 1;
            const int bit = (dz + 1) * 9 + (dy + 1) * 3 + dx + 1, to = (dz * h + dy) * h + dx;
            o.src[0] = grid + int64_t((sx & 1) | (sy & 1) << 1 | (sz & 1) << 2) * KP * n_grid;
#pragma unroll
            for (int c = 0; c < CG; ++c) o.at[c] = (inside[c] >> bit) & 1u ? at[c] + uint32_t(to) : uint32_t(n);
            return u;
        }
#pragma unroll
        for (int v = 0; v < NV; ++v) {
            const int sx = cx - ((v & 1) ? -ox : ox), sy = cy - ((v & 2) ? -oy : oy), sz = cz - oz;
            // folded: offsets lie in [c - 3, c + 2], so 3 occurs with one sign only, and 0 once
            const bool in = ((v & 1) ? ox != 0 && (ox != 3 || cx == 0) : ox != 3 || cx == 1) &&
                            ((v & 2) ? oy != 0 && (oy != 3 || cy == 0) : oy != 3 || cy == 1);
            const int pos = (sx & 1) | (sy & 1) << 1 | (sz & 1) << 2;
            o.src[v] = in ? grid + int64_t(pos) * KP * n_grid + ((sz >> 1) * s + (sy >> 1)) * s + (sx >> 1) : nullptr;
        }
        return u;
    };
    // one step's operator values and source terms
    struct Step {
        double a[NT];
        double v[CG][NV];
    };
    const auto load = [&](int st, const Operator& o, Step& k) {
        if constexpr (!FOLD) {
            // a step's terms past the last are zero times any operator value
            const bool last = st + 1 == NS;
            const int term = last ? grp_last : grp;
            const double* src = o.src[0] + int64_t(4 * st) * n_grid;
#pragma unroll
            for (int c = 0; c < CG; ++c) {
                const double v = src[uint32_t(term * n_grid) + o.at[c]];
                k.v[c][0] = last && grp >= REST ? 0.0 : v;
            }
#pragma unroll
            for (int i = 0; i < NT; ++i) k.a[i] = o.a[(4 * st + term) * KP + min(16 * i + col, KP - 1)];
            return;
        }
#pragma unroll
        for (int v = 0; v < NV; ++v) {
            if (o.src[v]) {
                const double* src = o.src[v] + int64_t(4 * st) * n_grid;
#pragma unroll
                for (int c = 0; c < CG; ++c) k.v[c][v] = src[at[c]];
            } else {
#pragma unroll
                for (int c = 0; c < CG; ++c) k.v[c][v] = 0.0;
            }
        }
#pragma unroll
        for (int i = 0; i < NT; ++i) k.a[i] = o.a[(st * RT + I0 + i) * 64];
    };
    // the signed sums of the sources' terms, then their products
    const auto multiply = [&](auto stc, const Step& k) {
        constexpr int cl = step_class3(P, decltype(stc)::value);
        double hs[CG][NV];
#pragma unroll
        for (int c = 0; c < CG; ++c) {
            const auto& v = k.v[c];
            if constexpr (FOLD) {
                const double s0 = v[0] + v[1], d0 = v[0] - v[1], s1 = v[2] + v[3], d1 = v[2] - v[3];
                hs[c][0] = s0 + s1;
                hs[c][1] = d0 + d1;
                hs[c][2] = s0 - s1;
                hs[c][3] = d0 - d1;
            } else {
                hs[c][0] = v[0];
            }
        }
        each3(std::make_integer_sequence<int, C1 - C0>{}, [&](auto cnc) {
            constexpr int cn = C0 + decltype(cnc)::value, i0 = tile_base3(P, cn) - I0;
            each3(std::make_integer_sequence<int, class_tiles3(P, cn)>{}, [&](auto ic) {
                constexpr int i = i0 + decltype(ic)::value;
#pragma unroll
                for (int c = 0; c < CG; ++c)
                    acc[i][c] = __builtin_amdgcn_mfma_f64_16x16x4f64(k.a[i], hs[c][FOLD ? (cn ^ cl) : 0], acc[i][c], 0,
                                                                     0, 0);
            });
        });
    };
    // a step's loads are in flight during the products of the one before,
    // across operators too; the barrier keeps the scheduler from sinking them
    // to their uses
    Operator cur;
    Step now, ahead;
    int u = next(0, cur);
    if (u < NU) load(0, cur, now);
    while (u < NU) {
        each3(std::make_integer_sequence<int, NS>{}, [&](auto stc) {
            constexpr int st = decltype(stc)::value;
            if constexpr (st + 1 == NS) u = next(u + 1, cur);
            load((st + 1) % NS, cur, ahead);
            __builtin_amdgcn_sched_barrier(0);
            multiply(stc, now);
            __builtin_amdgcn_sched_barrier(0);
            now = ahead;
        });
    }
    // the wavefronts' sums, pairwise
#pragma unroll
    for (int d = W / 2; d >= 1; d >>= 1) {
        if (wave >= d && wave < 2 * d)
#pragma unroll
            for (int i = 0; i < NT; ++i)
#pragma unroll
                for (int c = 0; c < CG; ++c) sum[((wave - d) * NT * CG + i * CG + c) * 64 + lane] = acc[i][c];
        __syncthreads();
        if (wave < d)
#pragma unroll
            for (int i = 0; i < NT; ++i)
#pragma unroll
                for (int c = 0; c < CG; ++c) acc[i][c] += sum[(wave * NT * CG + i * CG + c) * 64 + lane];
        __syncthreads();
    }
    if (wave != 0) return;
    // lane l holds rows l / 16 + 4 r of column l mod 16
#pragma unroll
    for (int c = 0; c < CG; ++c) {
        if (!valid[c]) continue;
        double* dst = le + (lvl_off3(l) + box[c]) * KP;
        each3(std::make_integer_sequence<int, C1 - C0>{}, [&](auto clc) {
            constexpr int cl = C0 + decltype(clc)::value, i0 = tile_base3(P, cl) - I0;
            each3(std::make_integer_sequence<int, class_tiles3(P, cl)>{}, [&](auto ic) {
                constexpr int i = i0 + decltype(ic)::value;
                const f64x4 s = acc[i][c];
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int row = 16 * (i - i0) + grp + 4 * r;
                    if (row < class_size3(P, cl)) dst[class_base3(P, cl) + row] = s[r];
                }
            });
        });
    }
}

constexpr int kM2lGroups3 = 2;
constexpr int kM2lWaves3 = 4;

// wavefronts per SIMD the registers allow
__host__ __device__ constexpr int m2l_occupancy3(int p) { return tiles3(p) <= 4 ? 3 : 2; }

// many targets: every output class of 32 targets a workgroup
template <int P>
__global__ void __launch_bounds__(64 * kM2lWaves3, m2l_occupancy3(P))
k3_m2l(Levels3 lv, const double* __restrict__ mt, double* __restrict__ le, const double* __restrict__ op)
{
    __shared__ f64x4 sum[kM2lWaves3 / 2 * tiles3(P) * kM2lGroups3 * 64];
    m2l3<P, kM2lGroups3, kM2lWaves3, 0, classes3(P)>(lv, mt, le, op, sum);
}

// few targets (one wavefront's chain of operators would set the time): one
// output class of 16 targets a workgroup, blockIdx.y the class, eight
// wavefronts
constexpr int kM2lWavesFew3 = 8;

template <int P>
__global__ void __launch_bounds__(64 * kM2lWavesFew3, 2)
k3_m2l_few(Levels3 lv, const double* __restrict__ mt, double* __restrict__ le, const double* __restrict__ op)
{
    constexpr int W = kM2lWavesFew3;
    __shared__ f64x4 sum[W / 2 * class_tiles3(P, 0) * 64];     // class 0 has the most tiles
    if constexpr (fold3(P)) {
        switch (blockIdx.y) {
            case 0: m2l3<P, 1, W, 0, 1>(lv, mt, le, op, sum); break;
            case 1: m2l3<P, 1, W, 1, 2>(lv, mt, le, op, sum); break;
            case 2: m2l3<P, 1, W, 2, 3>(lv, mt, le, op, sum); break;
            default: m2l3<P, 1, W, 3, 4>(lv, mt, le, op, sum); break;
        }
    } else {
        m2l3<P, 1, W, 0, 1>(lv, mt, le, op, sum);
    }
}

// the kept local coefficients of `box`, spread to [r][a][b] in sK
template <int P>
__device__ __forceinline__ void load_kept3(const double* __restrict__ box, const int32_t* __restrict__ term,
                                           double* __restrict__ sK, int lane)
{
    for (int e = lane; e < stored3(P); e += 64) {
        const int id = term[e];
        if (id >= 0) sK[((id >> 16) * (P + 1) + (id & 255)) * (P + 1) + ((id >> 8) & 255)] = box[e];
    }
}

// the full set, dense [c][a][b], from the kept terms (its first two planes):
// plane c from plane c - 2 by L_(a, b, c) = -L_(a + 2, b, c - 2) - L_(a, b + 2, c - 2)
template <int P>
__device__ __forceinline__ void unfold_all3(double* __restrict__ sK, int lane)
{
    constexpr int Q = P + 1;
#pragma unroll
    for (int c = 2; c <= P; c += 2) {          // planes c and c + 1 together
        for (int e = lane; e < 2 * Q * Q; e += 64) {
            const int c1 = c + e / (Q * Q), ab = e % (Q * Q), a = ab / Q, b = ab % Q;
            if (c1 <= P && a + b + c1 <= P) {
                const double* lo = sK + (c1 - 2) * Q * Q + ab;
                sK[c1 * Q * Q + ab] = -(lo[2 * Q] + lo[2]);
            }
        }
        wave_sync3();
    }
}

// L2L from level l into its children: one wavefront per parent, one lane per
// kept output term.  A child's sign depends only on the parities of m - n, so
// a lane sums the parent's terms by these parities once and the eight
// children are signed sums of the eight (a Walsh-Hadamard transform).
// Depth 5, p = 6: 51 us for the three launches, against 209 us for one
// workgroup per child.
template <int P>
__global__ void __launch_bounds__(kTpb)
k3_l2l(int l, const int32_t* __restrict__ term, double* __restrict__ le)
{
    constexpr int KP = stored3(P), Q = P + 1, W = kTpb / 64;
    __shared__ double sK[W][Q * Q * Q];
    const int lane = int(threadIdx.x) & 63;
    const int wave = __builtin_amdgcn_readfirstlane(int(threadIdx.x) >> 6);
    const int64_t par = int64_t(blockIdx.x) * W + wave;      // 8^l parents, a multiple of W
    load_kept3<P>(le + (lvl_off3(l) + par) * KP, term, sK[wave], lane);
    wave_sync3();
    unfold_all3<P>(sK[wave], lane);
    double* dst = le + (lvl_off3(l + 1) + 8 * par) * KP;
    for (int e = lane; e < KP; e += 64) {
        const int id = term[e];
        if (id < 0) continue;
        const int a = id & 255, b = (id >> 8) & 255, c = id >> 16, m = P - a - b - c;
        double old[8];
#pragma unroll
        for (int ch = 0; ch < 8; ++ch) old[ch] = dst[ch * KP + e];
        const double* L = sK[wave] + (c * Q + a) * Q + b;
        double v[8];
#pragma unroll
        for (int pi = 0; pi < 8; ++pi) {
            double s = 0.0;
            for (int k = pi >> 2; k <= m; k += 2)
                for (int i = pi & 1; i + k <= m; i += 2) {
                    double row = 0.0;
                    for (int j = (pi >> 1) & 1; i + j + k <= m; j += 2) row += L[(k * Q + i) * Q + j] * quarter_f(j);
                    s += row * (quarter_f(i) * quarter_f(k));
                }
            v[pi] = s;
        }
#pragma unroll
        for (int h = 1; h < 8; h <<= 1)
#pragma unroll
            for (int ch = 0; ch < 8; ++ch)
                if (!(ch & h)) {
                    const double u = v[ch], w = v[ch | h];
                    v[ch] = u + w;
                    v[ch | h] = u - w;
                }
        // v[q] has the sign (-1)^popcount(pi & q): a child below the centre in the axes q
        const double sc = ldexp(1.0, -(1 + a + b + c));
#pragma unroll
        for (int ch = 0; ch < 8; ++ch) dst[ch * KP + e] = old[ch] + v[7 ^ ch] * sc;
    }
}

// ---- evaluation: L2P and the near field -----------------------------------------

constexpr int kEvalSrc3 = 256;        // sources staged at a time per wavefront
constexpr int kEvalWaves3 = 4;
constexpr int kEvalTail3 = 64;        // workgroups that clear the outputs of particles outside the cube

// One pair's term added to a target's sums.  About 25 vector instructions
// beside the reciprocal root: the hardware estimate (within 2^-24) and one
// third-order step y (1 + e/2 + 3 e^2 / 8), e = 1 - r2 y^2, which leaves
// rounding only.  Pairs at zero distance, and those whose r2 overflows (their
// terms vanish), are left out by class.  EXACT: the charge may be infinite or
// NaN, so a pair at zero distance is kept out of the product with it too.
template <bool EXACT>
__device__ __forceinline__ void pair3(double dx, double dy, double dz, double w, double& f, double& fx, double& fy,
                                      double& fz)
{
    const double r2 = fma(dx, dx, fma(dy, dy, dz * dz));
    const double y0 = __builtin_amdgcn_rsq(r2);
    const double e = fma(-(r2 * y0), y0, 1.0);
    const double y1 = fma(y0 * e, fma(e, 0.375, 0.5), y0);
    const bool ok = __builtin_amdgcn_class(r2, 0x180);       // positive normal or subnormal
    const double ir = ok ? y1 : 0.0;
    const double qr = EXACT && r2 == 0.0 ? 0.0 : w * ir;
    const double cc = qr * ir * ir;
    f += qr;
    fx = fma(-cc, dx, fx);
    fy = fma(-cc, dy, fy);
    fz = fma(-cc, dz, fz);
}

// R targets per lane; TG = ceil(t / R) lanes make a group that holds all t
// targets of a chunk, S = 64 / TG groups share the sources.  Adds the pairs of
// `cnt` staged sources (a multiple of S, padded with sources of charge zero).
template <int R>
__device__ __forceinline__ void near3(const double4* __restrict__ src, int cnt, int slice, int S, const double (&x)[R],
                                      const double (&y)[R], const double (&z)[R], double (&f)[R], double (&fx)[R],
                                      double (&fy)[R], double (&fz)[R])
{
    for (int j = slice; j < cnt; j += S) {
        const double4 s = src[j];
#pragma unroll
        for (int i = 0; i < R; ++i) pair3<false>(x[i] - s.x, y[i] - s.y, z[i] - s.z, s.w, f[i], fx[i], fy[i], fz[i]);
    }
}

// L2P of one target at offset (ux, uy, uz) box widths from the centre: the
// potential and its derivatives, summed c first, then b, then a
template <int P>
__device__ __forceinline__ void l2p3(const double* __restrict__ sL, double ux, double uy, double uz, double& f,
                                     double& fx, double& fy, double& fz)
{
    double py[P + 1], pz[P + 1];
    py[0] = pz[0] = 1.0;
#pragma unroll
    for (int k = 1; k <= P; ++k) {
        const double rk = 1.0 / double(k);     // a compile-time constant once unrolled
        py[k] = py[k - 1] * uy * rk;
        pz[k] = pz[k - 1] * uz * rk;
    }
    f = fx = fy = fz = 0.0;
    double px = 1.0, qx = 0.0;                 // ux^a / a!, ux^(a-1) / (a-1)!
#pragma unroll
    for (int a = 0; a <= P; ++a) {
        double F = 0.0, Fy = 0.0, Fz = 0.0;
#pragma unroll
        for (int b = 0; a + b <= P; ++b) {
            double s0 = 0.0, s1 = 0.0;
#pragma unroll
            for (int c = 0; a + b + c <= P; ++c) {
                const double v = sL[(c * (P + 1) + a) * (P + 1) + b];
                s0 = fma(v, pz[c], s0);
                if (c > 0) s1 = fma(v, pz[c - 1], s1);
            }
            F = fma(s0, py[b], F);
            if (b > 0) Fy = fma(s0, py[b - 1], Fy);
            Fz = fma(s1, py[b], Fz);
        }
        f = fma(px, F, f);
        fx = fma(qx, F, fx);
        fy = fma(px, Fy, fy);
        fz = fma(px, Fz, fz);
        qx = px;
        px *= ux * (1.0 / double(a + 1));
    }
}

// One chunk of t targets: the near field of the wavefront's share of the
// sources, the slices' sums through LDS, the output (by the first wavefront of
// the leaf: s holds the far field of target `lane` there).
template <int R, int WPL>
__device__ __forceinline__ void chunk3(double4 s, int t0, int t, int part, int nseg_total, const int* __restrict__ seg,
                                       const double* __restrict__ xs, const double* __restrict__ ys,
                                       const double* __restrict__ zs, const double* __restrict__ qs,
                                       const uint32_t* __restrict__ perm, double4* __restrict__ buf,
                                       double4* __restrict__ all, double* __restrict__ phi, double* __restrict__ gx, double* __restrict__ gy, double* __restrict__ gz)
{
    const int lane = int(threadIdx.x) & 63;
    const int TG = (t + R - 1) / R, S = 64 / TG;
    const int slice = lane / TG, tg = lane - slice * TG;
    const bool live = slice < S;
    double x[R], y[R], z[R], f[R], fx[R], fy[R], fz[R];
#pragma unroll
    for (int i = 0; i < R; ++i) {
        const int k = t0 + min(tg + i * TG, t - 1);
        x[i] = xs[k];
        y[i] = ys[k];
        z[i] = zs[k];
        f[i] = fx[i] = fy[i] = fz[i] = 0.0;
    }
    // this wavefront's share of the sources
    const int c_end = int(int64_t(nseg_total) * (part + 1) / WPL);
    for (int c0 = int(int64_t(nseg_total) * part / WPL); c0 < c_end; c0 += kEvalSrc3) {
        const int cnt = min(kEvalSrc3, c_end - c0);
        double4 v[kEvalSrc3 / 64];
#pragma unroll
        for (int q = 0; q < kEvalSrc3 / 64; ++q) {
            // the leaf that holds source c0 + 64 q + lane: the last whose first source is not past it
            const int k = c0 + min(64 * q + lane, cnt - 1);
            int lo = 0;
#pragma unroll
            for (int h = 16; h > 0; h >>= 1)
                if (seg[32 + lo + h] <= k) lo += h;
            const int j = seg[lo] + (k - seg[32 + lo]);
            v[q] = double4{xs[j], ys[j], zs[j], 64 * q + lane < cnt ? qs[j] : 0.0};
        }
        wave_sync3();
        bool bad = false;
#pragma unroll
        for (int q = 0; q < kEvalSrc3 / 64; ++q) {
            buf[64 * q + lane] = v[q];
            bad = bad || __builtin_amdgcn_class(v[q].w, 0x207);
        }
        wave_sync3();
        // Infinite and NaN charges act here, one after another, and are zero from
        // then on: times the zero of a coincident pair (a particle and itself)
        // they would be NaN, and a select in near3 costs every call 1.5 to 3 %
        // (octree of 2^20 charges, p = 6: 1486 us without, 1511 and 1535 with).
        if (__ballot(bad) != 0) {
#pragma unroll 1
            for (int j = 0; j < kEvalSrc3; ++j) {
                const double4 c = buf[j];
                if (!__builtin_amdgcn_class(c.w, 0x207)) continue;
                if (slice == 0)
#pragma unroll
                    for (int i = 0; i < R; ++i)
                        pair3<true>(x[i] - c.x, y[i] - c.y, z[i] - c.z, c.w, f[i], fx[i], fy[i], fz[i]);
                wave_sync3();
                buf[j].w = 0.0;
                wave_sync3();
            }
        }
        if (live) near3<R>(buf, min(kEvalSrc3, (cnt + S - 1) / S * S), slice, S, x, y, z, f, fx, fy, fz);
    }
    // sums of the slices (and, WPL > 1, of the leaf's wavefronts) in order
    wave_sync3();
    if constexpr (WPL > 1) __syncthreads();      // every wavefront's sources are behind it
    double4* mine = WPL > 1 ? all + part * kEvalSrc3 : buf;
    if (live)
#pragma unroll
        for (int i = 0; i < R; ++i)
            if (tg + i * TG < t) mine[slice * t + tg + i * TG] = double4{f[i], fx[i], fy[i], fz[i]};
    wave_sync3();
    if constexpr (WPL > 1) __syncthreads();
    if (part == 0 && lane < t) {
        for (int q = 0; q < WPL; ++q)
            for (int k = 0; k < S; ++k) {
                const double4 v = (WPL > 1 ? all + q * kEvalSrc3 : buf)[k * t + lane];
                s.x += v.x;
                s.y += v.y;
                s.z += v.z;
                s.w += v.w;
            }
        const uint32_t o = perm[t0 + lane];
        phi[o] = s.x;
        gx[o] = s.y;
        gy[o] = s.z;
        gz[o] = s.w;
    }
    wave_sync3();
    if constexpr (WPL > 1) __syncthreads();
}

// WPL = 1: one wavefront per leaf, four leaves to a workgroup; WPL = 4: four
// wavefronts per leaf, each a quarter of the source chunks (few leaves).
// Targets in chunks of 64, laid out as R per lane (near3) for the most lanes
// on real pairs; the sources of the near leaves staged in LDS, 256 at a time,
// leaf after leaf without gaps.  Held to 128 registers (four wavefronts per
// SIMD) it spills 3 to 11 of them from p = 1 on, 15 at p = 7, outside the
// pair loop; three wavefronts without spills are slower (p = 6: 1,500 us a
// whole evaluation instead of 1,485; 2^21 charges, depth 6, p = 2: 1,913 and
// 1,826).  Bound by the vector units: 2^20 charges,
// depth 5 (about 32 per leaf, 864 near sources), p = 6: 861 us, against 2,510
// us with one target per lane (half the lanes idle at 32 per leaf) and a
// library square root and division per pair.
template <int P, int WPL>
__global__ void __launch_bounds__(64 * kEvalWaves3, 4)
k3_eval(Geo3 g, int far, int n, const int32_t* __restrict__ ls, const double* __restrict__ xs,
        const double* __restrict__ ys, const double* __restrict__ zs, const double* __restrict__ qs,
        const uint32_t* __restrict__ perm, const double* __restrict__ le, const int32_t* __restrict__ term,
        double* __restrict__ phi, double* __restrict__ gx, double* __restrict__ gy, double* __restrict__ gz)
{
    constexpr int LPB = kEvalWaves3 / WPL;
    __shared__ double4 sbuf[kEvalWaves3][kEvalSrc3];
    __shared__ int sseg[kEvalWaves3][64];
    const int lane = int(threadIdx.x) & 63;
    const int wave = __builtin_amdgcn_readfirstlane(int(threadIdx.x) >> 6);
    const int nleaf = 1 << (3 * g.L);
    const int leaf_blocks = (nleaf + LPB - 1) / LPB;
    if (int(blockIdx.x) >= leaf_blocks) {       // particles outside the cube sort behind the last leaf
        for (int i = ls[nleaf] + (int(blockIdx.x) - leaf_blocks) * 64 * kEvalWaves3 + int(threadIdx.x); i < n;
             i += kEvalTail3 * 64 * kEvalWaves3) {
            const uint32_t o = perm[i];
            phi[o] = gx[o] = gy[o] = gz[o] = 0.0;
        }
        return;
    }
    const int leaf = int(blockIdx.x) * LPB + wave / WPL;
    if (leaf >= nleaf) return;                  // WPL = 1 only: no workgroup barrier follows there
    const int t0 = ls[leaf], t1 = ls[leaf + 1];
    if (t0 == t1) return;                       // the same for all wavefronts of a leaf
    const int side = 1 << g.L;
    int la, lb, lc;
    unmorton3(uint32_t(leaf), la, lb, lc);
    const double w = ldexp(g.W, -g.L);
    const double cx = g.x0 + (la + 0.5) * w, cy = g.y0 + (lb + 0.5) * w, cz = g.z0 + (lc + 0.5) * w;
    // the near leaves: first particle, and how many lie in the leaves before it (the lanes past 26 hold none)
    int* seg = sseg[wave];
    int s0 = 0, cn = 0;
    if (lane < 27) {
        const int na = la + lane % 3 - 1, nbx = lb + (lane / 3) % 3 - 1, nc = lc + lane / 9 - 1;
        if (na >= 0 && nbx >= 0 && nc >= 0 && na < side && nbx < side && nc < side) {
            const uint32_t nl = spread3(uint32_t(na)) | spread3(uint32_t(nbx)) << 1 | spread3(uint32_t(nc)) << 2;
            s0 = ls[nl];
            cn = ls[nl + 1] - s0;
        }
    }
    int inc = cn;
#pragma unroll
    for (int d = 1; d < 32; d <<= 1) {
        const int o = __shfl_up(inc, d, 64);
        if (lane >= d) inc += o;
    }
    const int total = __builtin_amdgcn_readlane(inc, 31);
    if (lane < 32) {
        seg[lane] = s0;
        seg[32 + lane] = inc - cn;
    }
    wave_sync3();
    const int part = wave % WPL;
    double4* buf = sbuf[wave];
    double4* all = sbuf[wave - part];
    for (int b = t0; b < t1; b += 64) {
        const int t = min(64, t1 - b);
        double4 s{0.0, 0.0, 0.0, 0.0};
        if (far && part == 0) {
            double* sL = reinterpret_cast<double*>(buf);
            static_assert((P + 1) * (P + 1) * (P + 1) <= 4 * kEvalSrc3, "the full set fits in the source stage");
            load_kept3<P>(le + (lvl_off3(g.L) + leaf) * stored3(P), term, sL, lane);
            wave_sync3();
            unfold_all3<P>(sL, lane);
            wave_sync3();
            if (lane < t) {
                double lf, lx, ly, lz;
                l2p3<P>(sL, (xs[b + lane] - cx) / w, (ys[b + lane] - cy) / w, (zs[b + lane] - cz) / w, lf, lx, ly, lz);
                const double w2 = w * w;
                s = double4{lf / w, lx / w2, ly / w2, lz / w2};
            }
        }
        // pairs per lane step on real targets: t S / (64 R)
        const int s1 = 64 / t, s2 = 64 / ((t + 1) / 2), s4 = 64 / ((t + 3) / 4);
        const int e1 = 4 * t * s1, e2 = 2 * t * s2, e4 = t * s4;
        if (e4 >= e2 && e4 >= e1)
            chunk3<4, WPL>(s, b, t, part, total, seg, xs, ys, zs, qs, perm, buf, all, phi, gx, gy, gz);
        else if (e2 >= e1)
            chunk3<2, WPL>(s, b, t, part, total, seg, xs, ys, zs, qs, perm, buf, all, phi, gx, gy, gz);
        else
            chunk3<1, WPL>(s, b, t, part, total, seg, xs, ys, zs, qs, perm, buf, all, phi, gx, gy, gz);
    }
}

int blocks(int64_t n) { return int((n + kTpb - 1) / kTpb); }

}  // namespace

hipError_t launch3_clear(const Bufs3& b, hipStream_t st)
{
    hipLaunchKernelGGL(k3_clear, dim3(1), dim3(1), 0, st, b.nbad);
    return hipGetLastError();
}

hipError_t launch3_tree(const Bufs3& b, const Geo3& g, int n, const double* x, const double* y, const double* z,
                        const double* q, hipStream_t st)
{
    hipLaunchKernelGGL(k3_keys, dim3(blocks(n)), dim3(kTpb), 0, st, n, x, y, z, g, b.key, b.nbad);
    const hipError_t e = fmm::launch_sort_keys(b.sort, n, b.key, x, y, q, b.ks, b.perm, b.xs, b.ys, b.qs,
                                               3 * g.L + 1, st);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k3_gather, dim3(blocks(n)), dim3(kTpb), 0, st, n, b.perm, z, b.zs);
    const int64_t nleaf = int64_t(1) << (3 * g.L);
    hipLaunchKernelGGL(k3_leaf_start, dim3(blocks(nleaf + 1)), dim3(kTpb), 0, st, nleaf, n, b.ks, b.leaf_start);
    return hipGetLastError();
}

namespace {

template <int P>
hipError_t upward_p(const Bufs3& b, const Geo3& g, hipStream_t st)
{
    const unsigned nleaf = 1u << (3 * g.L);
    hipLaunchKernelGGL((k3_p2m<P>), dim3((nleaf + 3) / 4), dim3(kTpb), 0, st, g, b.leaf_start, b.xs, b.ys, b.zs, b.qs,
                       b.term, b.me);
    const unsigned nt = (tet3(P + 1) + 63) / 64 * 64;       // one thread per term of the full set
    for (int l = g.L - 1; l >= 2; --l)
        hipLaunchKernelGGL((k3_m2m<P>), dim3(1u << (3 * l)), dim3(nt), 0, st, l, b.term, b.me);
    return hipGetLastError();
}

template <int P>
hipError_t m2l_p(const Bufs3& b, const Geo3& g, hipStream_t st)
{
    Levels3 sp{}, lv{}, few{};
    sp.n_levels = lv.n_levels = few.n_levels = g.L - 1;
    int ns = 0, nm = 0, nf = 0;
    for (int l = 2; l <= g.L; ++l) {
        const int64_t n = int64_t(1) << (3 * (l - 1));
        sp.blk_begin[l - 2] = ns;
        lv.blk_begin[l - 2] = nm;
        few.blk_begin[l - 2] = nf;
        nf += 8 * int((n + 15) / 16);
        ns += 8 * int((grid3(P, l) + 63) / 64);
        nm += 8 * int((n + 16 * kM2lGroups3 - 1) / (16 * kM2lGroups3));
    }
    sp.blk_begin[g.L - 1] = ns;
    lv.blk_begin[g.L - 1] = nm;
    few.blk_begin[g.L - 1] = nf;
    hipLaunchKernelGGL((k3_spread<P>), dim3(unsigned(ns)), dim3(kTpb), 0, st, sp, b.me, b.mt);
    // below two workgroups a CU (depth <= 4): whole evaluations at p = 6 / 9 of
    // 2,000 charges, depth 2, 185 / 435 us with 32-target workgroups, 101 /
    // 183 with these; 16,000, depth 3, 256 / 521 and 165 / 269; 131,072,
    // depth 4, 397 / 695 and 384 / 674
    if (nm < 512)
        hipLaunchKernelGGL((k3_m2l_few<P>), dim3(unsigned(nf), unsigned(classes3(P))), dim3(64 * kM2lWavesFew3), 0, st, few,
                           b.mt, b.le, b.op);
    else
        hipLaunchKernelGGL((k3_m2l<P>), dim3(unsigned(nm)), dim3(64 * kM2lWaves3), 0, st, lv, b.mt, b.le, b.op);
    return hipGetLastError();
}

template <int P>
hipError_t l2l_p(const Bufs3& b, const Geo3& g, hipStream_t st)
{
    for (int l = 2; l < g.L; ++l)
        hipLaunchKernelGGL((k3_l2l<P>), dim3((1u << (3 * l)) / 4), dim3(kTpb), 0, st, l, b.term, b.le);
    return hipGetLastError();
}

// Four wavefronts share a leaf's sources where leaves are few, or are too few
// to fill the chip and dense enough for four (whole evaluations with one / four
// at p = 4: 2,000 charges in 64 leaves 159 / 129 us, 16,000 in 512 207 / 189,
// 131,072 in 4,096 332 / 325, but 40,000 in 4,096 210 / 238).
bool eval_shared3(int64_t nleaf, int n) { return nleaf <= 1024 || (nleaf <= 4096 && n >= 24 * nleaf); }

template <int P>
hipError_t eval_p(const Bufs3& b, const Geo3& g, int n, double* phi, double* gx, double* gy, double* gz, hipStream_t st)
{
    const unsigned nleaf = 1u << (3 * g.L);
    const int far = g.L >= 2 ? 1 : 0;
    if (!eval_shared3(nleaf, n))
        hipLaunchKernelGGL((k3_eval<P, 1>), dim3((nleaf + 3) / 4 + kEvalTail3), dim3(64 * kEvalWaves3), 0, st, g, far,
                           n, b.leaf_start, b.xs, b.ys, b.zs, b.qs, b.perm, b.le, b.term, phi, gx, gy, gz);
    else
        hipLaunchKernelGGL((k3_eval<P, 4>), dim3(nleaf + kEvalTail3), dim3(64 * kEvalWaves3), 0, st, g, far, n,
                           b.leaf_start, b.xs, b.ys, b.zs, b.qs, b.perm, b.le, b.term, phi, gx, gy, gz);
    return hipGetLastError();
}

// f(std::integral_constant<int, p>) for the plan's degree
template <typename F>
hipError_t by_degree(int p, F&& f)
{
    switch (p) {
        case 0: return f(std::integral_constant<int, 0>{});
        case 1: return f(std::integral_constant<int, 1>{});
        case 2: return f(std::integral_constant<int, 2>{});
        case 3: return f(std::integral_constant<int, 3>{});
        case 4: return f(std::integral_constant<int, 4>{});
        case 5: return f(std::integral_constant<int, 5>{});
        case 6: return f(std::integral_constant<int, 6>{});
        case 7: return f(std::integral_constant<int, 7>{});
        case 8: return f(std::integral_constant<int, 8>{});
        case 9: return f(std::integral_constant<int, 9>{});
        default: return hipErrorInvalidValue;
    }
}

}  // namespace

hipError_t launch3_upward(const Bufs3& b, const Geo3& g, hipStream_t st)
{
    return by_degree(g.p, [&](auto d) { return upward_p<decltype(d)::value>(b, g, st); });
}

hipError_t launch3_m2l(const Bufs3& b, const Geo3& g, hipStream_t st)
{
    return by_degree(g.p, [&](auto d) { return m2l_p<decltype(d)::value>(b, g, st); });
}

hipError_t launch3_l2l(const Bufs3& b, const Geo3& g, hipStream_t st)
{
    return by_degree(g.p, [&](auto d) { return l2l_p<decltype(d)::value>(b, g, st); });
}

hipError_t launch3_eval(const Bufs3& b, const Geo3& g, int n, double* phi, double* gx, double* gy, double* gz,
                        hipStream_t st)
{
    return by_degree(g.p, [&](auto d) { return eval_p<decltype(d)::value>(b, g, n, phi, gx, gy, gz, st); });
}

}  // namespace fmm3
