// fmm_fgt.hip -- the fast Gauss transform on the quadtree's leaf boxes
// (Section 8 names the fast Gauss transform among the transforms the library
// should take next):
//   G(y_i) = sum_j q_j exp(-|y_i - x_j|^2 / delta),   delta = 2 sigma^2,
// at the particles (the term j = i included), by the published algorithm of
// Greengard and Strain (SIAM J. Sci. Stat. Comput. 12, 1991):
//   P2H  every leaf box B: A_a = sum_j q_j s1^a1 s2^a2 / (a1! a2!),
//        s = (x_j - c_B) / sqrt(delta), a1, a2 < p (its Hermite expansion);
//   H2T  every leaf box C, from every box B within Chebyshev box distance nc:
//        B_b += sum_a A_a h_{a1+b1}(tau1) h_{a2+b2}(tau2),
//        tau = (c_C - c_B) / sqrt(delta), h_n the Hermite functions;
//   T2P  G(y) = sum_b B_b (-1)^(b1+b2) u1^b1 u2^b2 / (b1! b2!),
//        u = (y - c_C) / sqrt(delta) (the Taylor expansion about c_C).
// The box offsets are integers, so tau takes the values d w / sqrt(delta),
// |d| <= nc, and the h_n(tau) form one small table (built on the host).
// H2T separates into a pass along x and one along y (k_h2t_axis).
#include "fmm_device.h"

namespace fmm {
namespace {

constexpr int kFgtThreads = 256;
typedef double f64x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ double box_centre(uint32_t k, double o, double w)
{
    return o + (double(k) + 0.5) * w;
}

// the lanes of a wavefront see each other's LDS writes past this point
__device__ __forceinline__ void wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// P2H: A_{a1, a2} = sum_j (q s2^a2) (s1^a1), scaled by 1/(a1! a2!) (zero for
// terms >= p, which the table fk holds).  The sum is a matrix product over
// the box's particles, so it runs on v_mfma_f64_16x16x4: four particles per
// instruction, lane l holding s1^(l mod 16) and q s2^(l mod 16) of particle
// l / 16; rows and columns >= P are computed and not written.  W wavefronts
// share a box (their sums meet in LDS, added in wavefront order).
// Every lane forms the powers of one particle and hands them over through
// LDS.  Bound by that staging and the load latency of a box's particles: 2^20
// particles in 4,096 boxes (P = 12) take 21 us (31 us with every lane forming
// its own powers; 127 us for one lane per (box, a1) summing its particles one
// after another).
template <int P, int W>
__global__ void __launch_bounds__(W == 16 ? 1024 : kFgtThreads, 2)
k_p2h(int L, const Inst* __restrict__ inst, const int32_t* __restrict__ leaf_start, const double* __restrict__ xs,
      const double* __restrict__ ys, const double* __restrict__ gs, const double* __restrict__ fk, double rsd,
      double* __restrict__ A)
{
    constexpr int kThreads = W == 16 ? 1024 : kFgtThreads, kWaves = kThreads / 64, kBoxes = kWaves / W;
    // per wavefront the powers of C particles, kStride apart (8 a + k mod 32:
    // the 16 x 4 values of an instruction lie in different banks); later the
    // wavefronts' sums
    constexpr int C = W == 16 ? 32 : 64, kStride = C + 4, kShare = 2 * P * kStride;
    static_assert(W == 1 || kShare >= 256, "room for a wavefront's sums");
    __shared__ double sh[kWaves][kShare];
    const int lane = threadIdx.x & 63, wv = int(threadIdx.x) >> 6;
    const int64_t m = int64_t(blockIdx.x) * kBoxes + wv / W;
    const bool box = m < (int64_t(1) << (2 * L));
    const Domain d = inst[0].dom;
    const double w = ldexp(d.W, -L);
    const double cx = box_centre(morton_x(uint32_t(m)), d.x0, w);
    const double cy = box_centre(morton_y(uint32_t(m)), d.y0, w);
    const int a = lane & 15, k = lane >> 4;
    double* s1 = sh[wv];
    double* s2 = s1 + P * kStride;
    const int ar = a < P ? a : 0;      // columns >= P repeat one that exists
    f64x4 acc = {0.0, 0.0, 0.0, 0.0};
    if (box) {
        const int j1 = leaf_start[m + 1];
        int jb = leaf_start[m] + C * (wv % W);
        const auto load = [&](int j, double& x, double& y, double& q) {
            const bool in = lane < C && j < j1;
            x = in ? (xs[j] - cx) * rsd : 0.0;
            y = in ? (ys[j] - cy) * rsd : 0.0;
            q = in ? gs[j] : 0.0;
        };
        double x, y, q;
        load(jb + lane, x, y, q);
        for (; jb < j1; jb += C * W) {
            if (lane < C) {
                double px = 1.0, py = q;
#pragma unroll
                for (int t = 0; t < P; ++t) {
                    s1[t * kStride + lane] = px;
                    s2[t * kStride + lane] = py;
                    px *= x;
                    py *= y;
                }
            }
            load(jb + C * W + lane, x, y, q);       // the next ones, in flight during the products
            wave_sync();
            const int steps = (min(C, j1 - jb) + 3) / 4;
#pragma unroll 4
            for (int t = 0; t < steps; ++t) {
                const int j = ar * kStride + 4 * t + k;
                acc = __builtin_amdgcn_mfma_f64_16x16x4f64(s1[j], s2[j], acc, 0, 0, 0);
            }
            wave_sync();
        }
    }
    // lane l holds rows l / 16 + 4 r, column l mod 16
    if constexpr (W == 1) {
        if (!box || a >= P) return;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int a1 = k + 4 * r;
            if (a1 < P) A[m * (P * P) + a1 * P + a] = acc[r] * fk[a1] * fk[a];
        }
    } else {
        static_assert(W == 1 || kBoxes == 1, "one box per workgroup where wavefronts share it");
        // a wavefront's own powers are behind it (wave_sync above)
#pragma unroll
        for (int r = 0; r < 4; ++r) sh[wv][(k + 4 * r) * 16 + a] = acc[r];
        __syncthreads();
        const int a1 = int(threadIdx.x) >> 4, a2 = int(threadIdx.x) & 15;
        if (threadIdx.x >= 256 || a1 >= P || a2 >= P) return;
        double s = 0.0;
#pragma unroll
        for (int q = 0; q < W; ++q) s += sh[q][threadIdx.x];
        A[m * (P * P) + a1 * P + a2] = s * fk[a1] * fk[a2];
    }
}

// H2T along one axis.  h_{a1+b1}(tau1) h_{a2+b2}(tau2) is a product and the
// range a square of boxes, so the sum over the (2 nc + 1)^2 boxes separates
// into a pass along x and one along y over the result,
//   C_{b1,a2} = sum_da sum_a1 h_{a1+b1}(da) A_{a1,a2}(da),
//   B_{b1,b2} = sum_db sum_a2 h_{a2+b2}(db) C_{b1,a2}(db),
// 2 (2 nc + 1) p^3 multiply-adds per box instead of 2 (2 nc + 1)^2 p^3.  Both
// passes are this kernel: it contracts the first index of `in` and writes the
// result with its two indices exchanged, so the second pass contracts the
// other one.  It is a product of the P x P Hankel matrix h_{a+b}(d) with the
// box's coefficients for every d, so it runs on v_mfma_f64_16x16x4: rows are
// the outputs b, columns the other index (16 / P boxes side by side for
// P = 8, else one box), four a per instruction; rows and columns >= P are
// computed and not written.  A wavefront takes its boxes along a line, the
// table h_n(d w / sqrt(delta)) at [(d + nc) (2P - 1) + n] comes from LDS, the
// coefficients straight from memory with those of the next d in flight.  The
// last pass (LAST) scales by (-1)^(b1+b2) / (b1! b2!), zero for terms >= p.
// On 4,096 boxes (nc = 11, P = 12) a pass takes 20 us (matrix cores alone
// 8 us; 28 us with vector multiply-adds, four outputs per thread); the sum
// over all pairs of boxes took 812 us.
template <int P, bool LAST>
__global__ void __launch_bounds__(kFgtThreads, 2)
k_h2t_axis(int L, int nc, int axis, const double* __restrict__ in, const double* __restrict__ ht,
           const double* __restrict__ fk, double* __restrict__ out)
{
    constexpr int NH = 2 * P - 1, kBoxes = 16 / P, K = P / 4;
    static_assert(P % 4 == 0 && P <= 16, "whole matrix instructions");
    extern __shared__ double sht[];
    const int nt = (2 * nc + 1) * NH;
    for (int e = threadIdx.x; e < nt; e += kFgtThreads) sht[e] = ht[e];
    __syncthreads();
    const int64_t side = int64_t(1) << L;
    const int lane = threadIdx.x & 63, col = lane & 15, k = lane >> 4;
    const int G = int(gridDim.x);
    const int wave = __builtin_amdgcn_readfirstlane(int(threadIdx.x) >> 6);
    // the wavefront's first box: box q of the lines along the axis, one line after another
    const int64_t q0 = (int64_t(xcd_runs(int(blockIdx.x), G, G / kXcds)) * (kFgtThreads / 64) + wave) * kBoxes;
    if (q0 >= side * side) return;
    const int line = int(q0 >> L), c0 = int(q0 & (side - 1));
    const int box = col / P < kBoxes ? col / P : 0, j = col % P;
    const int c = c0 + box;
    const double* src = in + k * P + j;
    const int d0 = max(-nc, c0 - int(side) + 1), d1 = min(nc, c0 + kBoxes - 1);
    const auto load = [&](int d, double (&v)[K]) {
        const int s = c - d;
        const bool ok = s >= 0 && s < int(side) && d <= d1;
        const uint32_t so = uint32_t(ok ? s : 0);
        const double* a = src + int64_t(axis == 0 ? morton(so, uint32_t(line)) : morton(uint32_t(line), so)) * (P * P);
#pragma unroll
        for (int t = 0; t < K; ++t) v[t] = ok ? a[4 * t * P] : 0.0;
    };
    const int row = min(col, P - 1) + k;       // a + b of the lane's Hankel entry, a = 4 t + k
    f64x4 acc = {0.0, 0.0, 0.0, 0.0};
    double v[K], nx[K];
    load(d0, v);
    for (int d = d0; d <= d1; ++d) {
        load(d + 1, nx);
        const double* h = sht + (d + nc) * NH + row;
#pragma unroll
        for (int t = 0; t < K; ++t) acc = __builtin_amdgcn_mfma_f64_16x16x4f64(h[4 * t], v[t], acc, 0, 0, 0);
#pragma unroll
        for (int t = 0; t < K; ++t) v[t] = nx[t];
    }
    // lane l holds rows l / 16 + 4 r of column l mod 16
    if (col >= kBoxes * P || q0 + box >= side * side) return;
    const uint32_t m = axis == 0 ? morton(uint32_t(c), uint32_t(line)) : morton(uint32_t(line), uint32_t(c));
    double* dst = out + int64_t(m) * (P * P) + j * P;
#pragma unroll
    for (int r = 0; r < K; ++r) {
        const int b = k + 4 * r;
        if constexpr (LAST)
            dst[b] = acc[r] * (((j + b) & 1) ? -fk[j] : fk[j]) * fk[b];
        else
            dst[b] = acc[r];
    }
}

// T2P: one particle (or target point) per thread in sorted order, G to its
// input position; v is cleared.  Where the points of a wavefront lie in at most
// kT2pBoxes boxes, the coefficients of each come through scalar loads, shared
// by all lanes (every lane evaluates every box of its wavefront and keeps its
// own); otherwise each lane gathers those of its own box.  Bound by the vector
// loads of the coefficients when gathered; the scalar ones are a chain of
// latencies, which pays for one box only, and from four wavefronts a SIMD on.
// Whole evaluations gathered / one box shared / up to four, us: 2^20 particles,
// 4,096 boxes 154 / 144 / 148 (p = 12), 194 / 166 / 183 (16); 2^18, 256 boxes
// 73 / 69 / 78 (16); 2^17, 256 boxes 57 / 59 / 69 (16); 2^18, 4,096 boxes
// 112 / 112 / 125 (16).
constexpr int kT2pBoxes = 1;
constexpr int kT2pSharedMin = 1 << 18;

template <int P, typename Coef>
__device__ __forceinline__ double taylor2(const Coef* __restrict__ b, double u1, double u2)
{
    double acc = 0.0;
#pragma unroll
    for (int b1 = P - 1; b1 >= 0; --b1) {
        double r = 0.0;
#pragma unroll
        for (int b2 = P - 1; b2 >= 0; --b2) r = fma(r, u2, b[b1 * P + b2]);
        acc = fma(acc, u1, r);
    }
    return acc;
}

template <int P>
__global__ void __launch_bounds__(kFgtThreads)
k_t2p(int n, int L, const Inst* __restrict__ inst, const uint32_t* __restrict__ ksorted,
      const double* __restrict__ xs, const double* __restrict__ ys, const uint32_t* __restrict__ perm,
      const double* __restrict__ Bc, double rsd, double* __restrict__ u, double* __restrict__ v)
{
    const int i = blockIdx.x * kFgtThreads + threadIdx.x;
    const bool act = i < n;
    const int ic = act ? i : n - 1;
    const uint32_t m = ksorted[ic];                // single instance: the key is the leaf
    const uint32_t o = perm[ic];
    const Domain d = inst[0].dom;
    const double w = ldexp(d.W, -L);
    const double u1 = (xs[ic] - box_centre(morton_x(m), d.x0, w)) * rsd;
    const double u2 = (ys[ic] - box_centre(morton_y(m), d.y0, w)) * rsd;
    const uint32_t prev = uint32_t(__shfl_up(int(m), 1, 64));
    const int boxes = 1 + __popcll(__ballot(__lane_id() > 0 && m != prev));
    double acc = 0.0;
    if (n >= kT2pSharedMin && boxes <= kT2pBoxes) {
        uint64_t todo = __ballot(true);
        while (todo) {
            const uint32_t mu = uint32_t(__builtin_amdgcn_readlane(int(m), __ffsll((unsigned long long)todo) - 1));
            const double r = taylor2<P>(Bc + int64_t(mu) * (P * P), u1, u2);
            if (m == mu) acc = r;
            todo &= ~__ballot(m == mu);
        }
    } else {
        acc = taylor2<P>(Bc + int64_t(m) * (P * P), u1, u2);
    }
    if (!act) return;
    u[o] = acc;
    v[o] = 0.0;
}

template <int P>
hipError_t fgt_impl(const Buffers& b, int n, int L, double sigma, int nc, int m, double* u, double* v,
                    hipStream_t st)
{
    const int64_t nbox = int64_t(1) << (2 * L);
    const double rsd = 1.0 / std::sqrt(2.0 * sigma * sigma);
    // wavefronts per box: enough to fill the chip's 1,024 SIMDs (the whole
    // transform of 2^20 particles, P = 12, with 1 / 4 / 16 per box: 64 boxes
    // 472 / 178 / 146 us, 256 boxes 189 / 116 / 108, 1,024 boxes 154 / 144 /
    // 149, 4,096 boxes 161 / 162 / 186, 16,384 boxes 250 / 284 / 376)
    if (nbox >= 4096)
        hipLaunchKernelGGL((k_p2h<P, 1>), dim3(unsigned((nbox + 3) / 4)), dim3(kFgtThreads), 0, st, L, b.inst,
                           b.leaf_start, b.xs, b.ys, b.gs, b.t_sout, rsd, b.fgt_a);
    else if (nbox >= 1024)
        hipLaunchKernelGGL((k_p2h<P, 4>), dim3(unsigned(nbox)), dim3(kFgtThreads), 0, st, L, b.inst, b.leaf_start,
                           b.xs, b.ys, b.gs, b.t_sout, rsd, b.fgt_a);
    else
        hipLaunchKernelGGL((k_p2h<P, 16>), dim3(unsigned(nbox)), dim3(1024), 0, st, L, b.inst, b.leaf_start, b.xs,
                           b.ys, b.gs, b.t_sout, rsd, b.fgt_a);
    const size_t lds = sizeof(double) * size_t(2 * nc + 1) * (2 * P - 1);
    constexpr int kBoxes = 16 / P * (kFgtThreads / 64);
    const dim3 grid(unsigned((nbox + kBoxes - 1) / kBoxes));
    hipLaunchKernelGGL((k_h2t_axis<P, false>), grid, dim3(kFgtThreads), lds, st, L, nc, 0, b.fgt_a, b.fgt_h,
                       b.t_sout, b.fgt_b);
    hipLaunchKernelGGL((k_h2t_axis<P, true>), grid, dim3(kFgtThreads), lds, st, L, nc, 1, b.fgt_b, b.fgt_h,
                       b.t_sout, b.fgt_a);
    if (m > 0)   // at the sorted target points
        hipLaunchKernelGGL(k_t2p<P>, dim3(unsigned((m + kFgtThreads - 1) / kFgtThreads)), dim3(kFgtThreads), 0, st,
                           m, L, b.inst, b.tks, b.txs, b.tys, b.tperm, b.fgt_a, rsd, u, v);
    else
        hipLaunchKernelGGL(k_t2p<P>, dim3(unsigned((n + kFgtThreads - 1) / kFgtThreads)), dim3(kFgtThreads), 0, st,
                           n, L, b.inst, b.ksorted, b.xs, b.ys, b.perm, b.fgt_a, rsd, u, v);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_fgt(const Buffers& b, int P, int n, int L, double sigma, int nc, int m, double* u, double* v,
                      hipStream_t st)
{
    if (n <= 0) return hipSuccess;
    switch (P) {
        case 8: return fgt_impl<8>(b, n, L, sigma, nc, m, u, v, st);
        case 12: return fgt_impl<12>(b, n, L, sigma, nc, m, u, v, st);
        case 16: return fgt_impl<16>(b, n, L, sigma, nc, m, u, v, st);
        default: return hipErrorInvalidValue;
    }
}

void fgt_hermite_table(int P, int nc, double w_over_sd, double* out)
{
    const int NH = 2 * P - 1;
    for (int d = -nc; d <= nc; ++d) {
        const double t = double(d) * w_over_sd;
        double* h = out + (d + nc) * NH;
        h[0] = std::exp(-t * t);
        if (NH > 1) h[1] = 2.0 * t * h[0];
        for (int k = 1; k + 1 < NH; ++k) h[k + 1] = 2.0 * t * h[k] - 2.0 * double(k) * h[k - 1];
    }
}

}  // namespace fmm
