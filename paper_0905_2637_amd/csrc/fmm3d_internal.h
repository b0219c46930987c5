// fmm3d_internal.h -- device buffers, geometry and launchers of the 3D form
// (fmm3d.hip, fmm3d_api.cpp).
//
// Expansions.  A coefficient has a multi-index (a, b, c) of total degree <= p.
// 1/r is harmonic, so its derivatives D_m satisfy D_(m + 2 e_z) = -D_(m + 2 e_x)
// - D_(m + 2 e_y): moments only matter up to that relation, and the local
// coefficients obey it.  Both are therefore kept for c <= 1 alone, (p + 1)^2
// terms instead of (p + 1)(p + 2)(p + 3)/6; the other terms of a moment set
// are folded into these, those of a local set follow from these, in either
// case within one degree, so nothing but rounding changes.
//
// Kept terms are stored by class, the parities of (a, b): four classes where
// the M2L folds reflections (fold3(p)), each padded to a multiple of 4 with
// zeros, since the M2L's matrix instructions take four source terms of one
// class; else one class, not padded.  Graded order (degree, then s = b + c, then c) puts
// (a, b, c) of a full set at tet(a + b + c) + tri(b + c) + c with tet(d) =
// d (d+1) (d+2) / 6 and tri(s) = s (s+1) / 2.
#pragma once

#include "fmm_internal.h"

namespace fmm {
// Stable LSD radix sort of n precomputed 32-bit keys (key_bits of them
// significant) carrying (input index, x, y, g); final arrays in (ks, perm,
// xs, ys, gs).  Uses the radix temporaries of b.  n >= 1.
hipError_t launch_sort_keys(const Buffers& b, int n, const uint32_t* key, const double* x, const double* y,
                            const double* g, uint32_t* ks, uint32_t* perm, double* xs, double* ys, double* gs,
                            int key_bits, hipStream_t st);
}  // namespace fmm

namespace fmm3 {

constexpr int kP3Max = 9;          // expansion degree
constexpr int kDepth3Max = 7;      // 21 key bits plus the outside flag
constexpr int kOffsets3 = 343;     // offsets in [-3, 3]^3

__host__ __device__ constexpr int tet3(int d) { return d * (d + 1) * (d + 2) / 6; }
__host__ __device__ constexpr int tri3(int s) { return s * (s + 1) / 2; }
__host__ __device__ constexpr int pos3(int a, int b, int c) { return tet3(a + b + c) + tri3(b + c) + c; }
__host__ __device__ constexpr int64_t lvl_off3(int l) { return ((int64_t(1) << (3 * l)) - 1) / 7; }
__host__ __device__ constexpr int off3_index(int ox, int oy, int oz) { return ((oz + 3) * 7 + (oy + 3)) * 7 + (ox + 3); }

// The M2L folds the reflections of x and y (one operator for up to four
// offsets, its rows split into the four classes) where the split rows fill
// their 16-row tiles well enough: from p = 5 on (p = 4: 2,688 matrix
// instructions per 16 targets folded against 2,646 unfolded; p = 5: 3,360
// against 5,103; p = 6: 4,368 against 9,828).
__host__ __device__ constexpr bool fold3(int p) { return p >= 5; }
__host__ __device__ constexpr int classes3(int p) { return fold3(p) ? 4 : 1; }
__host__ __device__ constexpr int class3(int p, int a, int b) { return fold3(p) ? (a & 1) | ((b & 1) << 1) : 0; }
// kept terms of a class, and stored ones
__host__ __device__ constexpr int class_terms3(int p, int cl)
{
    int n = 0;
    for (int c = 0; c <= 1 && c <= p; ++c)
        for (int a = 0; a + c <= p; ++a)
            for (int b = 0; a + b + c <= p; ++b) n += class3(p, a, b) == cl ? 1 : 0;
    return n;
}
__host__ __device__ constexpr int class_size3(int p, int cl)
{
    return fold3(p) ? (class_terms3(p, cl) + 3) / 4 * 4 : class_terms3(p, cl);
}
__host__ __device__ constexpr int class_base3(int p, int cl)
{
    int n = 0;
    for (int k = 0; k < cl; ++k) n += class_size3(p, k);
    return n;
}
// stored doubles per box
__host__ __device__ constexpr int stored3(int p) { return class_base3(p, classes3(p)); }

// M2L matrix instructions: steps of four source terms, 16-row tiles of output
// terms.
__host__ __device__ constexpr int steps3(int p) { return (stored3(p) + 3) / 4; }
__host__ __device__ constexpr int class_tiles3(int p, int cl) { return (class_size3(p, cl) + 15) / 16; }
__host__ __device__ constexpr int tile_base3(int p, int cl)
{
    int n = 0;
    for (int k = 0; k < cl; ++k) n += class_tiles3(p, k);
    return n;
}
__host__ __device__ constexpr int tiles3(int p) { return tile_base3(p, classes3(p)); }
// operators of the M2L: folded, offsets (|ox|, |oy|, oz); else all offsets
__host__ __device__ constexpr int operators3(int p) { return fold3(p) ? 4 * 4 * 7 : kOffsets3; }
__host__ __device__ constexpr int operator3(int p, int ox, int oy, int oz)
{
    return fold3(p) ? ((oz + 3) * 4 + oy) * 4 + ox : off3_index(ox, oy, oz);
}

// doubles of one operator: folded, a lane's value of every matrix instruction
// (steps, tiles, 64); else the stored terms' square, [source][output]
__host__ __device__ constexpr int operator_size3(int p)
{
    return fold3(p) ? steps3(p) * tiles3(p) * 64 : stored3(p) * stored3(p);
}

// M2L sources of level l (l >= 2): the boxes of one child position form the
// grid of their parents, 2^(l-1) a side.  The sources of a box lie under its
// parent and the parents touching that one: at a fixed distance, zero outside
// the cube.  Folded: with a border of one, so that they are found there.  Else
// one zero box behind the grid and a lane turned to it where its source is
// outside, which keeps the few terms of these degrees within the workspace of
// two full sets (a border adds 7 to 12 % at depth 7, six times the boxes at 2).
__host__ __device__ constexpr int64_t grid3(int p, int l)
{
    const int64_t h = int64_t(1) << (l - 1), s = h + 2;
    return fold3(p) ? s * s * s : h * h * h + 1;
}
// first source double of level l, in boxes (times stored3(p))
__host__ __device__ constexpr int64_t grid_off3(int p, int l)
{
    int64_t n = 0;
    for (int k = 2; k < l; ++k) n += 8 * grid3(p, k);
    return n;
}

// Cube [x0, x0 + W)^3, depth L, degree p.
struct Geo3 {
    double x0, y0, z0, W;
    int L, p;
};

struct Bufs3 {
    fmm::Buffers sort;          // radix temporaries only (hist, scan_part, ktmp, itmp, xt, yt, gt)
    uint32_t* key;              // [n_max] leaf key per input particle (2^(3L) outside the cube)
    uint32_t* ks;               // [n_max] sorted keys
    uint32_t* perm;             // [n_max] sorted position -> input index
    double *xs, *ys, *zs, *qs;  // [n_max] sorted particles
    int32_t* leaf_start;        // [8^L + 1] sorted range of every leaf; the last entry counts the inside ones
    double* me;                 // [boxes of levels 0..L][stored3(p)] scaled moments
    double* mt;                 // levels 2..L: the moments again as the M2L reads them, [child position][stored3(p)]
                                // [parents of the level above, x fastest, and zeros: grid3]
    double* le;                 // [boxes of levels 0..L][stored3(p)] scaled local coefficients (over me: the M2L
                                // reads mt alone)
    double* op;                 // [operators3(p)][operator_size3(p)] M2L operators
    int32_t* term;              // [stored3(p)] a | b << 8 | c << 16 of every stored position, -1: padding
    unsigned long long* nbad;   // particles outside the cube or NaN
};

hipError_t launch3_tree(const Bufs3& b, const Geo3& g, int n, const double* x, const double* y, const double* z,
                        const double* q, hipStream_t st);
hipError_t launch3_upward(const Bufs3& b, const Geo3& g, hipStream_t st);
hipError_t launch3_m2l(const Bufs3& b, const Geo3& g, hipStream_t st);
hipError_t launch3_l2l(const Bufs3& b, const Geo3& g, hipStream_t st);
hipError_t launch3_eval(const Bufs3& b, const Geo3& g, int n, double* phi, double* gx, double* gy, double* gz,
                        hipStream_t st);
hipError_t launch3_clear(const Bufs3& b, hipStream_t st);

}  // namespace fmm3
