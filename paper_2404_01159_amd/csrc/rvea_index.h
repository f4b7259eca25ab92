// rvea_index.h -- the cell of a reference vector (or a row direction) in
// the association index: a G x G grid over the scaled simplex for three
// objectives, a line of G cells for two.  Shared by the index build
// (k_grid.hip) and the adaptation, which counts each adapted vector into
// its cell as it writes it (k_vectors.hip).
#pragma once

#include <hip/hip_runtime.h>

#include "rvea_dev.h"

namespace rvea {

// cell (its place in row order) of a direction x >= 0 (x != 0); q pulled onto the simplex if rounding
// left it just outside.  -1 if the coordinates are not finite.
__device__ __forceinline__ int cell_of(double x0, double x1, double x2, const double *r, int G)
{
    const double y0 = x0 / r[0], y1 = x1 / r[1], y2 = x2 / r[2];
    const double s = y0 + y1 + y2;
    double q1 = y0 / s, q2 = y1 / s;
    if (!(q1 >= 0.0 && q2 >= 0.0 && q1 <= 2.0 && q2 <= 2.0)) return -1;
    const double t = q1 + q2;
    if (t > 1.0) {
        q1 /= t;
        q2 /= t;
    }
    int ci = (int)floor(q1 * G), cj = (int)floor(q2 * G);
    ci = ci < 0 ? 0 : (ci > G - 1 ? G - 1 : ci);
    const int end = ci <= 1 ? G - 1 : G - ci;
    cj = cj < 0 ? 0 : (cj > end ? end : cj);
    return (int)(grid_row(G, ci) + (uint32_t)cj);
}

// Vectors that a grid cell holds (two on average, at most four of a lattice under
// its own scaling; a cell with more leaves the cells around it to full scans).
// Fixed places, cell c's from c * bucket_places on, let the pass that writes a
// vector put it there at once: with ranges sized to the cells a rebuild needed two
// kernels more.  Half as many for few vectors, where a full scan is short and
// sixteen places a cell would be more memory than those ranges took.
constexpr int kBucket = 16;  // at most
__host__ __device__ inline int bucket_places(int64_t K) { return K <= 128 ? kBucket / 2 : kBucket; }

// Vector j = v (norm vn) into cell c of the grid: counted, and its id and (v,
// |v|) at the next place (counts start at zero).
__device__ __forceinline__ void bucket_vector(const RunView &R, int64_t j, int c, const double *v,
                                              double vn)
{
    const int k = atomicAdd(&R.gcnt[c], 1);
    const int places = bucket_places(R.K);
    if (k >= places) {
        R.gtot[2] = 1;
        return;
    }
    const int64_t p = (int64_t)c * places + k;
    R.gvec[p] = (int32_t)j;
    reinterpret_cast<double4 *>(R.gvh)[p] = make_double4(v[0], v[1], v[2], vn);
}

// share u of a direction x on the scaled simplex and its cell; -1 unless
// both components are >= 0 and finite with a positive sum
__device__ __forceinline__ int line_cell_of(double x0, double x1, const double *r, int G,
                                            double &u)
{
    const double a = x0 / r[0], b = x1 / r[1];
    const double s = a + b;
    u = b / s;
    if (!(a >= 0.0 && b >= 0.0 && s > 0.0 && s <= 1.79e308 && u >= 0.0 && u <= 1.0))
        return -1;
    const int c = (int)(u * G);
    return c < G ? c : G - 1;
}

}  // namespace rvea
