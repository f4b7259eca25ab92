// k_grid.hip -- association (Alg. 1, Eq. 2) through an index of the
// reference vectors, three objectives.
//
// The association of a row is the vector of largest cosine (lowest index on
// ties).  Here each row looks only at a short candidate list that provably
// holds that vector and every vector tied with it, and computes the binary64
// cosines of those candidates exactly as the full re-rank does, so the
// result is the same as a scan of all K vectors.
//
// Index.  A direction x >= 0 is mapped to the simplex point q of x / r
// (componentwise; r > 0 is the range vector of the last adaptation, scaled
// to max 1, so that the adapted lattice is again a uniform lattice in q) and
// q (its first two coordinates) to a cell of a G x G grid over [0, 1]^2.  A
// cell C is the square clipped to the simplex, a polygon of at most five
// vertices; the directions of the rows that land in C form the cone over
// that polygon (up to rounding).  Distances between directions are chord
// lengths |u - v| of unit vectors (a metric, monotone in the angle), so no
// inverse trigonometric function is needed.  For each cell, built whenever
// V changes:
//   u_c    the unit direction of the polygon's vertex mean; rho the largest
//          distance from u_c to a vertex (the largest to any point of the
//          cell: the distance to a fixed direction is quasi-convex on the
//          plane of q, so its maximum over the polygon is at a vertex)
//   b      an upper bound of the distance from any point of C to its nearest
//          vector: min over the vectors k of the cells around C of the largest
//          distance from a vertex to v_k (again attained at a vertex)
//   box    the (2 kStage + 1)^2 cells around C: its boundary (clipped to the
//          simplex) must be farther than b + rho from u_c: that ball around
//          u_c is convex in q, so it lies inside the box
//   P      the vectors within b + rho of u_c: a vector that is the nearest
//          for some row direction in C is within b of it, so it is among them
//   list   P without the vectors that a champion (a vector near a vertex or
//          u_c) beats at every vertex by more than 1e-12: the cosine
//          difference is linear on the cone, so such a vector loses to the
//          champion for every row direction in C, with a margin far above
//          binary64 rounding (any vector may serve as a champion, so they are
//          found from binary32 chords)
// Lists longer than kSlot, cells whose ball passes the box, cells with no
// vector in the box and cells near one with more
// vectors than places are marked for a full scan (correct for any
// vector set, counted as full rescans).  The same pass gives Eq. 5's gamma of
// the cell's vectors: from the staged neighbourhood where that provably holds
// the nearest other vector (the nearest staged one is closer than the
// neighbourhood's boundary), else by a scan of all vectors.  A cell's vectors
// have fixed places and its list kSlot records; the order
// of a cell's vectors varies from build to build (no result depends on it).
// After an adaptation the rebuild is one kernel, the adaptation having put each
// vector into its cell; with ranges allocated to the cells, a fill and the full
// gamma pass's two kernels behind it (which exited at once) it was five, about
// 4.5 us each beside the cells' own time.
//
// Two objectives.  The index is a line: a direction x >= 0 maps to its share
// u = (x1 / r1) / (x0 / r0 + x1 / r1) of the scaled simplex (u = j / H for
// the adapted lattice again) and u to one of G = K equal cells.  In the
// quadrant the angle of a direction is monotone in u, so a row needs no
// candidate list: it scans its own cell and the cells on either side, then
// keeps stepping outward on a side while the cosine to the direction of that
// side's next cell boundary (moved outward by far more than u's rounding)
// is not below the best cosine found by more than 1e-12.  Every vector
// beyond that boundary has a smaller cosine than the boundary direction, so
// the vector of largest cosine and all vectors tied with it have been seen.
// A walk past kLineWalk cells on a side, or any vector outside the quadrant
// (which the bucket leaves out and flags), makes the row scan all vectors
// (counted).  Eq. 5's gamma of each vector comes from the same walk, with
// the vector as the row, itself and the vectors parallel to it skipped, or past
// the limit from a scan of all vectors by its wavefront.
#include <algorithm>

#include "rvea_dev.h"
#include "rvea_index.h"
#include "rvea_internal.h"

namespace rvea {

constexpr int kSlot = 24;      // list records per cell (longer lists: a full scan)
constexpr int kChamps = 6;     // champions per cell: five vertices and the centre
constexpr int kGridRowLanes = 4;  // lanes per row of the association
constexpr double kDomMargin = 1e-12;
// Vectors that a scan for gamma takes at once, the most that leaves the kernel six
// wavefronts per SIMD without spills: with eight the shared scans of 100,128
// vectors take 2.7 ms instead of 4.0, but every rebuild pays for it.
constexpr int kScan = 4;
constexpr int kGammaLanes = 4;    // lanes per vector of the line's gamma
constexpr int kKeepGamma = 2;     // gate of a build that leaves gamma as it is
// Scaling below which the launch shares the scans for gamma: from about there on
// cells are too flat for their neighbourhoods to hold the nearest vector, and most
// vectors are left.  An adaptation of 100,128 vectors takes 4.0 ms shared, and
// with each cell scanning its own 0.65 at ranges 1 : 0.15 : 0.15, 5.4 at
// 1 : 1 : 0.1 and 7.8 at 1 : 1e-4 : 1e-4; 10,011 vectors 78 us, and 88, 111 and 112.
constexpr double kFlat = 0.125;

struct D3 {
    double x, y, z;
};
__device__ __forceinline__ D3 d3(double x, double y, double z) { return D3{x, y, z}; }
__device__ __forceinline__ double dot3(const D3 &a, const D3 &b)
{
    return a.x * b.x + a.y * b.y + a.z * b.z;
}
__device__ __forceinline__ D3 unit3(const D3 &a)
{
    const double inv = 1.0 / sqrt(dot3(a, a));
    return d3(a.x * inv, a.y * inv, a.z * inv);
}

// Binary32 versions for the geometric tests of the build.  Those tests only
// have to keep every possible candidate, so they run in single precision
// with hardware square root and reciprocal (1 ulp) and a slack kSlack on
// every comparison, far above their rounding (chords of unit vectors in
// [0, 2], each off by well under 1e-6); the tests that decide exclusion
// for good (domination) stay in binary64.
constexpr float kSlack = 4e-6f;
struct F3 {
    float x, y, z;
};
__device__ __forceinline__ F3 f3(float x, float y, float z) { return F3{x, y, z}; }
__device__ __forceinline__ F3 f3of(const D3 &a) { return F3{(float)a.x, (float)a.y, (float)a.z}; }
__device__ __forceinline__ float fdot(const F3 &a, const F3 &b)
{
    return a.x * b.x + a.y * b.y + a.z * b.z;
}
__device__ __forceinline__ F3 fsub(const F3 &a, const F3 &b) { return f3(a.x - b.x, a.y - b.y, a.z - b.z); }
__device__ __forceinline__ F3 fcross(const F3 &a, const F3 &b)
{
    return f3(a.y * b.z - a.z * b.y, a.z * b.x - a.x * b.z, a.x * b.y - a.y * b.x);
}
__device__ __forceinline__ float fsqrt(float x) { return __builtin_amdgcn_sqrtf(x); }
__device__ __forceinline__ F3 funit(const F3 &a)
{
    const float inv = __builtin_amdgcn_rcpf(fsqrt(fdot(a, a)));
    return f3(a.x * inv, a.y * inv, a.z * inv);
}
// unit direction of a record (v, |v|) for the geometric tests, from binary64 (a
// norm may be outside binary32's range); the hardware's reciprocal is off by less
// than 2^-24 (over 5e8 arguments of every size)
__device__ __forceinline__ F3 unit_of(const double4 &r)
{
    const double inv = __builtin_amdgcn_rcp(r.w);
    return f3((float)(r.x * inv), (float)(r.y * inv), (float)(r.z * inv));
}
// squared chord, and the chord (minima and maxima of chords are taken on
// the squares, with one square root at the end: the square root is
// monotone, so the result moves by at most its last-bit rounding)
__device__ __forceinline__ float fchord2(const F3 &a, const F3 &b)
{
    const F3 d = fsub(a, b);
    return fdot(d, d);
}
__device__ __forceinline__ float fchord(const F3 &a, const F3 &b) { return fsqrt(fchord2(a, b)); }
__device__ float farc_chord(const F3 &u, const F3 &a, const F3 &b, const F3 &n, bool valid)
{
    const float ends2 = fminf(fchord2(u, a), fchord2(u, b));
    if (!valid) return fsqrt(ends2);
    const float un = fdot(u, n);
    const F3 w = f3(u.x - un * n.x, u.y - un * n.y, u.z - un * n.z);
    const float wn = fsqrt(fdot(w, w));
    if (wn > 0.0f && fdot(fcross(a, w), n) >= 0.0f && fdot(fcross(w, b), n) >= 0.0f)
        return fsqrt(fminf(ends2, 2.0f * un * un * __builtin_amdgcn_rcpf(1.0f + wn)));
    return fsqrt(ends2);
}
__device__ float farc_chord_of(const F3 &u, const F3 &A, const F3 &B)
{
    const F3 a = funit(A), b = funit(B);
    const F3 n = fcross(a, b);
    const float nn = fsqrt(fdot(n, n));
    const bool valid = nn > 1e-30f;
    const float inv = valid ? __builtin_amdgcn_rcpf(nn) : 0.0f;
    return farc_chord(u, a, b, f3(n.x * inv, n.y * inv, n.z * inv), valid);
}
__device__ __forceinline__ F3 flift(float q1, float q2, const double *r)
{
    return f3((float)r[0] * q1, (float)r[1] * q2, (float)r[2] * (1.0f - q1 - q2));
}

// the direction of simplex point (q1, q2) scaled back by r
__device__ __forceinline__ D3 lift(double q1, double q2, const double *r)
{
    return d3(r[0] * q1, r[1] * q2, r[2] * (1.0 - q1 - q2));
}


// One cell's geometry, held in LDS by the cell's workgroup: the square
// [a, a+h] x [b, b+h] clipped to q1 + q2 <= 1 as five vertices in order
// (with corner sums s0 <= s1 = s3 <= s2: the whole square when s2 <= 1, a
// pentagon when only the far corner is cut, a triangle (or a point) when
// s1 > 1; fewer distinct vertices repeat the last) and their mean u_c after
// them: unit directions in binary64 (domination) and binary32 (the geometric
// tests), and rho.
constexpr int kNv = 5;
struct CellGeo {
    double X[kNv + 1][3];
    float Xf[kNv + 1][3];
    float rho;
};

__device__ __forceinline__ F3 ld3(const float (&a)[3]) { return f3(a[0], a[1], a[2]); }
__device__ __forceinline__ D3 ld3(const double (&a)[3]) { return d3(a[0], a[1], a[2]); }

// the cell's vertex v (v < kNv) in q, for a cell (ci, cj) with ci + cj <= G
// (its corner (a, b) on or below the diagonal; at ci + cj = G all five are
// that corner, up to rounding)
__device__ __forceinline__ void cell_vertex(int G, int c, int v, double &px, double &py)
{
    const double h = 1.0 / G;
    const double a = (c / G) * h, b = (c % G) * h;
    const double s1 = a + h + b, s2 = a + b + 2.0 * h;
    if (s2 <= 1.0) {  // the whole square
        const double x[kNv] = {a, a + h, a + h, a, a}, y[kNv] = {b, b, b + h, b + h, b + h};
        px = x[v];
        py = y[v];
    } else if (s1 <= 1.0) {  // the corner (a+h, b+h) cut off
        const double x[kNv] = {a, a + h, a + h, 1.0 - b - h, a};
        const double y[kNv] = {b, b, 1.0 - a - h, b + h, b + h};
        px = x[v];
        py = y[v];
    } else {  // only the corner (a, b) inside
        const double x[kNv] = {a, 1.0 - b, a, a, a}, y[kNv] = {b, b, 1.0 - a, 1.0 - a, 1.0 - a};
        px = x[v];
        py = y[v];
    }
}

// the geometry of a live cell, by the workgroup: lanes 0..4 the vertices,
// lane 5 u_c; then lanes 0..4 rho (as the bits of a non-negative float,
// combined by an LDS max)
__device__ void cell_geo(const RunView &R, int c, CellGeo &g, int lane)
{
    if (lane <= kNv) {
        double px = 0.0, py = 0.0;
        if (lane < kNv) {
            cell_vertex(R.gG, c, lane, px, py);
        } else {
            for (int v = 0; v < kNv; ++v) {
                double x, y;
                cell_vertex(R.gG, c, v, x, y);
                px += x;
                py += y;
            }
            px /= kNv;
            py /= kNv;
        }
        const D3 X = unit3(lift(px, py, R.gr));
        const F3 Xf = f3of(X);
        g.X[lane][0] = X.x;
        g.X[lane][1] = X.y;
        g.X[lane][2] = X.z;
        g.Xf[lane][0] = Xf.x;
        g.Xf[lane][1] = Xf.y;
        g.Xf[lane][2] = Xf.z;
    }
    if (lane == 0) g.rho = 0.0f;
    __syncthreads();
    if (lane < kNv)
        atomicMax(reinterpret_cast<unsigned int *>(&g.rho),
                  __float_as_uint(fchord(ld3(g.Xf[kNv]), ld3(g.Xf[lane]))));
    __syncthreads();
}

// first position of a range of n items allocated by the whole wavefront
// with one atomic add on *total (every lane active; lanes without items pass 0)
__device__ __forceinline__ int64_t wave_alloc(int n, unsigned long long *total)
{
    const int incl = wave_incl_scan(n);
    const int sum = __builtin_amdgcn_readlane(incl, 63);
    unsigned long long base = 0;
    if ((threadIdx.x & 63) == 0 && sum > 0) base = atomicAdd(total, (unsigned long long)sum);
    base = __shfl(base, 0, 64);
    return (int64_t)base + incl - n;
}

// ------------------------------------------------------------- line
constexpr int kLineWalk = 64;        // cells a row steps outward on a side at most
constexpr double kLineEps = 1e-12;   // outward shift of a boundary's u
constexpr double kLineTau = 1e-12;   // cosine margin of the stopping test


// binary64 cosine of f (norm nrm) and the direction of share u
__device__ __forceinline__ double line_bound(double f0, double f1, double nrm, double u,
                                             const double *r)
{
    const double b0 = (1.0 - u) * r[0], b1 = u * r[1];
    return (f0 * b0 + f1 * b1) / (nrm * sqrt(b0 * b0 + b1 * b1));
}

// ------------------------------------------------------------- build
// vectors into the grid's cells, or counted into the line's (counts start at
// zero); a rebuild after an adaptation skips this pass, the adaptation having
// done it for each vector as it wrote it (k_vectors.hip)
__device__ __forceinline__ void grid_bucket_body(const RunView &R, int64_t bx)
{
    const int64_t j = bx * 256 + threadIdx.x;
    if (j == 0 && R.m != 3) R.gtot[1] = 0;  // no vector outside the line (yet)
    if (j >= R.K) return;
    if (R.m == 3) {
        const int c = cell_of(R.V[j * 3], R.V[j * 3 + 1], R.V[j * 3 + 2], R.gr, R.gG);
        bucket_vector(R, j, c < 0 ? 0 : c, R.V + j * 3, R.vn[j]);
        return;
    }
    double u;
    const int c = line_cell_of(R.V[j * 2], R.V[j * 2 + 1], R.gr, R.gG, u);
    R.gcell[j] = c;
    if (c >= 0) atomicAdd(&R.gcnt[c], 1);
}

// line: each cell's range of positions (one atomic add per wavefront); the
// counts become the fill cursors, counting down to zero
__device__ __forceinline__ void grid_ranges_body(const RunView &R, int64_t bx, int gate)
{
    if (!gate && *R.vchanged == 0) return;
    const int64_t c = bx * 256 + threadIdx.x;
    const int64_t cells = index_cells(R.m, R.gG);
    const int n = c < cells ? R.gcnt[c] : 0;
    const int64_t st = wave_alloc(n, &R.gtot[0]);
    if (c < cells) {
        R.gstart[c] = (int32_t)st;
        R.gnum[c] = n;
    }
}

// line: vectors into their cells' ranges, with (v, |v|); the range allocator
// cleared
__device__ __forceinline__ void grid_fill_body(const RunView &R, int64_t bx, int gate)
{
    if (!gate && *R.vchanged == 0) return;
    const int64_t j = bx * 256 + threadIdx.x;
    if (j == 0) R.gtot[0] = 0;
    if (j >= R.K) return;
    const int c = R.gcell[j];
    if (c < 0) {  // outside the line: every row scans all vectors
        R.gtot[1] = 1;
        return;
    }
    const int64_t p = R.gstart[c] + atomicSub(&R.gcnt[c], 1) - 1;
    R.gvec[p] = (int32_t)j;
    reinterpret_cast<double4 *>(R.gvh)[p] = make_double4(R.V[j * 2], R.V[j * 2 + 1], 0.0, R.vn[j]);
}

// Wavefront-wide minimum / best (largest value, lowest id on ties) over
// the 64 lanes (every lane active): the pairings of partner32 within each
// half, then the two halves' results read out and combined (the result is
// uniform).
__device__ __forceinline__ double wave_fmin(double v)
{
    v = fmin(v, partner32<0>(v));
    v = fmin(v, partner32<1>(v));
    v = fmin(v, partner32<2>(v));
    v = fmin(v, partner32<3>(v));
    v = fmin(v, partner32<4>(v));
    RVEA_ASSERT_FULL_WAVE();
    const double a = __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), 0),
                                      __builtin_amdgcn_readlane(__double2loint(v), 0));
    const double b = __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), 32),
                                      __builtin_amdgcn_readlane(__double2loint(v), 32));
    return fmin(a, b);
}
__device__ __forceinline__ double first_lane(double v)
{
    return __hiloint2double(__builtin_amdgcn_readfirstlane(__double2hiint(v)),
                            __builtin_amdgcn_readfirstlane(__double2loint(v)));
}

// The cosine of Eq. 5's gamma of up to kScan vectors by the whole wavefront, those
// whose ids the lowest lanes of `mask` hold, into these lanes: the largest binary64
// cosine to another vector that is not parallel to it, over all vectors (as the
// full gamma pass computes it).
// The vectors themselves are scalars; a loaded vector serves all, and a cosine
// is divided out only where it may be above the best so far.  The 64 vectors
// around the id come first: in a lattice they hold its nearest or nearly so, and
// few divisions are left.
template <int M>
__device__ __forceinline__ void gamma_block(const double *V, const double *vn, int64_t K,
                                            unsigned long long mask, int32_t id, int lane, double &cosine)
{
    constexpr int B = kScan;
    int32_t ids[B], at[B];
    double vi[B][M], vni[B], best[B];
#pragma unroll
    for (int b = 0; b < B; ++b) {  // the last one again where the mask has fewer
        at[b] = b == 0 || mask ? __ffsll(mask) - 1 : at[b > 0 ? b - 1 : 0];
        ids[b] = __builtin_amdgcn_readlane(id, at[b]);
        mask &= mask - 1;
#pragma unroll
        for (int k = 0; k < M; ++k) vi[b][k] = first_lane(V[(int64_t)ids[b] * M + k]);
        vni[b] = first_lane(vn[ids[b]]);
    }
    auto dot = [&](int b, const double (&w)[M]) {
        double s = vi[b][0] * w[0];
#pragma unroll
        for (int k = 1; k < M; ++k) s = fma(vi[b][k], w[k], s);
        return s;
    };
    // a bound that s / n exceeds if its cosine is above the best so far, whatever
    // the rounding of the products
    auto below = [](double x) { return x - fabs(x) * 0x1p-50; };
    double low[B];
#pragma unroll
    for (int b = 0; b < B; ++b) {
        const int64_t j = (int64_t)ids[b] - 32 + lane;
        best[b] = -INFINITY;
        if (j >= 0 && j < K && j != ids[b]) {
            double w[M];
#pragma unroll
            for (int k = 0; k < M; ++k) w[k] = V[j * M + k];
            const double cv = dot(b, w) / (vni[b] * vn[j]);
            if (cv < 1.0) best[b] = cv;
        }
        best[b] = -wave_fmin(-best[b]);
        low[b] = below(best[b] * vni[b]);
    }
#pragma unroll 1
    for (int64_t j = lane; j < K; j += 64) {
        double w[M];
#pragma unroll
        for (int k = 0; k < M; ++k) w[k] = V[j * M + k];
        const double n = vn[j];
        bool any = false;
#pragma unroll
        for (int b = 0; b < B; ++b) any |= fma(-low[b], n, dot(b, w)) > 0.0;
        if (!any) continue;
#pragma unroll
        for (int b = 0; b < B; ++b) {
            const double s = dot(b, w);
            if (!(fma(-low[b], n, s) > 0.0) || j == ids[b]) continue;
            const double cv = s / (vni[b] * n);
            if (cv < 1.0 && cv > best[b]) {
                best[b] = cv;
                low[b] = below(cv * vni[b]);
            }
        }
    }
#pragma unroll
    for (int b = 0; b < B; ++b) {
        const double v = -wave_fmin(-best[b]);
        if (lane == at[b]) cosine = v;
    }
}

// the angle of that cosine; pi/2 without another vector
__device__ __forceinline__ double gamma_of(double cosine)
{
    return cosine > -INFINITY ? acos(cosine < -1.0 ? -1.0 : cosine) : 1.5707963267948966;
}

// the lanes left after a block took its kScan lowest
__device__ __forceinline__ unsigned long long past_block(unsigned long long mask)
{
#pragma unroll
    for (int b = 0; b < kScan; ++b) mask &= mask - 1;
    return mask;
}

// The vectors of the (2 kStage + 1)^2 cells around a cell, staged in LDS by
// its workgroup: the list record (v, |v|) and the id.  kStageCap entries at
// most, kStageLane per lane.
constexpr int kStage = 4;
constexpr int kStageW = 2 * kStage + 1;
constexpr int kStageLane = 3, kStageCap = 64 * kStageLane;
struct Stage {
    double4 rec[kStageCap];
    int32_t j[kStageCap];
};

// distance from unit u to side `side` (0..3) of the box of cells of radius
// kStage around (ci, cj), clipped to the simplex; a side on the grid's edge,
// where the simplex ends, does not count.  The sides are exact grid lines in
// binary64 (their ends on the simplex's edge), lifted in binary32, so the
// callers compare it with their slack
__device__ float box_side(const RunView &R, int ci, int cj, int side, const F3 &u)
{
    const int G = R.gG;
    const int i0 = max(0, ci - kStage), i1 = min(G - 1, ci + kStage);
    const int j0 = max(0, cj - kStage), j1 = min(G - 1, cj + kStage);
    const double h = 1.0 / G;
    const bool first = side < 2, low = (side & 1) == 0;  // a line of q1 or q2; the lower one
    const int line = low ? (first ? i0 : j0) : (first ? i1 + 1 : j1 + 1);
    const double at = line * h, from = (first ? j0 : i0) * h;
    const double to = fmin(((first ? j1 : i1) + 1) * h, 1.0 - at);
    if (!(low ? line > 0 : line < G) || to < from) return INFINITY;
    const F3 a = first ? flift((float)at, (float)from, R.gr) : flift((float)from, (float)at, R.gr);
    const F3 b = first ? flift((float)at, (float)to, R.gr) : flift((float)to, (float)at, R.gr);
    return farc_chord_of(u, a, b);
}

// One wavefront per cell (the simplex's cells only, in row order): the
// neighbourhood staged in LDS; each lane's three entries in binary32 registers
// with their squared chords to the five vertices and u_c, which serve b, P and
// the champions; the list from P, written into the cell's slot at each lane's
// prefix.
// A neighbourhood over kStageCap vectors or with a cell over its places, or a ball
// of radius b + rho that leaves it, marks the cell for a full scan.
// Bound by vector instructions at four wavefronts per SIMD: with exact distances
// to the cell's edges, the smallest of five boxes, binary64 champions and the
// vertex products formed per (entry, champion), it took 56 us at 10,011 vectors
// and 432 at 100,128; 26 and 162 so, with lists of the same length.
__device__ __forceinline__ void grid_cells_body(const RunView &R, int64_t bx, int gate)
{
    if (!gate && *R.vchanged == 0) return;
    const int G = R.gG;
    const int lane = threadIdx.x;
    if (bx >= index_cells(3, G)) return;  // uniform
    int ci = 0;  // the row of cell bx: the last row starting at or before it
    for (int hi = G - 1; ci < hi;) {
        const int mid = (ci + hi + 1) >> 1;
        if ((int64_t)grid_row(G, mid) <= bx) ci = mid; else hi = mid - 1;
    }
    const int cj = (int)(bx - grid_row(G, ci));
    const int64_t c = bx;
    __shared__ CellGeo g;
    __shared__ double champ[kChamps][kNv];  // products of the champions and the vertices
    __shared__ Stage st;
    // stage: each lane's cells of the neighbourhood, their vector counts
    // scanned over the wave, then the vectors
    const int places = bucket_places(R.K);
    int cnt[2] = {0, 0}, from[2] = {0, 0};
    bool over = false;
#pragma unroll
    for (int u = 0; u < 2; ++u) {
        const int t = lane + 64 * u;
        if (t < kStageW * kStageW) {
            const int i = ci - kStage + t / kStageW, jj = cj - kStage + t % kStageW;
            if (i >= 0 && i < G && jj >= 0 && jj < G && i + jj <= G) {
                const int near = (int)(grid_row(G, i) + (uint32_t)jj);
                from[u] = near * places;
                cnt[u] = R.gcnt[near];
                over = over || cnt[u] > places;
            }
        }
    }
    constexpr int own = kStage * kStageW + kStage;  // the centre cell's lane
    const int own_cnt = __builtin_amdgcn_readlane(cnt[0], own);
    const bool crowded = __any(over);
    const int mine0 = crowded ? 0 : cnt[0] + cnt[1];
    const int incl0 = wave_incl_scan(mine0);
    const int nst = __builtin_amdgcn_readlane(incl0, 63);
    cell_geo(R, ci * G + cj, g, lane);
    bool full = crowded || nst > kStageCap;
    if (!full) {
        int q = incl0 - mine0;
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            for (int k = 0; k < cnt[u]; ++k, ++q) {
                const int p = from[u] + k;
                st.j[q] = R.gvec[p];
                st.rec[q] = reinterpret_cast<const double4 *>(R.gvh)[p];
            }
        }
    }
    __syncthreads();
    const F3 uc = ld3(g.Xf[kNv]);
    const float rho = g.rho;
    // the least distance from u_c to the box's boundary, a side per lane
    float bsm = lane < 4 && !full ? box_side(R, ci, cj, lane, uc) : INFINITY;
    bsm = __uint_as_float(wave_min(__float_as_uint(bsm)));  // not negative: ordered as bits
    // this lane's entries: unit directions, squared chords to the vertices and
    // u_c (infinite without an entry)
    F3 vf[kStageLane];
    float c2[kStageLane][kNv + 1];
#pragma unroll
    for (int u = 0; u < kStageLane; ++u) {
        const int q = lane + 64 * u;
        const bool has = !full && q < nst;
        const double4 r = st.rec[has ? q : 0];
        vf[u] = unit_of(r);
#pragma unroll
        for (int e = 0; e <= kNv; ++e) c2[u][e] = has ? fchord2(ld3(g.Xf[e]), vf[u]) : INFINITY;
    }
    // Eq. 5's gamma of the cell's own vectors: the largest binary64 cosine
    // to another vector that is not parallel to it (cosine below 1, as the
    // full pass computes it), kept when the staged neighbourhood provably
    // holds that vector (the nearest staged one is closer than the
    // neighbourhood's boundary: every own vector lies within rho of u_c, so
    // its distance to that boundary is at least u_c's less rho); otherwise
    // by a scan of all vectors.  Where many are to be expected (a cell with more
    // vectors than places, flat scaling) the whole launch shares them evenly, so
    // that no cell's are one wavefront's: 10,011 vectors of ranges 1 : 1e-3 : 1e-3
    // under unit scaling took 223 ms with each cell scanning its own, one after the
    // other, 0.28 so.
    const bool shared = R.gtot[2] != 0 || fmin(R.gr[0], fmin(R.gr[1], R.gr[2])) < kFlat;
    // this lane's vector and its cosine, and the lanes left to scans at the end
    int32_t gid = -1;
    double gcos = 0.0;
    unsigned long long left = 0;
    if (gate == kKeepGamma) {
    } else if (shared) {  // a scan for each of up to half of the workgroups
        const int64_t first = kScan * bx;
        if (lane < kScan && first + lane < R.K) gid = (int32_t)(first + lane);
        left = __ballot(gid >= 0);
    } else if (full) {  // no crowded cell: at most its places
        if (lane < own_cnt) gid = R.gvec[c * places + lane];
        left = __ballot(gid >= 0);
    } else {
        const int oq0 = __builtin_amdgcn_readlane(incl0 - mine0, own);
        const int on = own_cnt;
        const float lo = bsm - rho - kSlack;
        bool gok = false;
        for (int o = oq0; o < oq0 + on; ++o) {  // uniform
            const double4 v = st.rec[o];
            const F3 ui = unit_of(v);
            double gb = -INFINITY;
            float dmin = INFINITY;  // squared
#pragma unroll
            for (int u = 0; u < kStageLane; ++u) {
                const int q = lane + 64 * u;
                if (q >= nst || q == o) continue;
                const double4 w = st.rec[q];
                double sd = v.x * w.x;
                sd = fma(v.y, w.y, sd);
                sd = fma(v.z, w.z, sd);
                const double cv = sd / (v.w * w.w);
                if (cv >= 1.0) continue;
                gb = fmax(gb, cv);
                dmin = fminf(dmin, fchord2(ui, vf[u]));
            }
            gb = -wave_fmin(-gb);
            dmin = fsqrt(__uint_as_float(wave_min(__float_as_uint(dmin))));
            const bool ok = dmin < INFINITY && lo > dmin + 2.0f * kSlack;
            if (lane == o - oq0) {
                gcos = gb;
                gok = ok;
            }
        }
        if (lane < on) gid = st.j[oq0 + lane];
        left = __ballot(lane < on && !gok);
    }
    // b: the vector that covers the cell best
    float cover = INFINITY;
#pragma unroll
    for (int u = 0; u < kStageLane; ++u) {
        float far = c2[u][0];
#pragma unroll
        for (int e = 1; e < kNv; ++e) far = fmaxf(far, c2[u][e]);
        cover = fminf(cover, far);
    }
    cover = fsqrt(__uint_as_float(wave_min(__float_as_uint(cover))));
    const float ball = cover + kSlack + rho + 2.0f * kSlack;  // b + rho and the comparisons' slack
    full = full || !(cover < INFINITY) || !(bsm > ball);
    if (!full) {
        // P, and the champions: for each vertex and u_c the entry of P with the
        // least squared chord, its last 8 bits replaced by the entry's number
        const float lim = ball * ball * 1.000002f;
        uint32_t key[kChamps];
#pragma unroll
        for (int d = 0; d < kChamps; ++d) key[d] = 0xffffffffu;
#pragma unroll
        for (int u = 0; u < kStageLane; ++u) {
            const bool in = c2[u][kNv] <= lim;
#pragma unroll
            for (int d = 0; d < kChamps; ++d) {
                const uint32_t k = (__float_as_uint(c2[u][d]) & ~0xffu) | (uint32_t)(lane + 64 * u);
                key[d] = in ? min(key[d], k) : key[d];
            }
        }
        int mine_d = -1;  // the champion of this lane's (champion, vertex) pair
#pragma unroll
        for (int d = 0; d < kChamps; ++d) {
            const uint32_t k = wave_min(key[d]);
            if (lane / kNv == d && k != 0xffffffffu) mine_d = (int)(k & 0xffu);
        }
        if (lane < kChamps * kNv) {
            double p = -INFINITY;
            if (mine_d >= 0) {
                const double4 r = st.rec[mine_d];
                const double inv = 1.0 / r.w;
                p = dot3(ld3(g.X[lane % kNv]), d3(r.x * inv, r.y * inv, r.z * inv));
            }
            champ[lane / kNv][lane % kNv] = p;
        }
        __syncthreads();
        // the list: members that no champion beats at every vertex (a champion
        // does not beat itself)
        uint32_t keep = 0;
        int mine = 0;
#pragma unroll
        for (int u = 0; u < kStageLane; ++u) {
            if (c2[u][kNv] <= lim) {
                const double4 r = st.rec[lane + 64 * u];
                const double inv = 1.0 / r.w;
                const D3 v = d3(r.x * inv, r.y * inv, r.z * inv);
                double x[kNv];
#pragma unroll
                for (int e = 0; e < kNv; ++e) x[e] = dot3(ld3(g.X[e]), v) + kDomMargin;
                bool beaten = false;
#pragma unroll
                for (int d = 0; d < kChamps; ++d) {
                    bool all = true;
#pragma unroll
                    for (int e = 0; e < kNv; ++e) all = all && champ[d][e] > x[e];
                    beaten = beaten || all;
                }
                if (!beaten) {
                    keep |= 1u << u;
                    ++mine;
                }
            }
        }
        const int incl = wave_incl_scan(mine);
        const int n = __builtin_amdgcn_readlane(incl, 63);
        full = n > kSlot;
        // the cell's records in its own slot, each lane at its prefix
        const int64_t base = c * kSlot;
        if (!full) {
            int64_t o = base + incl - mine;
#pragma unroll
            for (int u = 0; u < kStageLane; ++u) {
                if (!((keep >> u) & 1u)) continue;
                const int q = lane + 64 * u;
                reinterpret_cast<double4 *>(R.lrec)[o] = st.rec[q];
                R.lidx[o] = st.j[q];
                ++o;
            }
            if (lane == 0) R.lcnt[c] = n;
        }
    }
    if (full && lane == 0) R.lcnt[c] = -1;
    for (; left; left = past_block(left)) gamma_block<3>(R.V, R.vn, R.K, left, gid, lane, gcos);
    if (gid >= 0) R.gamma[gid] = gamma_of(gcos);
}

// ----------------------------------------------------------- association
// kGridRowLanes lanes per merged row: f' = F - z* in binary64 and |f'| as
// the re-rank forms them, the row's cell, the binary64 cosines of the
// cell's list (or of every vector for a cell marked for a full scan), the
// best with the lowest index on ties, then as the re-rank: angle, APD of
// Eq. 4 and the per-vector minimum of (APD, row).
__device__ __forceinline__ void assoc_grid_body(const RunView &R, int64_t bx)
{
    const int sub = threadIdx.x % kGridRowLanes;
    const int64_t i = (bx * 256 + threadIdx.x) / kGridRowLanes;
    const bool in = i < R.M;
    const int64_t pop = *R.t_done;
    const uint32_t *zb = zbuf(R, pop + 1);
    const float *Fm = fm_of(R, pop);
    float rf[3] = {0.f, 0.f, 0.f};
    if (in)
        for (int k = 0; k < 3; ++k) rf[k] = Fm[i * 3 + k];
    const bool act = in && R.mvalid[i];
    double f[3];
    for (int k = 0; k < 3; ++k) {
        const float zk = ord_dec(zb[k]);
        f[k] = act ? (double)rf[k] - (double)zk : 0.0;
    }
    double n2 = f[0] * f[0];
    n2 = fma(f[1], f[1], n2);
    n2 = fma(f[2], f[2], n2);
    const double nrm = sqrt(n2);
    const bool live = act && nrm > 0.0;
    // the cell's list: its length and, beside it (the cell's slot is at a
    // fixed place, whatever it holds), this lane's first two records
    int32_t n = 0;
    int64_t st = 0;
    double4 v0 = make_double4(0.0, 0.0, 0.0, 1.0), v1 = v0;
    int32_t j0 = 0, j1 = 0;
    const double4 *rec = reinterpret_cast<const double4 *>(R.lrec);
    if (live) {
        const int c = cell_of(f[0], f[1], f[2], R.gr, R.gG);
        if (c >= 0) {
            st = (int64_t)c * kSlot;
            n = R.lcnt[c];
            v0 = rec[st + sub];
            j0 = R.lidx[st + sub];
            v1 = rec[st + sub + kGridRowLanes];
            j1 = R.lidx[st + sub + kGridRowLanes];
        }
    }
    const bool full = live && n <= 0;
    // the best cosine, its vector and that vector's gamma (loaded with the
    // candidate, so the APD needs no further round trip)
    double best = -INFINITY, bg = 0.0;
    int64_t bj = R.K;
    if (live && !full) {
        for (int e = sub; e < n; e += kGridRowLanes) {
            const bool third = e >= 2 * kGridRowLanes;
            const double4 v = e == sub ? v0 : third ? rec[st + e] : v1;
            const int64_t j = e == sub ? j0 : third ? R.lidx[st + e] : j1;
            const double gj = R.gamma[j];
            double s = f[0] * v.x;
            s = fma(f[1], v.y, s);
            s = fma(f[2], v.z, s);
            const double cv = s / (nrm * v.w);
            if (cv > best || (cv == best && j < bj)) {
                best = cv;
                bj = j;
                bg = gj;
            }
        }
    } else if (full) {
        for (int64_t j = sub; j < R.K; j += kGridRowLanes) {
            double s = f[0] * R.V[j * 3];
            s = fma(f[1], R.V[j * 3 + 1], s);
            s = fma(f[2], R.V[j * 3 + 2], s);
            const double cv = s / (nrm * R.vn[j]);
            if (cv > best || (cv == best && j < bj)) {
                best = cv;
                bj = j;
                bg = R.gamma[j];
            }
        }
    }
    // the row's four lanes are a quad: combine them by the quad swaps of
    // partner32 (every lane active)
    static_assert(kGridRowLanes == 4, "rows are quads");
    {
        double ob = partner32<0>(best), og = partner32<0>(bg);
        int64_t oj = partner32<0>(bj);
        if (ob > best || (ob == best && oj < bj)) {
            best = ob;
            bj = oj;
            bg = og;
        }
        ob = partner32<1>(best);
        og = partner32<1>(bg);
        oj = partner32<1>(bj);
        if (ob > best || (ob == best && oj < bj)) {
            best = ob;
            bj = oj;
            bg = og;
        }
    }
    if (!in || sub != 0) return;
    if (!act) {
        R.assoc[i] = -1;
        R.apd[i] = INFINITY;
        return;
    }
    if (!live) {  // the row is the ideal point: vector 0, APD 0
        R.assoc[i] = 0;
        R.apd[i] = 0.0;
        atomicMin(&key_of(R, pop + 1)[0], (unsigned long long)i);
        return;
    }
    if (full) atomicAdd(&R.counters[1], 1ull);
    const double gj = bj < R.K ? bg : R.gamma[0];
    if (bj >= R.K) bj = 0;
    const double cc = best > 1.0 ? 1.0 : (best < -1.0 ? -1.0 : best);
    const double th = acos(cc);
    const double a = (1.0 + *R.pen * th / gj) * nrm;
    R.assoc[i] = (int32_t)bj;
    R.apd[i] = a;
    const unsigned long long ab = (unsigned long long)__double_as_longlong(a);
    atomicMin(&key_of(R, pop + 1)[bj], ((ab >> R.kb) << R.kb) | (unsigned long long)i);
}

// L = 4 or 1 lanes per merged row (two objectives): f' and |f'| as the
// re-rank forms them, the row's cell on the line, that cell and its neighbours (of
// four lanes at once: lane 0 the row's own, lanes 1 and 2 two cells of a side
// each), then the walk outward on both sides (or a scan of every vector if a walk
// is too long or the line incomplete), then as the re-rank: angle, APD of Eq. 4
// and the per-vector minimum of (APD, row).  Bound by its chain of memory round
// trips and binary64 divisions: one lane per row takes the cells one after the
// other, 10.8 us at 10,000 rows (8.6 at 8,192 policies) against 9.0 (6.0).
//
// From 100,000 to 350,000 rows the launch is bound by issue instead, and one lane
// per row has a quarter of the wavefronts to issue for (200,000 rows: 14.1 us,
// four lanes 16.5; 320,000: 22.4 and 23.3).  With more rows the walks' loads miss
// the L2 cache and four lanes have more of them in flight (400,000: 28.3 us, one
// lane 33.6).
__host__ __device__ __forceinline__ int line_lanes(int64_t rows)
{
    return rows >= 100000 && rows < 350000 ? 1 : kGridRowLanes;
}
template <int L>
__device__ __forceinline__ void line_combine(double &best, int64_t &bj)
{
    if (L == 1) return;
    double ob = partner32<0>(best);
    int64_t oj = partner32<0>(bj);
    if (ob > best || (ob == best && oj < bj)) {
        best = ob;
        bj = oj;
    }
    ob = partner32<1>(best);
    oj = partner32<1>(bj);
    if (ob > best || (ob == best && oj < bj)) {
        best = ob;
        bj = oj;
    }
}

template <int L>
__device__ __forceinline__ void assoc_line_body(const RunView &R, int64_t bx)
{
    const int sub = threadIdx.x % L;
    const int64_t i = (bx * 256 + threadIdx.x) / L;
    const bool in = i < R.M;
    const int64_t pop = *R.t_done;
    const uint32_t *zb = zbuf(R, pop + 1);
    const float *Fm = fm_of(R, pop);
    const float r0 = in ? Fm[i * 2] : 0.f, r1 = in ? Fm[i * 2 + 1] : 0.f;
    const bool act = in && R.mvalid[i];
    const bool outside = R.gtot[1] != 0;
    const double f0 = act ? (double)r0 - (double)ord_dec(zb[0]) : 0.0;
    const double f1 = act ? (double)r1 - (double)ord_dec(zb[1]) : 0.0;
    double n2 = f0 * f0;
    n2 = fma(f1, f1, n2);
    const double nrm = sqrt(n2);
    const bool live = act && nrm > 0.0;
    const int G = R.gG;
    const double *r = R.gr;
    double best = -INFINITY, u = 0.0;
    int64_t bj = R.K;
    const int c = live ? line_cell_of(f0, f1, r, G, u) : -1;
    bool full = live && (c < 0 || outside);
    const double4 *rec = reinterpret_cast<const double4 *>(R.gvh);
    auto take = [&](const double4 &v, int64_t j) {
        double s = f0 * v.x;
        s = fma(f1, v.y, s);
        const double cv = s / (nrm * v.w);
        if (cv > best || (cv == best && j < bj)) {
            best = cv;
            bj = j;
        }
    };
    auto scan = [&](int cc) {
        const int st = R.gstart[cc], n = R.gnum[cc];
        for (int e = 0; e < n; ++e) take(rec[st + e], R.gvec[st + e]);
    };
    const bool walk = live && !full;
    // `done` cells on a side taken: beyond those while the boundary direction
    // (moved outward by kLineEps in u) could still tie
    auto outward = [&](int side, int done) {
        int at = c + done * side, steps = done;
        while (at > 0 && at < G - 1 && !full) {
            const double edge = side < 0 ? (double)at / G + kLineEps : (double)(at + 1) / G - kLineEps;
            if (line_bound(f0, f1, nrm, edge, r) + kLineTau < best) break;
            at += side;
            scan(at);
            full = ++steps > kLineWalk;
        }
    };
    if constexpr (L == 1) {
        if (walk) {
            scan(c);
            if (c > 0) scan(c - 1);
            if (c < G - 1) scan(c + 1);
            outward(-1, 1);
            outward(1, 1);
        }
    } else {
        const int side = sub == 1 ? -1 : sub == 2 ? 1 : 0;
        if (walk && sub < 3) {
            // this lane's cells, their ranges read together, then their first
            // vectors together
            const int ca = c + side, cb = side == 0 ? -1 : c + 2 * side;
            const bool ha = ca >= 0 && ca < G, hb = cb >= 0 && cb < G;
            const int sa = ha ? R.gstart[ca] : 0, na = ha ? R.gnum[ca] : 0;
            const int sb = hb ? R.gstart[cb] : 0, nb = hb ? R.gnum[cb] : 0;
            const double4 va = rec[na > 0 ? sa : 0], vb = rec[nb > 0 ? sb : 0];
            const int32_t ja = R.gvec[na > 0 ? sa : 0], jb = R.gvec[nb > 0 ? sb : 0];
            if (na > 0) take(va, ja);
            if (nb > 0) take(vb, jb);
            for (int e = 1; e < na; ++e) take(rec[sa + e], R.gvec[sa + e]);
            for (int e = 1; e < nb; ++e) take(rec[sb + e], R.gvec[sb + e]);
        }
        line_combine<L>(best, bj);
        if (walk && side != 0) outward(side, 2);
        const int any = (int)full | partner32<0>((int)full);
        full = (any | partner32<1>(any)) != 0;  // of the row's lanes
    }
    if (full) {
        best = -INFINITY;
        bj = R.K;
        for (int64_t j = sub; j < R.K; j += L)
            take(make_double4(R.V[j * 2], R.V[j * 2 + 1], 0.0, R.vn[j]), j);
    }
    line_combine<L>(best, bj);
    if (!in || sub != 0) return;
    if (!act) {
        R.assoc[i] = -1;
        R.apd[i] = INFINITY;
        return;
    }
    if (!live) {  // the row is the ideal point: vector 0, APD 0
        R.assoc[i] = 0;
        R.apd[i] = 0.0;
        atomicMin(&key_of(R, pop + 1)[0], (unsigned long long)i);
        return;
    }
    if (full) atomicAdd(&R.counters[1], 1ull);
    if (bj >= R.K) bj = 0;
    const double gj = R.gamma[bj];
    const double cc = best > 1.0 ? 1.0 : (best < -1.0 ? -1.0 : best);
    const double th = acos(cc);
    const double a = (1.0 + *R.pen * th / gj) * nrm;
    R.assoc[i] = (int32_t)bj;
    R.apd[i] = a;
    const unsigned long long ab = (unsigned long long)__double_as_longlong(a);
    atomicMin(&key_of(R, pop + 1)[bj], ((ab >> R.kb) << R.kb) | (unsigned long long)i);
}

// Eq. 5's gamma of each vector on the line (by the first of kGammaLanes lanes,
// which leaves a wavefront few vectors to scan where walks fail): the walk
// of the association with the vector as the row, skipping itself and the
// vectors exactly parallel to it (binary64 cosine 1 or more), as the full
// gamma pass does; the largest cosine's angle (pi/2 without another
// vector).  A vector outside the line, or with a walk past kLineWalk cells on a
// side, is scanned against all vectors by the whole wavefront instead.
__device__ __forceinline__ void line_gamma_body(const RunView &R, int64_t bx, int gate)
{
    if (!gate && *R.vchanged == 0) return;
    const int64_t i = (bx * 256 + threadIdx.x) / kGammaLanes;
    const bool in = i < R.K && threadIdx.x % kGammaLanes == 0;
    const double f0 = in ? R.V[i * 2] : 1.0, f1 = in ? R.V[i * 2 + 1] : 0.0, nrm = in ? R.vn[i] : 1.0;
    const int G = R.gG;
    const double *r = R.gr;
    double u;
    const int c = line_cell_of(f0, f1, r, G, u);
    bool full = in && (c < 0 || R.gtot[1] != 0);
    const double4 *rec = reinterpret_cast<const double4 *>(R.gvh);
    double best = -INFINITY;
    auto scan = [&](int cc) {
        const int st = R.gstart[cc], n = R.gnum[cc];
        for (int e = 0; e < n; ++e) {
            if (R.gvec[st + e] == (int32_t)i) continue;
            const double4 v = rec[st + e];
            double s = f0 * v.x;
            s = fma(f1, v.y, s);
            const double cv = s / (nrm * v.w);
            if (cv >= 1.0) continue;
            best = fmax(best, cv);
        }
    };
    const bool walk = in && !full;
    if (walk) scan(c);
    int lo = c, hi = c, steps = 0;
    while (walk && lo > 0 && !full) {
        if (lo < c && line_bound(f0, f1, nrm, (double)lo / G + kLineEps, r) + kLineTau < best)
            break;
        scan(--lo);
        full = ++steps > kLineWalk;
    }
    steps = 0;
    while (walk && hi < G - 1 && !full) {
        if (hi > c && line_bound(f0, f1, nrm, (double)(hi + 1) / G - kLineEps, r) + kLineTau < best)
            break;
        scan(++hi);
        full = ++steps > kLineWalk;
    }
    // the wavefront's lanes again together: the vectors left
    for (unsigned long long left = __ballot(full); left; left = past_block(left))
        gamma_block<2>(R.V, R.vn, R.K, left, (int32_t)i, threadIdx.x & 63, best);
    if (in) R.gamma[i] = gamma_of(best);
}

// ------------------------------------------------------------- kernels
__global__ __launch_bounds__(256) void k_grid_clear(RunView R)
{
    clear_counts(R, (int64_t)blockIdx.x * 256 + threadIdx.x, (int64_t)gridDim.x * 256);
}
__global__ __launch_bounds__(256) void k_grid_bucket(RunView R) { grid_bucket_body(R, blockIdx.x); }
__global__ __launch_bounds__(256) void k_grid_ranges(RunView R, int gate)
{
    grid_ranges_body(R, blockIdx.x, gate);
}
__global__ __launch_bounds__(256) void k_grid_fill(RunView R, int gate)
{
    grid_fill_body(R, blockIdx.x, gate);
}
// (six wavefronts per SIMD, as without the scans for gamma)
__global__ __launch_bounds__(64, 6) void k_grid_cells(RunView R, int gate)
{
    grid_cells_body(R, blockIdx.x, gate);
}
__global__ __launch_bounds__(256) void k_assoc_grid(RunView R) { assoc_grid_body(R, blockIdx.x); }
template <int L>
__global__ __launch_bounds__(256) void k_assoc_line(RunView R) { assoc_line_body<L>(R, blockIdx.x); }
__global__ __launch_bounds__(256) void k_line_gamma(RunView R, int gate)
{
    line_gamma_body(R, blockIdx.x, gate);
}

// batched: blockIdx.x decoded into (run, local block) through the span
// table; the build phases run for the runs whose vectors changed
__global__ __launch_bounds__(256) void kb_grid_ranges(const RunView *runs, const Span *sp, int n)
{
    const int s = find_span(sp, n, blockIdx.x);
    grid_ranges_body(runs[sp[s].run], blockIdx.x - sp[s].start, 0);
}
__global__ __launch_bounds__(256) void kb_grid_fill(const RunView *runs, const Span *sp, int n)
{
    const int s = find_span(sp, n, blockIdx.x);
    grid_fill_body(runs[sp[s].run], blockIdx.x - sp[s].start, 0);
}
// one cell per workgroup: more per workgroup would keep more registers live
// in this heavy body, and it is the open generations' cost that matters here
__global__ __launch_bounds__(64, 6) void kb_grid_cells(const RunView *runs, const Span *sp, int n)
{
    const int s = find_span(sp, n, blockIdx.x);
    grid_cells_body(runs[sp[s].run], blockIdx.x - sp[s].start, 0);
}
// the indexed associations, m = 2 and 3 in one launch: neither fills the
// device for long (sixteen served runs: 9.3 and 9.6 us apart, 12.1 together)
__global__ __launch_bounds__(256) void kb_assoc_index(const RunView *runs, const Span *sp, int n)
{
    const int s = find_span(sp, n, blockIdx.x);
    const RunView &R = runs[sp[s].run];
    if (R.m == 3)
        assoc_grid_body(R, blockIdx.x - sp[s].start);
    else if (line_lanes(R.M) == 1)  // uniform
        assoc_line_body<1>(R, blockIdx.x - sp[s].start);
    else
        assoc_line_body<kGridRowLanes>(R, blockIdx.x - sp[s].start);
}
__global__ __launch_bounds__(256) void kb_line_gamma(const RunView *runs, const Span *sp, int n)
{
    const int s = find_span(sp, n, blockIdx.x);
    line_gamma_body(runs[sp[s].run], blockIdx.x - sp[s].start, 0);
}

// ------------------------------------------------------------- launchers
static int64_t line_gamma_blocks(const RunView &R) { return (R.K * kGammaLanes + 255) / 256; }

static hipError_t launch_grid_rest(const RunView &R, hipStream_t s, int gate)
{
    const unsigned vb = (unsigned)((R.K + 255) / 256);
    if (R.m == 3) {
        k_grid_cells<<<(unsigned)index_cells(3, R.gG), 64, 0, s>>>(R, gate);
    } else {
        k_grid_ranges<<<(unsigned)((R.gG + 255) / 256), 256, 0, s>>>(R, gate);
        k_grid_fill<<<vb, 256, 0, s>>>(R, gate);
        if (gate != kKeepGamma) k_line_gamma<<<(unsigned)line_gamma_blocks(R), 256, 0, s>>>(R, gate);
    }
    return hipGetLastError();
}

hipError_t launch_grid_build(const RunView &R, hipStream_t s, bool keep_gamma)
{
    if (R.gG <= 0) return hipSuccess;
    const unsigned vb = (unsigned)((R.K + 255) / 256);
    if (R.m == 3) k_grid_clear<<<vb, 256, 0, s>>>(R);
    k_grid_bucket<<<vb, 256, 0, s>>>(R);
    return launch_grid_rest(R, s, keep_gamma ? kKeepGamma : 1);
}

hipError_t launch_grid_rebuild(const RunView &R, hipStream_t s)
{
    return R.gG <= 0 ? hipSuccess : launch_grid_rest(R, s, 0);
}

hipError_t launch_assoc_grid(const RunView &R, hipStream_t s)
{
    const unsigned g = (unsigned)grid_phase_blocks(BP_ASSOC, R);
    if (R.m == 3)
        k_assoc_grid<<<g, 256, 0, s>>>(R);
    else
        (line_lanes(R.M) == 1 ? k_assoc_line<1> : k_assoc_line<kGridRowLanes>)<<<g, 256, 0, s>>>(R);
    return hipGetLastError();
}

hipError_t launch_batch_grid(int phase, int cls, const RunView *runs, const Span *sp, int n,
                             int64_t blocks, hipStream_t s)
{
    const dim3 g((unsigned)blocks);
    switch (phase) {
    case BP_ASSOC: kb_assoc_index<<<g, 256, 0, s>>>(runs, sp, n); break;
    case BP_GRID_RANGES: kb_grid_ranges<<<g, 256, 0, s>>>(runs, sp, n); break;
    case BP_GRID_FILL: kb_grid_fill<<<g, 256, 0, s>>>(runs, sp, n); break;
    case BP_GRID_CELLS:  // class: the objective count (3: cells, 2: the line's gamma)
        if (cls == 3)
            kb_grid_cells<<<g, 64, 0, s>>>(runs, sp, n);
        else
            kb_line_gamma<<<g, 256, 0, s>>>(runs, sp, n);
        break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

int64_t grid_phase_blocks(int phase, const RunView &R)
{
    if (R.gG <= 0) return 0;
    const int64_t cells = index_cells(R.m, R.gG);
    switch (phase) {
    case BP_ASSOC: return (R.M * (R.m == 3 ? kGridRowLanes : line_lanes(R.M)) + 255) / 256;
    case BP_GRID_FILL: return R.m == 3 ? 0 : (R.K + 255) / 256;
    case BP_GRID_RANGES: return R.m == 3 ? 0 : (cells + 255) / 256;
    case BP_GRID_CELLS: return R.m == 3 ? index_cells(3, R.gG) : line_gamma_blocks(R);
    }
    return 0;
}

int grid_slot() { return kSlot; }

int grid_side(int m, int64_t K)
{
    if (m == 2) return K < 2 ? 2 : (int)K;  // a line of K cells
    if (m != 3) return 0;
    int G = (int)ceil(1.0 * sqrt((double)K));
    return G < 2 ? 2 : G;
}

}  // namespace rvea
