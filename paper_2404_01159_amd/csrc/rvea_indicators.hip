// rvea_indicators.hip -- quality indicators of a population on the device:
// the hypervolume of App. C.2 (reference point ones on normalised
// objectives, m = 2 or 3) and the expected utility over a weight set (the
// neuroevolution appendix's EU).  Kernels and their C entry points.
//
// Hypervolume without a sequential sweep.  Order the counted points by their
// last objective z (ties by row).  The dominated volume is the integral over
// z of the area dominated in the first two objectives by the points at or
// below z, and that area grows by D_t, the part of point t's rectangle
// [x_t,1] x [y_t,1] not already covered by the rectangles of the points
// ordered before it, when t is reached.  Hence
//     HV = sum_t (1 - z_t) D_t,
// and every D_t is independent of the others:
//     D_t = integral over x in [x_t, 1] of max(0, Y_t(x) - y_t),
// with Y_t(x) the lowest y among the points before t whose x is at most x
// (1 if none).  With the points sorted once by x, Y_t at each point is a
// running minimum, so one wavefront per t integrates D_t in one pass over the
// sorted points: O(n^2) work in all, spread over n wavefronts, every term a
// product of non-negative differences.  For m = 2 every z is 0 and the order
// is the row order, so HV = sum_t D_t.  The x order is found by counting, for
// each point, the points before it in (x, row) order.
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdint>
#include <mutex>

#include "rvea.h"
#include "rvea_internal.h"

namespace {

constexpr int kMaxObj = 8;
constexpr int64_t kMaxRows = (int64_t)1 << 24;   // rows and weights of the expected utility
constexpr int64_t kMaxHvRows = (int64_t)1 << 18;  // rows of the hypervolume (O(n^2) work)

struct Norm {
    double lo[kMaxObj], inv[kMaxObj];  // f' = (f - lo) / (hi - lo), scale given as hi - lo
    int m;
};

// Workspace of the hypervolume for n rows: the normalised points by row
// (x, y, z), the points in x order (x, y, z, row) and each row's term;
// 256-byte aligned pieces (and one of the rows' size unused, so that the
// footprint callers sized their workspace by stays what it was).
struct HvSpace {
    double *px, *py, *pz;
    double *sx, *sy, *sz;
    int32_t *sk;
    double *term;
};

size_t up256(size_t b) { return (b + 255) / 256 * 256; }

size_t hv_bytes(int64_t n)
{
    const size_t nn = (size_t)(n > 0 ? n : 1);
    return 7 * up256(nn * 8) + 2 * up256(nn * 4);
}

HvSpace hv_space(void *ws, int64_t n)
{
    const size_t nn = (size_t)(n > 0 ? n : 1);
    char *p = (char *)ws;
    HvSpace S;
    auto take = [&](size_t b) {
        char *q = p;
        p += up256(b);
        return q;
    };
    S.px = (double *)take(nn * 8);
    S.py = (double *)take(nn * 8);
    S.pz = (double *)take(nn * 8);
    S.sx = (double *)take(nn * 8);
    S.sy = (double *)take(nn * 8);
    S.sz = (double *)take(nn * 8);
    S.sk = (int32_t *)take(nn * 4);
    S.term = (double *)take(nn * 8);
    return S;
}

// A row counts when it is marked valid (or no marks are given) and every
// objective is finite.
__device__ __forceinline__ bool row_counts(const float *F, const uint8_t *valid, int m,
                                           int64_t i)
{
    if (valid && !valid[i]) return false;
    for (int k = 0; k < m; ++k)
        if (!isfinite(F[i * m + k])) return false;
    return true;
}

// Normalised point of each row; a row that does not count, or that does not
// lie strictly inside the reference box, becomes (1, 1, 1), which neither
// adds volume nor covers any.
__global__ void k_hv_points(const float *F, const uint8_t *valid, int64_t n, Norm nm, HvSpace S)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    double p[3] = {1.0, 1.0, 0.0};
    bool in = row_counts(F, valid, nm.m, i);
    if (in) {
        for (int k = 0; k < nm.m; ++k) {
            p[k] = ((double)F[i * nm.m + k] - nm.lo[k]) / nm.inv[k];
            in = in && p[k] < 1.0;
        }
    }
    if (!in) p[0] = p[1] = p[2] = 1.0;
    S.px[i] = p[0];
    S.py[i] = p[1];
    S.pz[i] = p[2];
}

// x-rank of each row, the rows before it in (x, row) order, and the row
// written to its place in x order.  One workgroup counts kRankRows rows over
// all n: four threads take four rows each in registers, 256 groups of them
// every 256th k, so a loaded x serves four compares and the counts need no
// clearing and no device atomics (integer sums, any order).  Bound by the
// n^2 compares; rows before the workgroup's compare with <=, rows after with
// <, so that a pair costs one compare and one add.  10,011 rows: 21 us, where
// ranks by device atomics and a scatter pass took 50.
constexpr int kRankRows = 16;
__global__ __launch_bounds__(1024) void k_hv_order(int64_t n, HvSpace S)
{
    __shared__ int32_t total[kRankRows];
    if (threadIdx.x < kRankRows) total[threadIdx.x] = 0;
    const int64_t i0 = (int64_t)blockIdx.x * kRankRows;
    const int sub = threadIdx.x & 3, kl = threadIdx.x >> 2;
    double xi[4];
    int32_t cnt[4] = {0, 0, 0, 0};
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int64_t i = i0 + 4 * sub + r;
        xi[r] = i < n ? S.px[i] : 0.0;
    }
    __syncthreads();
    // whole 256-point steps before the workgroup's rows, the one or two steps
    // that hold them, the steps after (the loads of several steps in flight)
    const int64_t before = i0 / 256 * 256;
    const int64_t after = (i0 + kRankRows + 255) / 256 * 256;
    int64_t kb = 0;
#pragma unroll 8
    for (; kb < before; kb += 256) {
        const double xk = S.px[kb + kl];
#pragma unroll
        for (int r = 0; r < 4; ++r) cnt[r] += xk <= xi[r] ? 1 : 0;
    }
    for (; kb < after; kb += 256) {
        const int64_t k = kb + kl;
        const double xk = k < n ? S.px[k] : INFINITY;
#pragma unroll
        for (int r = 0; r < 4; ++r)
            cnt[r] += (xk < xi[r] || (xk == xi[r] && k < i0 + 4 * sub + r)) ? 1 : 0;
    }
#pragma unroll 8
    for (; kb < n; kb += 256) {
        const int64_t k = kb + kl;
        const double xk = k < n ? S.px[k] : INFINITY;  // counted by nobody
#pragma unroll
        for (int r = 0; r < 4; ++r) cnt[r] += xk < xi[r] ? 1 : 0;
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        // the 16 lanes of the wavefront that hold the same rows
        for (int off = 4; off < 64; off <<= 1) cnt[r] += __shfl_xor(cnt[r], off, 64);
        if ((threadIdx.x & 63) < 4) atomicAdd(&total[4 * sub + r], cnt[r]);
    }
    __syncthreads();
    const int64_t i = i0 + threadIdx.x;
    if (threadIdx.x < kRankRows && i < n) {
        const int32_t r = total[threadIdx.x];
        S.sx[r] = S.px[i];
        S.sy[r] = S.py[i];
        S.sz[r] = S.pz[i];
        S.sk[r] = (int32_t)i;
    }
}

// Running minimum over the lanes of a wavefront (lane l: min of lanes 0..l),
// every lane active: shifts within each row of 16 lanes, then the last lane
// of the rows before (a lane without a source keeps its own value).
template <int CTRL, int ROWS>
__device__ __forceinline__ double dpp_min(double v)
{
    const int lo = __double2loint(v), hi = __double2hiint(v);
    const double y = __hiloint2double(__builtin_amdgcn_update_dpp(hi, hi, CTRL, ROWS, 0xf, false),
                                      __builtin_amdgcn_update_dpp(lo, lo, CTRL, ROWS, 0xf, false));
    return v < y ? v : y;
}
__device__ __forceinline__ double wave_prefix_min(double v)
{
    v = dpp_min<0x111, 0xf>(v);  // row_shr:1
    v = dpp_min<0x112, 0xf>(v);
    v = dpp_min<0x114, 0xf>(v);
    v = dpp_min<0x118, 0xf>(v);
    v = dpp_min<0x142, 0xa>(v);  // row_bcast:15
    v = dpp_min<0x143, 0xc>(v);  // row_bcast:31
    return v;
}

__device__ __forceinline__ double lane63(double v)
{
    return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), 63),
                            __builtin_amdgcn_readlane(__double2loint(v), 63));
}

__device__ __forceinline__ double wave_sum(double v)
{
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
    return v;
}

// Terms (1 - z_t) D_t of kTermRows rows next to each other in x order.  The
// points left of them only lower Y_t at x_t (every strip there ends at or
// before x_t), so up to the rows' own 64-point step they are a plain minimum:
// the workgroup's wavefronts share its steps and every step serves all rows
// (one row per wavefront read 1 GB from L2 at 10,011 points and took 103 us,
// bound by that).  Then each wavefront integrates one row from that step on
// and stops as soon as Y_t <= y_t: Y_t only falls, so every
// further strip adds nothing; on a front of n points that is some sqrt(n)
// positions past t.  Skipped strips add exact zeros, so the term is the full
// pass's.  10,011 rows: 302 -> 47 us, now the longest right scans (rows with
// small y_t), a chain of wavefront minima.  More rows share the left pass's
// reads but a workgroup lasts as long as the longest scan of its rows: 64 us
// with 16 rows, 52 with 8, 47 with 4, 55 with 2; from the last rows on, whose left
// passes are the longest, 50 against 46 (8 rows).
constexpr int kTermRows = 4;
__global__ __launch_bounds__(64 * kTermRows) void k_hv_terms(int64_t n, HvSpace S)
{
    __shared__ double left_of[kTermRows][kTermRows];
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int64_t r0 = (int64_t)blockIdx.x * kTermRows;
    const int64_t first = r0 / 64 * 64;  // the same step for all rows: 64 is a multiple of them
    double zt[kTermRows], left[kTermRows];
    int32_t kt[kTermRows];
#pragma unroll
    for (int r = 0; r < kTermRows; ++r) {
        zt[r] = r0 + r < n ? S.sz[r0 + r] : 0.0;
        kt[r] = r0 + r < n ? S.sk[r0 + r] : 0;
        left[r] = 1.0;
    }
    for (int64_t base = 64 * wv; base < first; base += 64 * kTermRows) {
        const double y = S.sy[base + lane], z = S.sz[base + lane];
        const int32_t k = S.sk[base + lane];
#pragma unroll
        for (int r = 0; r < kTermRows; ++r) {
            const bool before = z < zt[r] || (z == zt[r] && k < kt[r]);
            left[r] = before && y < left[r] ? y : left[r];
        }
    }
#pragma unroll
    for (int r = 0; r < kTermRows; ++r) {
        const double v = lane63(wave_prefix_min(left[r]));
        if (lane == 0) left_of[wv][r] = v;
    }
    __syncthreads();
    if (r0 + wv >= n) return;  // uniform per wavefront
    double carry = 1.0, acc = 0.0;
    for (int w = 0; w < kTermRows; ++w)
        carry = left_of[w][wv] < carry ? left_of[w][wv] : carry;
    const double xt = S.sx[r0 + wv], yt = S.sy[r0 + wv], z1 = S.sz[r0 + wv];
    const int32_t t = S.sk[r0 + wv];
    // the next step's points load while this one's minima run
    struct Step {
        double x, y, z, xn;
        int32_t k;
    };
    auto load = [&](int64_t base) {
        const int64_t p = base + lane;
        Step q{1.0, 1.0, 2.0, 1.0, 0};  // past the end: before nobody
        if (p < n) q = Step{S.sx[p], S.sy[p], S.sz[p], p + 1 < n ? S.sx[p + 1] : 1.0, S.sk[p]};
        return q;
    };
    Step q = load(first);
    for (int64_t base = first; base < n && z1 < 1.0 && carry > yt; base += 64) {  // uniform
        const Step next = load(base + 64);
        const bool before = q.z < z1 || (q.z == z1 && q.k < t);
        double Y = wave_prefix_min(before ? q.y : 1.0);
        Y = Y < carry ? Y : carry;
        carry = lane63(Y);
        const double lo = q.x > xt ? q.x : xt;
        const double w = q.xn > lo ? q.xn - lo : 0.0;
        const double h = Y > yt ? Y - yt : 0.0;
        acc = fma(w, h, acc);
        q = next;
    }
    acc = wave_sum(acc);
    if (lane == 0) S.term[t] = (1.0 - z1) * acc;
}

// out = (sum of v[0..n)) / div in a fixed order: one workgroup, strided
// partial sums per thread, then a tree in LDS.  n = 0 writes `empty`.
__global__ __launch_bounds__(1024) void k_sum_fixed(const double *v, int64_t n, double div,
                                                    double empty, double *out)
{
    __shared__ double s[1024];
    double a = 0.0;
    for (int64_t i = threadIdx.x; i < n; i += 1024) a += v[i];
    s[threadIdx.x] = a;
    __syncthreads();
    for (int w = 512; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w) s[threadIdx.x] += s[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) *out = n > 0 ? s[0] / div : empty;
}

// Best utility -w.f' of each weight row over the counted rows (the dot product
// as an fma chain in objective order).  A workgroup takes W weights and all
// rows: it normalises kEuTile rows at a time into LDS (the divisions once per
// row and workgroup, not once per pair), the counted ones only (order-free: a
// maximum), and its 1,024 threads share them: thread t holds the four weights
// 4 (t % (W / 4)) .. + 3 (one LDS read serves four pairs; with one weight per
// thread the reads bound the pass, 43 us at 10,011 x 5,151) and takes every
// 1024 / (W / 4)-th row; now 29 us, against 233 with the divisions per pair.  W is the largest of 64, 32, 16 and 8 that leaves 128
// workgroups: more weights share a normalised row, fewer spread over the CUs.
constexpr int kEuTile = 1024;
template <int M, int W>
__global__ __launch_bounds__(1024) void k_eu_best(const float *F, const uint8_t *valid,
                                                  int64_t n, Norm nm, const double *Wt,
                                                  int64_t nw, double *best)
{
    constexpr int G = W / 4;  // threads side by side over the weights
    __shared__ double f[kEuTile][M];
    __shared__ double part[16][W];
    __shared__ int count;
    const int t = threadIdx.x, lane = t & 63;
    const int64_t w0 = (int64_t)blockIdx.x * W + 4 * (t % G);
    double wk[4][M], b[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        b[q] = -INFINITY;
#pragma unroll
        for (int k = 0; k < M; ++k) wk[q][k] = w0 + q < nw ? Wt[(w0 + q) * M + k] : 0.0;
    }
    // this thread's row of a tile, read while the tile before is scored
    float row[M];
    bool counts = false;
    auto load = [&](int64_t i) {
        counts = i < n && (!valid || valid[i]);
#pragma unroll
        for (int k = 0; k < M; ++k) row[k] = i < n ? F[i * M + k] : 0.f;
    };
    load(t);
    for (int64_t base = 0; base < n; base += kEuTile) {
        if (t == 0) count = 0;
        __syncthreads();
#pragma unroll
        for (int k = 0; k < M; ++k) counts = counts && isfinite(row[k]);
        if (counts) {
            const int p = atomicAdd(&count, 1);
#pragma unroll
            for (int k = 0; k < M; ++k) f[p][k] = ((double)row[k] - nm.lo[k]) / nm.inv[k];
        }
        __syncthreads();
        load(base + kEuTile + t);
        const int c = count;
#pragma unroll 2
        for (int p = t / G; p < c; p += 1024 / G) {
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                double u = 0.0;
#pragma unroll
                for (int k = 0; k < M; ++k) u = fma(wk[q][k], f[p][k], u);
                b[q] = __builtin_fmax(b[q], -u);  // a NaN utility leaves the best as it is
            }
        }
        __syncthreads();
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) {
#pragma unroll
        for (int off = G; off < 64; off <<= 1) b[q] = __builtin_fmax(b[q], __shfl_xor(b[q], off, 64));
        if (lane < G) part[t >> 6][4 * lane + q] = b[q];
    }
    __syncthreads();
    if (t < W && (int64_t)blockIdx.x * W + t < nw) {
        double v = part[0][t];
        for (int wv = 1; wv < 16; ++wv) v = __builtin_fmax(v, part[wv][t]);
        best[(int64_t)blockIdx.x * W + t] = v;
    }
}

template <int M>
void launch_eu(const float *F, const uint8_t *valid, int64_t n, const Norm &nm, const double *Wt,
               int64_t nw, double *best, hipStream_t s)
{
    auto go = [&](auto kernel, int w) {
        hipLaunchKernelGGL(kernel, dim3((unsigned)((nw + w - 1) / w)), dim3(1024), 0, s, F, valid, n,
                           nm, Wt, nw, best);
    };
    if (nw >= 128 * 64) go(k_eu_best<M, 64>, 64);
    else if (nw >= 128 * 32) go(k_eu_best<M, 32>, 32);
    else if (nw >= 128 * 16) go(k_eu_best<M, 16>, 16);
    else go(k_eu_best<M, 8>, 8);
}

// Scratch of rvea_hypervolume_noalloc: a file-scope device array, one copy
// per GPU, held until the process ends; room for kNoAllocRows rows.  Host
// code must never pass `scratch` itself to a kernel (in host code the name
// stands for a host-side symbol, not a device address): its device address
// is looked up once per device and kept in g_scratch.
constexpr int64_t kNoAllocRows = (int64_t)1 << 17;
constexpr size_t kScratchBytes = 7 * ((size_t)kNoAllocRows * 8) + 2 * ((size_t)kNoAllocRows * 4);
static __device__ __align__(256) unsigned char scratch[kScratchBytes];

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void *g_scratch[kMaxDevices] = {};

// device address of the current device's scratch (looked up on the first
// call on that device, with that device current)
hipError_t scratch_of_current_device(void **out)
{
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (!g_scratch[dev]) {
        void *ptr = nullptr;
        e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        if (!ptr) return hipErrorInvalidSymbol;
        g_scratch[dev] = ptr;
    }
    *out = g_scratch[dev];
    return hipSuccess;
}

rvea_status norm_of(int m, const double *lo, const double *hi, Norm *nm)
{
    if (!lo || !hi) return RVEA_EINVAL;
    nm->m = m;
    for (int k = 0; k < m; ++k) {
        if (!std::isfinite(lo[k]) || !std::isfinite(hi[k]) || !(hi[k] > lo[k]))
            return RVEA_EINVAL;
        nm->lo[k] = lo[k];
        nm->inv[k] = hi[k] - lo[k];
    }
    return RVEA_OK;
}

rvea_status device_error(const char *what, hipError_t e)
{
    rvea::note_thread_error(what, e);
    return RVEA_EDEVICE;
}

// the hypervolume's launches on workspace ws (at least hv_bytes(n))
hipError_t enqueue_hv(const float *F, const uint8_t *valid, int64_t n, const Norm &nm,
                      double *out, void *ws, hipStream_t s)
{
    const HvSpace S = hv_space(ws, n);
    if (n > 0) {
        const unsigned nb = (unsigned)((n + 255) / 256);
        hipLaunchKernelGGL(k_hv_points, dim3(nb), dim3(256), 0, s, F, valid, n, nm, S);
        hipLaunchKernelGGL(k_hv_order, dim3((unsigned)((n + kRankRows - 1) / kRankRows)), dim3(1024),
                           0, s, n, S);
        hipLaunchKernelGGL(k_hv_terms, dim3((unsigned)((n + kTermRows - 1) / kTermRows)),
                           dim3(64 * kTermRows), 0, s, n, S);
    }
    hipLaunchKernelGGL(k_sum_fixed, dim3(1), dim3(1024), 0, s, S.term, n, 1.0, 0.0, out);
    return hipGetLastError();
}

}  // namespace

extern "C" {

rvea_status rvea_indicator_footprint(int m, int64_t n, int64_t nw, size_t *bytes)
{
    if (!bytes || m < 2 || m > kMaxObj || n < 0 || n > kMaxRows || nw < 0 || nw > kMaxRows)
        return RVEA_EINVAL;
    const size_t hv = m <= 3 && n <= kMaxHvRows ? hv_bytes(n) : 0;
    const size_t eu = up256((size_t)(nw > 0 ? nw : 1) * 8);
    *bytes = hv > eu ? hv : eu;
    return RVEA_OK;
}

rvea_status rvea_hypervolume(int m, int64_t n, const float *F, const uint8_t *valid,
                             const double *lo, const double *hi, double *out, void *workspace,
                             size_t workspace_bytes, void *hip_stream)
{
    if (m < 2 || m > 3 || n < 0 || n > kMaxHvRows || !out || (n > 0 && !F)) return RVEA_EINVAL;
    if (!workspace || ((uintptr_t)workspace & 255u)) return RVEA_EINVAL;
    Norm nm;
    rvea_status st = norm_of(m, lo, hi, &nm);
    if (st != RVEA_OK) return st;
    if (workspace_bytes < hv_bytes(n)) return RVEA_ENOMEM;
    const hipError_t e = enqueue_hv(F, valid, n, nm, out, workspace, (hipStream_t)hip_stream);
    return e == hipSuccess ? RVEA_OK : device_error("hypervolume launch", e);
}

rvea_status rvea_expected_utility(int m, int64_t n, const float *F, const uint8_t *valid,
                                  const double *lo, const double *hi, int64_t nw,
                                  const double *W, double *out, void *workspace,
                                  size_t workspace_bytes, void *hip_stream)
{
    if (m < 2 || m > kMaxObj || n < 0 || n > kMaxRows || nw < 1 || nw > kMaxRows || !W ||
        !out || (n > 0 && !F))
        return RVEA_EINVAL;
    if (!workspace || ((uintptr_t)workspace & 255u)) return RVEA_EINVAL;
    Norm nm;
    rvea_status st = norm_of(m, lo, hi, &nm);
    if (st != RVEA_OK) return st;
    if (workspace_bytes < (size_t)nw * 8) return RVEA_ENOMEM;
    hipStream_t s = (hipStream_t)hip_stream;
    double *best = (double *)workspace;
    switch (m) {
    case 2: launch_eu<2>(F, valid, n, nm, W, nw, best, s); break;
    case 3: launch_eu<3>(F, valid, n, nm, W, nw, best, s); break;
    case 4: launch_eu<4>(F, valid, n, nm, W, nw, best, s); break;
    case 5: launch_eu<5>(F, valid, n, nm, W, nw, best, s); break;
    case 6: launch_eu<6>(F, valid, n, nm, W, nw, best, s); break;
    case 7: launch_eu<7>(F, valid, n, nm, W, nw, best, s); break;
    default: launch_eu<8>(F, valid, n, nm, W, nw, best, s); break;
    }
    hipLaunchKernelGGL(k_sum_fixed, dim3(1), dim3(1024), 0, s, best, nw, (double)nw, -INFINITY,
                       out);
    const hipError_t e = hipGetLastError();
    return e == hipSuccess ? RVEA_OK : device_error("expected-utility launch", e);
}

rvea_status rvea_hypervolume_noalloc(int m, int64_t n, const float *F, const uint8_t *valid,
                                     const double *lo, const double *hi, double *out,
                                     void *hip_stream)
{
    if (m < 2 || m > 3 || n < 0 || !out || (n > 0 && !F)) return RVEA_EINVAL;
    if (n > kNoAllocRows) {
        rvea::note_thread_message("rvea_hypervolume_noalloc: more rows than its static "
                                  "scratch holds (at most 131072)");
        return RVEA_ENOMEM;
    }
    Norm nm;
    rvea_status st = norm_of(m, lo, hi, &nm);
    if (st != RVEA_OK) return st;
    void *ws = nullptr;
    hipError_t e = scratch_of_current_device(&ws);
    if (e != hipSuccess) return device_error("hipGetSymbolAddress(scratch)", e);
    if (hv_bytes(n) > kScratchBytes) return RVEA_ENOMEM;
    e = enqueue_hv(F, valid, n, nm, out, ws, (hipStream_t)hip_stream);
    return e == hipSuccess ? RVEA_OK : device_error("hypervolume launch", e);
}

}  // extern "C"
