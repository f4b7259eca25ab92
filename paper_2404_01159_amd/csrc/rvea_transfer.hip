// rvea_transfer.hip -- the run state between host memory and the workspace
// (rvea_get_state, rvea_set_state): kernels that read and write pinned host
// memory directly, and the pinned staging buffers.
//
// Copying array by array cost a synchronous copy of pageable memory each
// (15-20 us; ten of them for a population of 32), the whole gene pool instead
// of the population's rows, and a two-dimensional copy row by row on the way in
// (20.7 ms for a population of 2,016 x 1,000 in and out).  Here a chunk is one
// kernel over PCIe and one copy inside host memory, and the next chunk's kernel
// runs while the host copies this one.
#include <algorithm>
#include <cstring>
#include <mutex>
#include <new>
#include <vector>

#include "rvea_dev.h"
#include "rvea_internal.h"
#include "rvea_transfer.h"

namespace rvea {

// ------------------------------------------------------------ staging pool
// Pinned buffers of 64 KiB, 512 KiB or 4 MiB, each in use only inside one
// accessor call, kept for the next call of any run, thread or stream (portable
// memory): at most kIdleBytes idle, and only small ones while no run exists.
namespace {

constexpr size_t kClasses[] = {(size_t)64 << 10, (size_t)512 << 10, kStageBytes};
constexpr size_t kIdleBytes = 4 * kStageBytes, kIdleNoRuns = (size_t)512 << 10;
std::mutex g_mu;
std::vector<Staging> g_idle;
int g_runs = 0;

size_t idle_bytes()
{
    size_t b = 0;
    for (const Staging &s : g_idle) b += s.bytes;
    return b;
}

// frees idle buffers, the largest first, until at most `keep` bytes stay
void trim(size_t keep)
{
    std::sort(g_idle.begin(), g_idle.end(),
              [](const Staging &a, const Staging &b) { return a.bytes < b.bytes; });
    while (!g_idle.empty() && idle_bytes() > keep) {
        (void)hipHostFree(g_idle.back().p);
        g_idle.pop_back();
    }
}

}  // namespace

hipError_t staging_take(size_t bytes, Staging *out)
{
    size_t want = kStageBytes;
    for (size_t c : kClasses)
        if (bytes <= c) {
            want = c;
            break;
        }
    {
        std::lock_guard<std::mutex> lock(g_mu);
        for (size_t i = 0; i < g_idle.size(); ++i) {
            if (g_idle[i].bytes != want) continue;
            *out = g_idle[i];
            g_idle.erase(g_idle.begin() + (ptrdiff_t)i);
            return hipSuccess;
        }
    }
    out->bytes = want;
    return hipHostMalloc((void **)&out->p, want, hipHostMallocPortable | hipHostMallocCoherent);
}

void staging_give(const Staging &s)
{
    if (!s.p) return;
    std::lock_guard<std::mutex> lock(g_mu);
    try {
        g_idle.push_back(s);
    } catch (const std::bad_alloc &) {  // no place in the list: not kept
        (void)hipHostFree(s.p);
        return;
    }
    trim(g_runs > 0 ? kIdleBytes : kIdleNoRuns);
}

void staging_runs(int change)
{
    std::lock_guard<std::mutex> lock(g_mu);
    g_runs += change;
    if (g_runs == 0) trim(kIdleNoRuns);
}

// ----------------------------------------------------------------- kernels
// The parts of one chunk, device to staging (OUT) or back: words where both
// sides are aligned to them, else bytes.  src of a part that alternates with
// the population is moved by its stride at odd generations.
template <bool OUT>
__global__ __launch_bounds__(256) void k_parts(RunView R, PartList L, uint8_t *stage)
{
    const int64_t p = OUT ? *R.t_done : 0;
    const int64_t tid = (int64_t)blockIdx.x * 256 + threadIdx.x, step = (int64_t)gridDim.x * 256;
    for (int k = 0; k < L.n; ++k) {
        const Part &q = L.part[k];
        uint8_t *dev = (uint8_t *)q.dev + (OUT && (p & 1) ? q.stride : 0);
        uint8_t *st = stage + q.at;
        uint8_t *to = OUT ? st : dev;
        const uint8_t *from = OUT ? dev : st;
        int64_t words = 0;
        if ((((uintptr_t)dev | (uintptr_t)st) & 3) == 0) {
            words = (int64_t)(q.bytes / 4);
            for (int64_t i = tid; i < words; i += step) ((uint32_t *)to)[i] = ((const uint32_t *)from)[i];
        }
        for (int64_t i = 4 * words + tid; i < (int64_t)q.bytes; i += step) to[i] = from[i];
    }
}

// Gene rows of slots [r0, r0 + gridDim.y) between the pool and the staging
// buffer (rows of d values): out the rows that the slots of the current
// population point at (zeros for empty slots), in slot j's row j.
template <bool OUT>
__global__ __launch_bounds__(256) void k_rows(RunView R, int64_t r0, float *stage)
{
    const int64_t j = r0 + blockIdx.y;
    const int c = (int)(blockIdx.x * 256 + threadIdx.x);
    if (c >= R.d) return;
    float *st = stage + (int64_t)blockIdx.y * R.d + c;
    if (OUT) {
        const int64_t p = *R.t_done;
        const float v = R.X[(int64_t)slot_row_of(R, p)[j] * R.ld + c];
        *st = valid_of(R, p)[j] ? v : 0.f;
    } else {
        R.X[j * (int64_t)R.ld + c] = *st;
    }
}

// What a host-set state at generation t leaves besides its arrays: slots on
// their own rows, marks 0 or 1, no row stamps, no ideal points, the generation
// counter, and with `unscale` the index's scaling back at one.
__global__ __launch_bounds__(256) void k_set_reset(RunView R, int64_t t, int unscale)
{
    const int64_t j = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (j < R.K) {
        slot_row_of(R, t)[j] = (int32_t)j;
        uint8_t *v = valid_of(R, t) + j;
        *v = *v ? 1 : 0;
    }
    if (j < R.M) stamp_of(R, t)[j] = -1;
    if (j < 3 * R.m) R.zbits[j] = 0xffffffffu;
    if (unscale && j < R.m) R.gr[j] = 1.0;
    if (j == 0) *R.t_done = t;
}

hipError_t launch_set_reset(const RunView &R, hipStream_t s, int64_t t, int unscale)
{
    const int64_t n = std::max<int64_t>(R.M, 3 * kMaxM);
    k_set_reset<<<(unsigned)((n + 255) / 256), 256, 0, s>>>(R, t, unscale);
    return hipGetLastError();
}

// --------------------------------------------------------------- transfers
namespace {

struct Chunk {
    PartList parts;       // parts.n > 0: arrays
    uint8_t *user[kMaxParts];
    int64_t r0, rows;     // else gene rows
    uint8_t *x;
    size_t bytes;         // of the staging buffer
};

hipError_t launch_chunk(const RunView &R, const Chunk &c, uint8_t *stage, bool out, hipStream_t s)
{
    if (c.parts.n > 0) {
        const unsigned g = (unsigned)std::min<size_t>(1024, (c.bytes / 4 + 255) / 256 + 1);
        if (out)
            k_parts<true><<<g, 256, 0, s>>>(R, c.parts, stage);
        else
            k_parts<false><<<g, 256, 0, s>>>(R, c.parts, stage);
    } else {
        const dim3 g((unsigned)((R.d + 255) / 256), (unsigned)c.rows);
        if (out)
            k_rows<true><<<g, 256, 0, s>>>(R, c.r0, (float *)stage);
        else
            k_rows<false><<<g, 256, 0, s>>>(R, c.r0, (float *)stage);
    }
    return hipGetLastError();
}

// between the user's arrays and a chunk's staging buffer
void host_copy(const RunView &R, const Chunk &c, uint8_t *stage, bool out)
{
    auto move = [&](uint8_t *user, uint8_t *st, size_t n) {
        if (out)
            std::memcpy(user, st, n);
        else
            std::memcpy(st, user, n);
    };
    for (int k = 0; k < c.parts.n; ++k) move(c.user[k], stage + c.parts.part[k].at, c.parts.part[k].bytes);
    if (c.parts.n == 0) move(c.x, stage, (size_t)c.rows * R.d * 4);
}

// arrays packed into chunks (a large one over several), then the rows
void plan_chunks(const RunView &R, const StateArray *arrays, int n_arrays, float *X,
                 std::vector<Chunk> *chunks)
{
    for (int k = 0; k < n_arrays; ++k) {
        const StateArray &a = arrays[k];
        for (size_t o = 0; o < a.bytes;) {
            if (chunks->empty() || chunks->back().parts.n == kMaxParts || chunks->back().bytes >= kStageBytes)
                chunks->push_back(Chunk{});
            Chunk &c = chunks->back();
            const size_t n = std::min(a.bytes - o, kStageBytes - c.bytes);
            c.user[c.parts.n] = (uint8_t *)a.host + o;
            c.parts.part[c.parts.n++] = Part{(uint8_t *)a.dev + o, a.stride, c.bytes, n};
            c.bytes = std::min(kStageBytes, (c.bytes + n + 15) / 16 * 16);
            o += n;
        }
    }
    if (!X) return;
    const int64_t rowb = (int64_t)R.d * 4;  // at most one chunk: longer rows are the caller's
    const int64_t per = std::min<int64_t>(65535, (int64_t)kStageBytes / rowb);
    for (int64_t r = 0; r < R.K; r += per) {
        Chunk c{};
        c.r0 = r;
        c.rows = std::min(per, R.K - r);
        c.x = (uint8_t *)(X + r * R.d);
        c.bytes = (size_t)(c.rows * rowb);
        chunks->push_back(c);
    }
}

}  // namespace

hipError_t transfer_state(const RunView &R, const StateArray *arrays, int n_arrays, float *X, bool out,
                          hipStream_t s)
{
    // nothing may be captured here: the staging buffers serve this call only
    hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
    const hipError_t ec = hipStreamIsCapturing(s, &cap);
    if (ec != hipSuccess) return ec;
    if (X && (size_t)R.d * 4 > kStageBytes) return hipErrorInvalidValue;
    if (cap != hipStreamCaptureStatusNone) return hipErrorStreamCaptureUnsupported;
    std::vector<Chunk> chunks;
    try {
        plan_chunks(R, arrays, n_arrays, X, &chunks);
    } catch (const std::bad_alloc &) {
        return hipErrorOutOfMemory;
    }
    // two buffers in turn: a chunk's kernel is enqueued before the host copies
    // the chunk before it, and a buffer is taken again once its event is done
    Staging st[2] = {};
    hipEvent_t ev[2] = {};
    hipError_t e = hipSuccess;
    const size_t nc = chunks.size();
    size_t need[2] = {0, 0};
    for (size_t i = 0; i < nc; ++i) need[i & 1] = std::max(need[i & 1], chunks[i].bytes);
    for (int b = 0; b < 2 && e == hipSuccess; ++b) {
        if (need[b] == 0) continue;
        e = staging_take(need[b], &st[b]);
        if (e == hipSuccess) e = hipEventCreateWithFlags(&ev[b], hipEventDisableTiming);
    }
    auto enqueue = [&](size_t i) {
        hipError_t r = launch_chunk(R, chunks[i], st[i & 1].p, out, s);
        return r == hipSuccess ? hipEventRecord(ev[i & 1], s) : r;
    };
    if (out) {
        if (e == hipSuccess && nc > 0) e = enqueue(0);
        for (size_t i = 0; i < nc && e == hipSuccess; ++i) {
            if (i + 1 < nc) e = enqueue(i + 1);  // chunk i - 1 has left that buffer
            if (e == hipSuccess) e = hipEventSynchronize(ev[i & 1]);
            if (e == hipSuccess) host_copy(R, chunks[i], st[i & 1].p, true);
        }
    } else {
        for (size_t i = 0; i < nc && e == hipSuccess; ++i) {
            if (i >= 2) e = hipEventSynchronize(ev[i & 1]);
            if (e == hipSuccess) host_copy(R, chunks[i], st[i & 1].p, false);
            if (e == hipSuccess) e = enqueue(i);
        }
    }
    // no buffer goes back while a kernel may still use it
    if (!out || e != hipSuccess) {
        const hipError_t e2 = hipStreamSynchronize(s);
        if (e == hipSuccess) e = e2;
    }
    for (int b = 0; b < 2; ++b) {
        if (ev[b]) (void)hipEventDestroy(ev[b]);
        staging_give(st[b]);
    }
    return e;
}

}  // namespace rvea
