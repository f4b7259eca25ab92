// rvea_transfer.h -- host side of the state transfers (rvea_transfer.hip).
#pragma once

#include <hip/hip_runtime.h>

#include <vector>

#include "rvea_dev.h"

namespace rvea {

constexpr size_t kStageBytes = (size_t)4 << 20;  // largest staging buffer (one chunk)
constexpr int kMaxParts = 8;                     // arrays of a chunk

struct Staging {
    uint8_t *p;
    size_t bytes;
};
hipError_t staging_take(size_t bytes, Staging *out);
void staging_give(const Staging &s);
void staging_runs(int change);  // a run was created (1) or destroyed (-1)

// one array of a chunk: device address (moved by stride bytes when the
// population's generation is odd), place in the staging buffer, length
struct Part {
    void *dev;
    size_t stride, at, bytes;
};
struct PartList {
    int n;
    Part part[kMaxParts];
};

struct StateArray {
    void *dev;
    size_t stride;
    void *host;
    size_t bytes;
};
// Copies the arrays, and the slots' gene rows if X is given, between the host
// and the workspace on stream s; returns when the copies are done.  Refused on
// a capturing stream, before anything is enqueued, and for rows longer than a
// chunk.
hipError_t transfer_state(const RunView &R, const StateArray *arrays, int n_arrays, float *X, bool out,
                          hipStream_t s);
// the rest of a host-set state at generation t
hipError_t launch_set_reset(const RunView &R, hipStream_t s, int64_t t, int unscale);

}  // namespace rvea
