// Slots of library-owned device state, one per stream.
//
// The quantize and analysis kernels combine their per-block counts in words of static device memory that
// are zero between launches and are cleared again by the last block to finish, so that no clearing
// kernel has to run before it.  Calls on one stream are ordered and can
// share a piece; calls on different streams may run at the same time and must not.  Each stream
// handle seen is therefore given a slot of its own, for the life of the process.
#include <mutex>

#include "cq_kernels.h"

namespace cq {

int stream_slot(hipStream_t stream, SlotTable table) {
    // the per-thread default stream is one handle for many real streams: no slot
    if (stream == hipStreamPerThread) return -1;
    static std::mutex mu;
    static hipStream_t seen[kSlotTables][kStateSlots];
    static int n_seen[kSlotTables];
    std::lock_guard<std::mutex> lock(mu);
    int& n = n_seen[table];
    for (int i = 0; i < n; ++i)
        if (seen[table][i] == stream) return i;
    if (n == kStateSlots) return -1;            // callers fall back to the path that clears first
    seen[table][n] = stream;
    return n++;
}

int uncaptured_stream_slot(hipStream_t stream, SlotTable table) {
    const int slot = stream_slot(stream, table);
    hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
    return slot >= 0 && hipStreamIsCapturing(stream, &cap) == hipSuccess && cap == hipStreamCaptureStatusNone ? slot : -1;
}

}  // namespace cq
