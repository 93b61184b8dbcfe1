// snowlb_graph.h -- when a call of the 2D or 3D step replays captured graphs.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace snowlb {

// Whether a call of n steps from copy `par` replays graphs of K steps (which start from copy 0): they cover at least four
// fifths of it, and the lattice is small or the call eight graphs long.  A direct launch costs the host 2.5 us, a step of
// a graph 1.5, which bounds a program that keeps several small contexts on streams of their own: four of 128^2, 64 steps a
// call, 2.6 us a step launched directly, 1.5 from graphs; of 256^2 2.5 and 1.7.  From about 2^17 cells on the GPU is the
// bound (512^2 4.8 to 5.4 us either way).  On one stream direct steps follow each other 0.1 to 0.3 us closer (128^2 3.35 us
// against 3.50, 1024^2 19.8 against 20.1) and need no capture (the first call of 64 steps 230 us, 304 with one).
inline bool replays_graphs(int32_t n, int32_t K, int par, int64_t cells) {
    const int64_t runs = (n - (par ? 1 : 0)) / K, whole = runs * K;
    return whole > 0 && 5 * whole >= 4 * (int64_t)n && (cells <= (int64_t(1) << 17) || runs >= 8);
}

// Whether the caller is capturing the stream: a graph cannot be launched into a capture, single steps can.
inline bool being_captured(hipStream_t s) {
    hipStreamCaptureStatus status = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(s, &status) != hipSuccess) {
        (void)hipGetLastError();
        return false;
    }
    return status == hipStreamCaptureStatusActive;
}

}  // namespace snowlb
