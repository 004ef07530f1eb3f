// Which iterations of k_column_run exchange rows through LDS, and through which of its two buffers, in one place so that the
// kernel and the host-only check program (sanitizer build) run the same arithmetic.
//
// An exchange writes x^(k+1/2) of all rows, meets at a barrier and reads other wavefronts' rows; an average meets a second time
// before the mean is read.  With two buffers in turn no barrier is needed behind the reads: the next exchange writes
// the other buffer, and the one after it writes this one behind the barrier of the exchange between them, which a
// wavefront reaches after its reads.  The turns therefore count exchanges and not iterations: where nodes keep their own
// iterate (W = I) a gossip iteration has no barrier, so it writes no buffer and takes no turn.
#pragma once

#include <hip/hip_runtime.h>

// kOwn: W = I; shift < 0: a global average.
template <bool kOwn>
__host__ __device__ __forceinline__ bool exchanges_rows(int n, int shift) {
    return n > 1 && (!kOwn || shift < 0);
}
// Iteration t, `before` exchanges into the launch (other graphs exchange in every iteration).
template <bool kOwn>
__host__ __device__ __forceinline__ int exchange_buffer(int t, int before) {
    return (kOwn ? before : t) & 1;
}
