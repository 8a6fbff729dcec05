// Checkpoint copies on the device: the eight state fields and the scalars to or from one blob.
#include "vs_internal.h"

namespace vs {

namespace {

constexpr int kBlock = 256;
typedef double d2v __attribute__((ext_vector_type(2)));

// blockIdx.y: the field. Four 16-byte values per lane, a block apart, all loaded before they are
// stored; block (0, 0) also copies the scalars and, on a save, writes the header's fixed words.
// Bound by HBM: 96^3 (113 MB of traffic) 30 us in one launch, where eight copies and two header
// transfers took about 150 us a call.
__global__ __launch_bounds__(kBlock) void k_state_copy(StateCopy a, size_t n2) {
    const d2v* __restrict__ src = reinterpret_cast<const d2v*>(a.src[blockIdx.y]);
    d2v* __restrict__ dst = reinterpret_cast<d2v*>(a.dst[blockIdx.y]);
    const size_t t0 = (size_t)blockIdx.x * (4 * kBlock) + threadIdx.x;
    if (t0 + 3 * kBlock < n2) {
        d2v v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) v[u] = src[t0 + u * kBlock];
#pragma unroll
        for (int u = 0; u < 4; ++u) dst[t0 + u * kBlock] = v[u];
    } else {
        for (int u = 0; u < 4; ++u)
            if (t0 + u * kBlock < n2) dst[t0 + u * kBlock] = src[t0 + u * kBlock];
    }
    if (blockIdx.x == 0 && blockIdx.y == 0) {
        const int t = threadIdx.x;
        if (t < SC_NSCAL) a.scal_dst[t] = a.scal_src[t];
        if (a.head_dst && t < kStateHeadWords) a.head_dst[t] = a.head[t];
        if (a.hist && t < 2) a.hist[t] = 0;
    }
}

}  // namespace

void launch_state_copy(hipStream_t s, const StateCopy& a, size_t n) {
    const size_t n2 = n / 2;   // nx is even
    launch_kernel(k_state_copy, dim3((unsigned)((n2 + 4 * kBlock - 1) / (4 * kBlock)), 8), dim3(kBlock), 0, s,
                  a, n2);
}

}  // namespace vs
