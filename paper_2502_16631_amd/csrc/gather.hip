// DATA chunks to their payload records (see gather.h).
#include <hip/hip_runtime.h>

#include "gather.h"

namespace mk {
namespace {

constexpr int NT = 256;

// Bytes [lo, hi) of chunk g (lo and hi 16-byte multiples but for the chunk's
// end) to its record.
__device__ inline void copy_part(const GatherJob& j, uint64_t g, uint32_t lo, uint32_t hi) {
    const uint32_t C = j.C, tid = threadIdx.x;
    const AllocDesc* ad = j.allocs + j.amap[g];
    const uint64_t k = g - ad->first;
    const uint64_t nk = (ad->size + C - 1) / C;
    const uint32_t len = (k + 1 == nk) ? ad->tail_len : C;
    const uint4* src = reinterpret_cast<const uint4*>(ad->ptr + k * C);
    uint4* dst = reinterpret_cast<uint4*>(j.slot + j.off[g]);
    const uint32_t full = (hi < len ? hi : len) / 16, rem = len % 16;
#pragma unroll 4
    for (uint32_t i = lo / 16 + tid; i < full; i += NT) dst[i] = src[i];
    if (rem && len < hi && len > lo && tid == 0) {
        const uint8_t* sb = reinterpret_cast<const uint8_t*>(src + len / 16);
        uint32_t w[4] = {0, 0, 0, 0};
        for (uint32_t b = 0; b < rem; ++b) w[b >> 2] |= (uint32_t)sb[b] << (8 * (b & 3));
        dst[len / 16] = make_uint4(w[0], w[1], w[2], w[3]);
    }
}

// Bound by HBM (read and written once). A delta's DATA chunks are few and far
// between, and by chunk only as many work-groups as chunks had work: 29 chunks
// of 256 KiB took 33 us. From the list and in parts they spread over the chip.
__global__ void __launch_bounds__(NT) k_gather(GatherJob j) {
    if (j.stamp && blockIdx.x == 0 && threadIdx.x == 0) *j.stamp = wall_clock64();
    const uint32_t C = j.C, parts = C > kGatherPart ? C / kGatherPart : 1, len = C / parts;
    const uint64_t items = *j.n_list * parts;
    for (uint64_t i = blockIdx.x; i < items; i += gridDim.x) {
        const uint32_t p = (uint32_t)(i % parts);
        copy_part(j, j.list[i / parts], p * len, (p + 1) * len);
    }
}

}  // namespace

hipError_t launch_gather(const GatherJob& j, int grid, hipStream_t s) {
    if (!j.amap || !j.list || !j.n_list || grid < 1) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_gather, dim3(grid), dim3(NT), 0, s, j);
    return hipGetLastError();
}

}  // namespace mk
