// Device-wide exclusive prefix sum of uint64 counts, in two passes (per-block
// sums; per-block scan after the sum of the earlier blocks), or three for more
// than 4,096 blocks (the block sums are scanned in between). The element count is read on the device, so the passes can be
// captured in a graph sized for a capacity.
#include "rambo_int.h"
#include "scan.h"

namespace rambo {

static constexpr uint64_t kScanChunk = kScanThreads * kScanPer;  // elements per block

// exclusive scan of one value per thread across the workgroup; returns the
// workgroup total in *total
__device__ __forceinline__ uint64_t block_exclusive_scan(uint64_t x, uint64_t *total) {
    __shared__ uint64_t wsum[kScanThreads / 64];
    const uint32_t lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    uint64_t incl = x;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const uint64_t y = __shfl_up(incl, d);
        if ((int)lane >= d) incl += y;
    }
    if (lane == 63) wsum[wave] = incl;
    __syncthreads();
    uint64_t before = 0, all = 0;
#pragma unroll
    for (uint32_t w = 0; w < kScanThreads / 64; w++) {
        const uint64_t s = wsum[w];
        if (w < wave) before += s;
        all += s;
    }
    __syncthreads();
    *total = all;
    return before + incl - x;
}

__global__ __launch_bounds__(kScanThreads) void k_scan_reduce(const uint64_t *__restrict__ v, const uint64_t *n_ptr,
                                                             uint64_t *__restrict__ part) {
    const uint64_t n = *n_ptr;
    const uint64_t base = (uint64_t)blockIdx.x * kScanChunk;
    uint64_t s = 0;
#pragma unroll
    for (uint32_t k = 0; k < kScanPer; k++) {
        const uint64_t i = base + k * kScanThreads + threadIdx.x;
        if (i < n) s += v[i];
    }
    uint64_t total;
    (void)block_exclusive_scan(s, &total);
    if (threadIdx.x == 0) part[blockIdx.x] = total;
}

// exclusive scan of the block sums (one workgroup, looping)
__global__ __launch_bounds__(kScanThreads) void k_scan_parts(uint64_t *__restrict__ part, const uint64_t *n_ptr,
                                                            uint64_t chunk) {
    const uint64_t n = *n_ptr;
    const uint64_t nb = (n + chunk - 1) / chunk;
    uint64_t carry = 0;
    for (uint64_t base = 0; base < nb; base += kScanThreads) {
        const uint64_t i = base + threadIdx.x;
        const uint64_t x = i < nb ? part[i] : 0;
        uint64_t total;
        const uint64_t ex = block_exclusive_scan(x, &total);
        if (i < nb) part[i] = carry + ex;
        carry += total;
    }
}

// Each workgroup's kScanThreads * PER elements, after the sum of the earlier
// workgroups' elements: part[blockIdx.x] if the block sums are scanned already
// (scanned), otherwise added up here.
template <uint32_t PER>
__global__ __launch_bounds__(kScanThreads) void k_scan_apply(const uint64_t *__restrict__ v, const uint64_t *n_ptr,
                                                            const uint64_t *__restrict__ part,
                                                            uint64_t *__restrict__ off, int scanned) {
    const uint64_t n = *n_ptr;
    const uint64_t base = (uint64_t)blockIdx.x * (kScanThreads * PER);
    if (base >= n) {
        if (n == 0 && blockIdx.x == 0 && threadIdx.x == 0) off[0] = 0;
        return;
    }
    uint64_t run = 0;
    if (scanned) {
        run = part[blockIdx.x];
    } else {
        uint64_t s = 0;
        for (uint32_t j = threadIdx.x; j < blockIdx.x; j += kScanThreads) s += part[j];
        (void)block_exclusive_scan(s, &run);
    }
    // thread t owns elements base + t * PER .. + PER - 1
    uint64_t x[PER], s = 0;
#pragma unroll
    for (uint32_t k = 0; k < PER; k++) {
        const uint64_t i = base + threadIdx.x * PER + k;
        x[k] = i < n ? v[i] : 0;
        s += x[k];
    }
    uint64_t total;
    const uint64_t before = run;
    run += block_exclusive_scan(s, &total);
#pragma unroll
    for (uint32_t k = 0; k < PER; k++) {
        const uint64_t i = base + threadIdx.x * PER + k;
        if (i < n) off[i] = run;
        run += x[k];
    }
    if (n - base <= kScanThreads * PER && threadIdx.x == 0) off[n] = before + total;
}

uint64_t scan_parts_needed(uint64_t cap, uint32_t per) {
    return (cap + kScanThreads * per - 1) / (kScanThreads * per) + 1;
}

int launch_scan_parts(const uint64_t *v, const uint64_t *n_ptr, uint64_t cap, uint64_t *off, uint64_t *parts,
                      uint32_t per, hipStream_t s) {
    const uint64_t chunk = (uint64_t)kScanThreads * per;
    const unsigned blocks = (unsigned)std::max<uint64_t>(1, (cap + chunk - 1) / chunk);
    // a workgroup adds up to 4,096 block sums itself (16 loads a thread), which
    // spares a launch of one workgroup (4.5 us)
    const int scanned = blocks > 4096;
    if (scanned) hipLaunchKernelGGL(k_scan_parts, dim3(1), dim3(kScanThreads), 0, s, parts, n_ptr, chunk);
    if (per == 1) hipLaunchKernelGGL(k_scan_apply<1>, dim3(blocks), dim3(kScanThreads), 0, s, v, n_ptr, parts, off, scanned);
    else hipLaunchKernelGGL(k_scan_apply<kScanPer>, dim3(blocks), dim3(kScanThreads), 0, s, v, n_ptr, parts, off, scanned);
    HIP_CHECK(hipGetLastError());
    return RAMBO_OK;
}

int launch_exclusive_scan(const uint64_t *v, const uint64_t *n_ptr, uint64_t cap, uint64_t *off, uint64_t *parts,
                          hipStream_t s) {
    const unsigned blocks = (unsigned)std::max<uint64_t>(1, (cap + kScanChunk - 1) / kScanChunk);
    hipLaunchKernelGGL(k_scan_reduce, dim3(blocks), dim3(kScanThreads), 0, s, v, n_ptr, parts);
    return launch_scan_parts(v, n_ptr, cap, off, parts, kScanPer, s);
}

}  // namespace rambo
