// Device-wide exclusive scan of uint64 counts (scan.hip).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace rambo {

constexpr uint32_t kScanThreads = 256, kScanPer = 4;

// Scratch words `parts` must hold for a capacity of cap elements, kScanThreads *
// per of them a block.
uint64_t scan_parts_needed(uint64_t cap, uint32_t per = kScanPer);

// off[i] = v[0] + ... + v[i-1] for i < n, off[n] = total, with n = *n_ptr
// (device) and n <= cap. Enqueued on s; capturable in a graph.
int launch_exclusive_scan(const uint64_t *v, const uint64_t *n_ptr, uint64_t cap, uint64_t *off, uint64_t *parts,
                          hipStream_t s);

// As launch_exclusive_scan where parts already holds the sums of each
// kScanThreads * per elements (per 1 or kScanPer).
int launch_scan_parts(const uint64_t *v, const uint64_t *n_ptr, uint64_t cap, uint64_t *off, uint64_t *parts,
                      uint32_t per, hipStream_t s);

}  // namespace rambo
