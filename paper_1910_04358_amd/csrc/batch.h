// Batched-form state shared by the query entry point and the serving loop.
#pragma once

#include <functional>

#include "rambo_int.h"

namespace rambo {

struct BatchBufs {
    uint32_t *rmask;           // [cap][R * RW] running AND per multi-tile read
    unsigned long long *done;  // [cap] per multi-tile read: finished tiles (low 32 bits) and
                               // finished tiles that held a valid window (high 32 bits)
    uint64_t *extra;           // [cap] tiles beyond the first, per read
    uint64_t *extra_off;       // [cap + 1] exclusive scan of extra
    uint32_t *order;           // [4][cap] reads by size class of their first tile
    unsigned long long *cls;   // reads of size class v at cls[16 v]
    unsigned long long *head;  // queue position
    unsigned long long *work;  // windows of the reads that the scout pass leaves, in 16 parts (part v at
                               // work[16 v]); zero between batches
    uint32_t *tile;            // windows per work item of this batch
    uint32_t *smask;           // [cap][RW] repetition-0 AND over the scout windows (SCHED_PRESCOUT)
    uint32_t *live;            // [cap] bit 0: read not ended by the scout pass; bit 1: a scout
                               // window was valid (SCHED_PRESCOUT)
    uint64_t cap;
};

// Events of a direct launch: before prep, before main, after main. Kept apart from
// the state, which other calls may take while rambo_last_batch_ms still asks for them.
struct BatchEvents {
    hipEvent_t e[3] = {nullptr, nullptr, nullptr};
    ~BatchEvents();
};

// Work-queue state for batches of up to cap reads, with the captured graphs of
// the server's slots (prep: scout pass and queue; absent for the plain form) or,
// for the query entry point, without any: its launches are direct. The batch is
// described by the device header `in`, which the server copies and a direct
// launch's first kernel writes (own).
struct BatchGraph {
    uint64_t cap = 0;
    unsigned blocks = 0;  // workgroups of the persistent launch
    Tune tune;
    BatchBufs bb{};
    const InputHdr *in = nullptr;  // device
    InputHdr *own = nullptr;
    uint64_t *parts = nullptr;     // scan scratch
    void *mem = nullptr;
    hipGraph_t graph_prep = nullptr, graph_main = nullptr;
    hipGraphExec_t exec_prep = nullptr, exec_main = nullptr;
    std::shared_ptr<BatchEvents> ev;  // of the last direct launch
    hipStream_t stream = nullptr;     // its stream
    bool used = false;                // there was one
    uint64_t turn = 0;                // its place in the order of the handle's launches
    ~BatchGraph();
};

// Persistent batched form, captured, for batches described by in_dev (device),
// up to cap reads.
int make_batch_graph(rambo_s *h, const Tune &tu, const InputHdr *in_dev, uint64_t cap, uint64_t *out,
                     std::shared_ptr<BatchGraph> &res);
// One-node graph of the plain kernel for batches described by in_dev.
int make_plain_graph(rambo_s *h, const InputHdr *in_dev, uint64_t cap, uint64_t *out,
                     std::shared_ptr<BatchGraph> &res);
// Enqueue the graphs on s.
int launch_batch_graph(rambo_s *h, BatchGraph &bg, hipStream_t s);
bool tune_valid(const rambo_s *h, const Tune &t);
int autotune(rambo_s *h, const uint8_t *seqs, const uint64_t *offs, uint64_t n, uint64_t *out, hipStream_t s);

}  // namespace rambo
