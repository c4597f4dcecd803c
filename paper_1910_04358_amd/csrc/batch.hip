// Batched sequence queries: a scout pass over every read (scout schedule),
// then one persistent launch over a work queue of (read, tile of windows)
// items of the reads still alive, with a launch shape chosen by an autotuner.
//
// Most reads end on their scout windows (Section 3.3.1: once a term has
// emptied the running intersection, no later term can bring a document
// back); the scout pass answers them and leaves them out of the queue.
// The queue runs longest work first (see the order below). A read that fits
// one tile is finished by the wave that took it, from its LDS masks. Longer
// reads are spread over many waves; their tiles AND into a per-read mask in
// global memory (AND is associative and commutative, so the order does not
// matter), a tile whose read is already dead skips its probes, and the wave
// that finishes a read's last tile resolves it.
//
// The batch size lives in device memory, so one captured graph serves any
// batch up to its capacity (the serving loop's slots rely on this). The query
// entry point launches the same kernels directly.
#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <fstream>
#include <type_traits>

#include "batch.h"
#include "scan.h"

namespace rambo {

// Queue order of the persistent kernel, longest work first so that the last
// items to start are short. Class c holds the reads whose first tile has
// [c, c+1) quarters of a tile of windows (class 3 up to a full tile, which
// includes every multi-tile read). Order: class 3 first tiles, then every
// extra tile (tiles 1.. of multi-tile reads; after their read's first tile,
// which may empty the read's masks and let them skip), then classes 2, 1, 0.
// (the four class counters are 128 bytes apart: their atomics use different
// cache lines)
// A direct launch's header (own): written by its first kernel.
constexpr uint32_t kWorkParts = 16;
__global__ void k_batch_reset(BatchBufs bb, InputHdr val, InputHdr *own) {
    if (threadIdx.x == 0) *bb.head = 0;
    if (threadIdx.x == 0 && own) *own = val;
    if (threadIdx.x < 4) bb.cls[16 * threadIdx.x] = 0;
    if (threadIdx.x < kWorkParts) bb.work[16 * threadIdx.x] = 0;
}

// Windows per work item: `most`, the tuned tile, or fewer where the batch's items
// would then be too few to keep the chip busy, down to `least` -- a tile takes about
// as long as G (lanes that split a row) times its windows. What counts are the
// windows that are left to probe: those of the reads that the scout pass has not
// ended (without one, of all reads). Best tiles of 64 .. 2,048 measured, reads of
// which 4 % (K=101,000, G=8) and 25 % (K=10,000, G=1) are left: G=1 512 at 500 to
// 8,000 reads, 1,024 at 30,000, 2,048 at 100,000; G=8 64 at 64 to 8,000 reads, 128
// at 30,000, 256 at 100,000, 512 at 300,000: 1,500 items, at least 512 / G windows
// each. (By the number of reads alone, 8,000 reads of 10 kbp that all live came in
// 1.2 million items of 64: 21.4 ms at K=101,000, 19.6 with tiles of 1,024.)
// left: the windows in this lane's part. All 64 lanes; the same in every wave.
__device__ __forceinline__ uint32_t batch_tile(uint64_t left, uint32_t least, uint32_t most) {
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) left += __shfl_xor(left, d);
    uint32_t t = least;
    while (t < most && 2 * (uint64_t)t <= left / 1500) t *= 2;
    return min(t, most);
}

// With a scout pass before it (prescout), reads that pass ended are
// answered already and left out of the queue, and a multi-tile read's
// running mask starts from its scout AND in repetition 0.
// Each thread takes kPrepReads reads (kThreads apart), so a workgroup makes one
// atomic per size class for kThreads x kPrepReads reads: same-address atomics
// serialise, and one per 256 reads made the pass over 10^6 reads wait on them
// (52 -> 23 us with 4); small batches keep one read per thread (100,000
// reads: 9 us with 1, 19 us with 4, where fewer workgroups wait longer).
// The workgroup's sum of extra tiles goes to part, for the scan. A batch that
// one workgroup holds (kOne, up to 2,048 reads) is scanned here too, and needs
// neither the reset nor the scan's launches (1,999 reads: 24 us in five
// launches, now one of 7).
template <uint32_t kPrepReads, uint32_t kThreads, bool kOne>
__global__ __launch_bounds__(kThreads) void k_batch_prep(const InputHdr *in, uint32_t mw, uint32_t rw, uint32_t least,
                                                         uint32_t most, BatchBufs bb, int prescout,
                                                         uint64_t *__restrict__ part) {
    constexpr uint32_t kWaves = kThreads / 64;
    const InputHdr hd = *in;
    const uint64_t n = hd.n;
    const uint64_t *__restrict__ offs = hd.offs;
    const uint32_t lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    bool real[kPrepReads];
    uint32_t cls[kPrepReads];
    uint64_t extra[kPrepReads], nws[kPrepReads];
    // (every load before the first use)
    uint64_t left = 0;
    if (prescout) left = lane < kWorkParts ? bb.work[16 * lane] : 0;
    else if (lane == 0 && n) left = offs[n] - offs[0];
#pragma unroll
    for (uint32_t k = 0; k < kPrepReads; k++) {
        const uint64_t i = ((uint64_t)blockIdx.x * kPrepReads + k) * kThreads + threadIdx.x;
        real[k] = i < n;
        nws[k] = 0;
        if (real[k]) {
            const uint64_t beg = offs[i], end = offs[i + 1];
            const uint32_t live = prescout ? bb.live[i] : 1u;
            nws[k] = n_windows(beg, end);
            real[k] = live & 1u;
        }
    }
    const uint32_t tile = batch_tile(left, least, most);
    if (blockIdx.x == 0 && threadIdx.x == 0) *bb.tile = tile;
#pragma unroll
    for (uint32_t k = 0; k < kPrepReads; k++) {
        const uint64_t i0 = ((uint64_t)blockIdx.x * kPrepReads + k) * kThreads, i = i0 + threadIdx.x;
        cls[k] = 0;
        extra[k] = 0;
        if (real[k]) {
            const uint64_t nw = nws[k], tiles = nw ? (nw + tile - 1) / tile : 1;
            extra[k] = tiles - 1;
            cls[k] = (uint32_t)min<uint64_t>(3, min<uint64_t>(nw, tile) * 4 / tile);
        }
        if (!kOne && i < n) bb.extra[i] = extra[k];
        // the multi-tile reads' masks, a wave per read (192 words each at R=6,
        // B=1,000)
        if (extra[k]) bb.done[i] = 0;
        uint64_t multi = __ballot(extra[k] != 0);
        while (multi) {
            const uint64_t j = i0 + wave * 64 + (uint64_t)__builtin_ctzll(multi);
            multi &= multi - 1;
            for (uint32_t w = lane; w < mw; w += 64)
                bb.rmask[j * mw + w] = (prescout && w < rw) ? bb.smask[j * rw + w] : 0xFFFFFFFFu;
        }
    }
    // slots in the class lists, in read order: ranks within the wave
    // (ballots), offsets of the earlier (read group, wave) pairs of the
    // workgroup (LDS), one atomic per class and workgroup
    __shared__ uint32_t wcount[kPrepReads][kWaves][4];  // [read group][wave][class]
    __shared__ unsigned long long bbase[4], esum[kPrepReads][kWaves];
    uint64_t mine[kPrepReads], eincl[kPrepReads];
#pragma unroll
    for (uint32_t k = 0; k < kPrepReads; k++) {
        mine[k] = 0;
        for (uint32_t v = 0; v < 4; v++) {
            const uint64_t mask = __ballot(real[k] && cls[k] == v);
            if (cls[k] == v) mine[k] = mask;
            if (lane == 0) wcount[k][wave][v] = (uint32_t)__popcll(mask);
        }
        uint64_t e = extra[k];
        if (__ballot(e != 0)) {
#pragma unroll
            for (int d = 1; d < 64; d <<= 1) {
                const uint64_t y = __shfl_up(e, d);
                if ((int)lane >= d) e += y;
            }
        }
        eincl[k] = e;
        if (lane == 63) esum[k][wave] = e;
    }
    __syncthreads();
    if (threadIdx.x < 4) {
        const uint32_t v = threadIdx.x;
        uint32_t tot = 0;
        for (uint32_t k = 0; k < kPrepReads; k++)
            for (uint32_t w = 0; w < kWaves; w++) tot += wcount[k][w][v];
        if constexpr (kOne) {
            bbase[v] = 0;
            bb.cls[16 * v] = tot;
        } else {
            bbase[v] = tot ? atomicAdd(bb.cls + 16 * v, (unsigned long long)tot) : 0ull;
        }
    }
    if (kOne && threadIdx.x == 4) *bb.head = 0;
    if (!kOne && threadIdx.x == 64) {
        uint64_t sum = 0;
        for (uint32_t k = 0; k < kPrepReads; k++)
            for (uint32_t w = 0; w < kWaves; w++) sum += esum[k][w];
        part[blockIdx.x] = sum;
    }
    __syncthreads();
#pragma unroll
    for (uint32_t k = 0; k < kPrepReads; k++) {
        const uint64_t i = ((uint64_t)blockIdx.x * kPrepReads + k) * kThreads + threadIdx.x;
        if constexpr (kOne) {
            uint64_t before = 0;
            for (uint32_t j = 0; j < k * kWaves + wave; j++) before += esum[j / kWaves][j % kWaves];
            if (i < n) bb.extra_off[i] = before + eincl[k] - extra[k];
            if (i + 1 == n) bb.extra_off[n] = before + eincl[k];
            if (n == 0 && i == 0) bb.extra_off[0] = 0;
        }
        if (!real[k]) continue;
        const uint32_t c = cls[k];
        uint64_t slot = bbase[c] + __popcll(mine[k] & ((1ULL << lane) - 1));
        for (uint32_t kk = 0; kk < k; kk++)
            for (uint32_t w = 0; w < kWaves; w++) slot += wcount[kk][w][c];
        for (uint32_t w = 0; w < wave; w++) slot += wcount[k][w][c];
        bb.order[(uint64_t)c * bb.cap + slot] = (uint32_t)i;
    }
}

// lanes per read in the scout pass
__host__ __device__ constexpr int scout_group(int G, bool narrow) {
    return (narrow && G >= 8) ? G : (16 * G < 64 ? 16 * G : 64);
}

// The scout pass's window arithmetic within one read (a read holds fewer
// than 2^32 bytes): windows, scout windows and scout positions as in
// n_windows, scout_count and scout_pos over the whole read, in 32 bits.
__device__ __forceinline__ uint32_t windows32(uint64_t beg, uint64_t end) {
    return end >= beg + 31 ? (uint32_t)(end - beg - 30) : 0u;
}
__device__ __forceinline__ uint32_t scout_count32(uint32_t nw) {
    return nw ? (nw + 30) / 31 + ((nw - 1) % 31 != 0 ? 1u : 0u) : 0u;
}
__device__ __forceinline__ uint32_t scout_pos32(uint32_t nw, uint32_t k) { return min(31u * k, nw - 1); }

// Scout pass of the batched form (SCHED_SCOUT), before the queue is
// built: repetition 0 on every read's scout windows (every 31st window and
// the last, which together cover every base of the read). A group of GS
// lanes takes one read at a time, GS / G windows per round (G lanes split a
// row, as in the main kernel), and ANDs the rounds' rows by lane exchanges.
// The AND is stored in smask[i], the starting repetition-0 mask of the read's
// items, and live[i] says whether it is non-empty. With early exit an empty
// AND ends the read here (Section 3.3.1): its answer (a zero bitset, or a
// zero answer size in id-list mode) is written now and the read never enters
// the queue.
//
// Most reads end after a round or two, so the pass is a chain of short
// dependent steps (offsets, window bytes, rows) per read. Each group walks
// its own reads (every stride-th one) independently of the other groups of
// its wave -- a group whose read ended starts the next at once -- and loads
// one round ahead: while a round's rows are in flight, the group also loads
// the bytes of its read's next round and of its next read's first round, and
// the offsets two reads ahead. A round then costs one memory round trip,
// whichever way the read goes. The grid is what fits on the device at once.
// NARROW (where an ended read costs no output here: id lists, and large batches of
// bitsets) gives rows split
// over 8 or more lanes one window per round (a group of G lanes per read)
// instead of 8: the read ends at its first empty window, with no probes of
// the windows after it, and a wave holds as many rows in flight as with wider
// groups, as it walks 8 reads at once; where this pass writes the zero bitsets
// (zero), the wider groups write them faster.
// In id-list mode with split rows a wave keeps only 8 reads' rounds in
// flight and the pass waits on their round trips: 8 waves per SIMD instead of
// the 7 its 71 VGPRs allow (two values spilled to scratch) make it 12 % faster
// (K=101,000: 0.44 -> 0.39 ms).
template <int SEG, int G, int NARROW>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu((NARROW && G >= 8) ? 8 : 1))) void k_batch_scout(Index ix, const InputHdr *in, uint64_t *__restrict__ out,
                                                     BatchBufs bb, QueryOpts opt, InputHdr val, InputHdr *own,
                                                     bool zero) {
    constexpr int GS = scout_group(G, NARROW != 0);  // lanes per read
    constexpr int SLOTS = GS / G;                   // windows per round
    const InputHdr hd = own ? val : *in;
    const uint8_t *__restrict__ seqs = hd.seqs;
    const uint64_t *__restrict__ offs = hd.offs;
    const uint64_t n = hd.n;
    if (own && blockIdx.x == 0 && threadIdx.x == 0) *own = val;
    const uint32_t lane = threadIdx.x & 63;
    const uint32_t sub = lane % GS, seg = sub % G, slot = sub / G;
    const uint64_t gmask = (GS >= 64) ? ~0ULL : (((1ULL << GS) - 1) << (lane - sub));  // the group's lanes
    constexpr uint32_t GPB = 256 / GS;  // groups per workgroup
    const uint64_t stride = (uint64_t)gridDim.x * GPB;
    __shared__ unsigned long long blk_issued, blk_left;
    if (threadIdx.x == 0) blk_issued = blk_left = 0;
    // (the queue that is built next starts empty)
    if (blockIdx.x == 0 && threadIdx.x == 0) *bb.head = 0;
    if (blockIdx.x == 0 && threadIdx.x < 4) bb.cls[16 * threadIdx.x] = 0;
    __syncthreads();
    uint64_t issued = 0;

    // the group's current read i, with the offsets of the next two at hand
    uint64_t i = (uint64_t)blockIdx.x * GPB + threadIdx.x / GS;
    // (offsets read as global memory, as the window bytes are: a generic
    // load would also count against the scalar-load counter, and each wait
    // for the hash parameters would wait for it; a read with end < beg has no
    // window, which n_windows gives without clamping)
    typedef const uint64_t __attribute__((address_space(1))) *goffs;
    auto bounds = [&](uint64_t r, uint64_t &b, uint64_t &e) {
        b = e = 0;
        if (r < n) {
            b = ((goffs)offs)[r];
            e = ((goffs)offs)[r + 1];
        }
    };
    uint64_t beg, end, nbeg, nend, nnbeg = 0, nnend = 0;
    bounds(i, beg, end);
    bounds(i + stride, nbeg, nend);
    bool need_offs = true;  // the offsets of read i + 2 stride are still to load
    uint32_t nw = windows32(beg, end), ns = scout_count32(nw);
    uint32_t k0 = 0;  // first scout window of the current round
    // A window's bytes are loaded and decoded by the P lanes that split its
    // rows (P = 1: each lane takes a whole window).
    constexpr int P = G >= 8 ? 8 : G;
    using Bytes = std::conditional_t<(P > 1), WinPart<P>, WinBytes>;
    auto load_win = [&](Bytes &b, const uint8_t *p) {
        if constexpr (P > 1) load_window_part<P>(b, p, seg % P);
        else load_window_bytes(b, p);
    };
    auto decode_win = [&](const Bytes &b) -> Window {
        if constexpr (P > 1) return decode_window_parts<P>(b, seg % P);
        else return decode_window(b);
    };
    Bytes cur{}, next_round{}, next_read{};
    bool next_read_loaded = false;
    if (i < n && slot < ns) load_win(cur, seqs + beg + scout_pos32(nw, slot));
    // repetition 0's hash functions (eta <= 2), held for the whole pass
    const HashRec h0 = hash_rec(ix.hp->h, 0), h1 = hash_rec(ix.hp->h, ix.eta >= 2 ? 1 : 0);
    Seg<SEG> acc;
#pragma unroll
    for (int s = 0; s < SEG; s++) acc.w[s] = 0xFFFFFFFFu;
    bool saw = false;  // some scout window of the read was valid (uniform over the group)
    // Every load a round issues has completed when the round ends (explicit
    // wait at its end): the loads ahead are issued first, then the round's
    // rows, and the wait for the rows covers them all. The compiler's waits
    // inside the loop then never hold a load ahead back.
    __builtin_amdgcn_s_waitcnt(0);
    for (;;) {
        const bool have = i < n;
        if (__ballot(have) == 0) break;
        // loads ahead: the offsets two reads on, the bytes of this read's
        // next round and of the next read's first round
        const bool more = have && k0 + SLOTS < ns;
        if (need_offs) {
            bounds(i + 2 * stride, nnbeg, nnend);
            need_offs = false;
        }
        if (more && k0 + SLOTS + slot < ns) load_win(next_round, seqs + beg + scout_pos32(nw, k0 + SLOTS + slot));
        if (!next_read_loaded && i + stride < n) {
            const uint32_t w2 = windows32(nbeg, nend);
            if (slot < scout_count32(w2)) load_win(next_read, seqs + nbeg + scout_pos32(w2, slot));
            next_read_loaded = true;
        }
        // this round (every lane decodes: the lanes of a window exchange parts)
        Window wv = decode_win(cur);
        wv.valid = wv.valid && have && k0 + slot < ns;
        Seg<SEG> cm[1];
#pragma unroll
        for (int s = 0; s < SEG; s++) cm[0].w[s] = 0xFFFFFFFFu;
        if (wv.valid) {
            if (ix.eta <= 2) {
                // both rows in flight together (with one hash function the
                // same row twice)
                const Seg<SEG> a = load_seg<SEG>(row_ptr(ix, 0, bloom_pos(h0, ix.m, wv.canon)) + seg * SEG);
                const Seg<SEG> b = load_seg<SEG>(row_ptr(ix, 0, bloom_pos(h1, ix.m, wv.canon)) + seg * SEG);
#pragma unroll
                for (int s = 0; s < SEG; s++) cm[0].w[s] = a.w[s] & b.w[s];
            } else {
                probe_reps<SEG, 0, 1>(ix, ix.hp->h, wv.canon, seg, cm);
            }
        }
        const uint64_t vb = __ballot(wv.valid && seg == 0);
        issued += (uint64_t)__popcll(vb);
        saw |= (vb & gmask) != 0;
        uint32_t o = 0;
#pragma unroll
        for (int s = 0; s < SEG; s++) {
            uint32_t v = cm[0].w[s];
#pragma unroll
            for (int d = G; d < GS; d <<= 1) v &= (uint32_t)__shfl_xor((int)v, d);
            acc.w[s] &= v;
            o |= acc.w[s];
        }
        const bool live = !opt.early_exit || (__ballot(o != 0) & gmask) != 0;
        if (have && live && more) {
            k0 += SLOTS;
            cur = next_round;
        } else if (have) {
            // read i is done: its scout AND, and the answer of an ended read
            if (slot == 0)
#pragma unroll
                for (int s = 0; s < SEG; s++) bb.smask[i * ix.RW + seg * SEG + s] = acc.w[s];
            if (sub == 0) bb.live[i] = (live ? 1u : 0u) | (saw ? 2u : 0u);
            if (live && sub == 0) atomicAdd(&blk_left, (unsigned long long)nw);
            if (!live) {
                if (opt.counts) {
                    if (sub == 0) opt.counts[i] = 0;
                } else if (zero) {  // (otherwise k_batch_zero's work)
                    for (uint32_t w = sub; w < ix.W; w += GS) out[i * ix.W + w] = 0;
                }
            }
            // on to the next read
            i += stride;
            beg = nbeg;
            end = nend;
            nbeg = nnbeg;
            nend = nnend;
            need_offs = true;
            nw = windows32(beg, end);
            ns = scout_count32(nw);
            k0 = 0;
            cur = next_read;
            next_read_loaded = false;
#pragma unroll
            for (int s = 0; s < SEG; s++) acc.w[s] = 0xFFFFFFFFu;
            saw = false;
        }
        __builtin_amdgcn_s_waitcnt(0);
    }
    // one counter update per workgroup (same-address atomics serialise), and the
    // windows left spread over several
    if (opt.probes && lane == 0 && issued) atomicAdd(&blk_issued, (unsigned long long)issued);
    __syncthreads();
    if (threadIdx.x == 0) {
        if (blk_left) atomicAdd(bb.work + 16 * (blockIdx.x % kWorkParts), blk_left);
        if (opt.probes && blk_issued) atomicAdd(opt.probes, blk_issued * ix.eta);
    }
}

// The zero bitsets of the reads that the scout pass ended, where it leaves them to
// this kernel: a wave takes eight consecutive reads and writes their rows 1 KB a
// store, and waits for none (K=101,000, 10^5 reads, 1.2 GB: the pass and this
// kernel 80 and 195 us, 298 in one).
__global__ __launch_bounds__(256) void k_batch_zero(const InputHdr *in, const uint32_t *__restrict__ live,
                                                    uint64_t *__restrict__ out, uint64_t W) {
    const uint64_t n = in->n;
    const uint32_t lane = threadIdx.x & 63;
    const uint64_t stride = (uint64_t)gridDim.x * (blockDim.x >> 6) * 8;
    const uint64_t zero[2] = {0, 0};
    for (uint64_t i0 = (((uint64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6) * 8; i0 < n; i0 += stride) {
        uint64_t ended = __ballot(lane < 8 && i0 + lane < n && !(live[min(i0 + lane, n - 1)] & 1u));
        while (ended) {
            uint64_t *row = out + (i0 + (uint64_t)__builtin_ctzll(ended)) * W;
            ended &= ended - 1;
            for (uint64_t w = 2 * lane; w + 1 < W; w += 128) __builtin_memcpy(row + w, zero, 16);
            if ((W & 1) && lane == 0) row[W - 1] = 0;
        }
    }
}

// largest i < n with off[i] <= u, by a 64-way search (one load per lane per round)
__device__ __forceinline__ uint64_t find_read(const uint64_t *off, uint64_t n, uint64_t u, uint32_t lane) {
    uint64_t lo = 0, hi = n;  // invariant: off[lo] <= u, answer in [lo, hi)
    while (hi - lo > 1) {
        const uint64_t step = (hi - lo + 63) / 64;
        const uint64_t idx = lo + (uint64_t)lane * step;
        const bool pred = idx < hi && off[idx] <= u;
        const uint32_t k = (uint32_t)__popcll(__ballot(pred)) - 1;  // pred holds on a prefix of lanes
        lo = lo + (uint64_t)k * step;
        hi = min(hi, lo + step);
    }
    return lo;
}

__device__ __forceinline__ uint32_t load_coherent(const uint32_t *p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// some repetition of the read's global running mask is already empty
__device__ __forceinline__ bool read_dead(const Index &ix, const uint32_t *rm, uint32_t lane) {
    bool dead = false;
    for (uint32_t r = 0; r < ix.R; r++) {
        uint32_t o = 0;
        for (uint32_t w = lane; w < ix.RW; w += 64) o |= load_coherent(rm + r * ix.RW + w);
        dead |= __ballot(o != 0) == 0;
    }
    return dead;
}

// Rows split over G > 1 lanes: the compiler's default would take 172 VGPRs
// (2 waves per SIMD); 3 waves fit without spilling.
template <int SEG, int G>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(G == 1 ? 1 : 3))) void k_batch_main(Index ix, const InputHdr *in, uint64_t *__restrict__ out,
                                                    BatchBufs bb, QueryOpts opt, int use_res, uint32_t grab) {
    const uint8_t *__restrict__ seqs = in->seqs;
    const uint64_t *__restrict__ offs = in->offs;
    extern __shared__ __align__(16) uint64_t smem64[];
    const uint32_t lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const uint32_t mw = ix.R * ix.RW;
    // (no staging area: this form scouts in a pass of its own)
    const WaveLds L = wave_lds(mw, ix.W, use_res != 0, false);
    uint32_t *M = reinterpret_cast<uint32_t *>(smem64) + wave * L.total;
    uint64_t *res = use_res ? reinterpret_cast<uint64_t *>(M + L.res) : nullptr;
    uint8_t *stage = nullptr;

    const uint64_t n = in->n;
    const uint32_t tile = __builtin_amdgcn_readfirstlane(*bb.tile);
    // (read by the queue's kernels, which have ended: zero for the next batch)
    if (blockIdx.x == 0 && threadIdx.x < kWorkParts) bb.work[16 * threadIdx.x] = 0;
    const uint64_t n_extra = bb.extra_off[n];
    const uint64_t c3 = uniform64(bb.cls[48]), c2 = uniform64(bb.cls[32]), c1 = uniform64(bb.cls[16]);
    const uint64_t total = c3 + c2 + c1 + uniform64(bb.cls[0]) + n_extra;  // queued reads and extra tiles
    uint64_t issued = 0;
    // A wave's first items come with its place in the grid, the longest to
    // different workgroups; the queue's head counts from there. (Taken from the
    // head as well, by all 4,096 waves at once, they came 30 us late: the atomics
    // on one word are performed one after the other.)
    const uint64_t waves = (uint64_t)gridDim.x * (blockDim.x >> 6);
    bool started = false;
    for (;;) {
        uint64_t t0 = ((uint64_t)wave * gridDim.x + blockIdx.x) * grab;
        if (started) {
            if (lane == 0) t0 = waves * grab + atomicAdd(bb.head, (unsigned long long)grab);
            t0 = __shfl(t0, 0);
        }
        started = true;
        t0 = uniform64(t0);
        if (t0 >= total) break;
        const uint64_t t1 = min(total, t0 + grab);
        for (uint64_t t = t0; t < t1; t++) {
            uint64_t i, c = 0;
            if (t >= c3 && t < c3 + n_extra) {
                const uint64_t u = t - c3;
                i = uniform64(find_read(bb.extra_off, n, u, lane));
                c = uniform64(1 + (u - bb.extra_off[i]));
            } else {
                uint64_t u = t, v = 3;
                if (u >= c3) {
                    u -= c3 + n_extra;
                    v = 2;
                    if (u >= c2) { u -= c2; v = 1; }
                    if (v == 1 && u >= c1) { u -= c1; v = 0; }
                }
                i = uniform64(bb.order[v * bb.cap + u]);
            }
            const uint64_t beg = uniform64(offs[i]);
            uint64_t end = uniform64(offs[i + 1]);
            if (end < beg) end = beg;
            const uint64_t nwin = n_windows(beg, end);
            const uint64_t ntiles = nwin ? (nwin + tile - 1) / tile : 1;
            uint32_t *rm = bb.rmask + i * mw;
            uint64_t *o = out + i * ix.W;

            // another tile of the read may have emptied its masks already
            const bool skip = ntiles > 1 && opt.early_exit && read_dead(ix, rm, lane);
            init_masks(ix, M, lane);
            if (opt.sched == SCHED_PRESCOUT && ntiles == 1)
                for (uint32_t w = lane; w < ix.RW; w += 64) M[w] = bb.smask[i * ix.RW + w];
            uint64_t got = 0;  // probes this item issued (0: no valid window in it)
            if (!skip) {
                const uint64_t w_hi = min(nwin, (c + 1) * (uint64_t)tile);
                got = probe_windows<SEG, G>(ix, seqs, beg, end, c * (uint64_t)tile, w_hi, lane, M,
                                            opt.early_exit != 0, opt.sched, stage);
                issued += got;
            }
            // a scout window of the read was valid (it was probed by the scout pass)
            const bool scout_saw = opt.sched == SCHED_PRESCOUT && (bb.live[i] & 2u);
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            if (ntiles == 1) {
                // the whole read was in this tile: resolve from its masks
                if (got == 0 && !scout_saw && lane == 0) atomicAdd(opt.emptyq, 1ULL);
                answer_read(ix, M, res, o, lane, opt.rmode, opt.counts, i, opt.wm);
                __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
                __builtin_amdgcn_wave_barrier();
                continue;
            }
            // Publish this tile's masks, then count the tile done. Every
            // access to rm and done is an agent-scope atomic read-modify-write,
            // performed at the device's point of coherence (one for all XCDs),
            // and a returning RMW's old value comes back only once the RMW has
            // been performed there. The ANDs return their old values, the
            // wave folds them into one value (a ballot over every lane's
            // results) and the count's operand is made to depend on it, so
            // the count is issued only after each of this tile's ANDs has
            // been performed. The last tile issues its mask reads only after
            // its own count has returned, i.e. after every other tile's count
            // and hence after every other tile's ANDs. (A release fence at
            // agent scope would also order them, but on a multi-XCD device it
            // writes back the XCD's whole L2, which made small tiles 4.5x
            // slower; nothing here needs it, as no plain store is published.)
            uint32_t olds = 0;
            if (!skip) {
                for (uint32_t w = lane; w < mw; w += 64) {
                    const uint32_t v = M[w];
                    if (v != 0xFFFFFFFFu)
                        olds |= __hip_atomic_fetch_and(rm + w, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                }
            }
            // (a skipped tile belongs to a read whose answer is empty anyway:
            // it counts as holding a valid window)
            const unsigned long long inc = 1ull + ((got > 0 || skip) ? (1ull << 32) : 0ull);
            const uint32_t zero = opaque_zero(__ballot(olds != 0));
            unsigned long long prev = 0;
            if (lane == 0)
                prev = __hip_atomic_fetch_add(bb.done + i, inc + zero, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            prev = uniform64(__shfl(prev, 0));
            if ((prev & 0xFFFFFFFFull) + 1 == ntiles) {
                if ((prev >> 32) + (inc >> 32) == 0 && !scout_saw && lane == 0) atomicAdd(opt.emptyq, 1ULL);
                // last tile of read i: read the masks with atomic RMWs too,
                // at the same point of coherence as the ANDs
                for (uint32_t w = lane; w < mw; w += 64)
                    M[w] = __hip_atomic_fetch_or(rm + w, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
                __builtin_amdgcn_wave_barrier();
                answer_read(ix, M, res, o, lane, opt.rmode, opt.counts, i, opt.wm);
                __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
                __builtin_amdgcn_wave_barrier();
            }
        }
    }
    if (opt.probes && lane == 0 && issued) atomicAdd(opt.probes, (unsigned long long)(issued * ix.eta));
}


// Resident workgroups per compute unit of a kernel at a launch shape, asked of
// the runtime once per shape.
template <class F>
static int resident(rambo_s *h, uint64_t key, F kernel, int threads, size_t lds, int *fit) {
    auto it = h->resident.find(key);
    if (it == h->resident.end()) {
        int f = 0;
        HIP_CHECK(hipOccupancyMaxActiveBlocksPerMultiprocessor(&f, kernel, threads, lds));
        it = h->resident.emplace(key, std::max(1, f)).first;
    }
    *fit = it->second;
    return RAMBO_OK;
}

// Result words of a batch, with rows split over 8 or more lanes, from which the
// zero bitsets of the reads that the scout pass ends are left to k_batch_zero: in
// the scout pass a wave waits for the rows it writes, from here on that costs more
// than the launch (K=101,000, 12.6 KB a read, whole calls, us: 1,200 reads 88
// without and 94 with it, 5,000 96 / 100, 10,000 121 / 118, 20,000 185 / 178,
// 100,000 574-598 / 530, 10^6 5,057 / 4,429).
static constexpr uint64_t kZeroApart = 1 << 24;

// Scout pass and queue of a batch of up to n reads (n <= bg.cap); with val, a
// direct launch of that batch.
static int enqueue_prep(rambo_s *h, const Tune &tu, BatchGraph &bg, uint64_t n, const InputHdr *val, uint64_t *out,
                        const IdsOut &io, hipStream_t s) {
    const uint32_t mw = h->R * h->RW;
    const bool pre = tu.sched == SCHED_SCOUT;
    const bool one = n <= 2048;
    const InputHdr hd = val ? *val : InputHdr{};
    InputHdr *own = val ? bg.own : nullptr;
    if (!pre && (!one || own)) hipLaunchKernelGGL(k_batch_reset, dim3(1), dim3(64), 0, s, bg.bb, hd, own);
    HIP_CHECK(hipGetLastError());
    if (pre) {
        const Index ix = make_index(h);
        const int G = (int)h->RW / tu.seg;
        // a grid of what fits on the device at once strides over the reads
        // (a captured graph, whose batches are mostly smaller than n, keeps one kernel)
        const bool apart = val && !io.counts && G >= 8 && n * h->W >= kZeroApart;
        // without rows to write, narrow groups, where each has two reads or more
        // (in the setting above 20,000 reads 178 with wide groups and 197 with narrow
        // ones, 100,000 530 / 529, 200,000 987 / 956, 10^6 4,429 / 4,233)
        const bool narrow =
            io.counts != nullptr || (apart && n * (uint64_t)G >= 2 * (uint64_t)h->n_cu * 2048);
        const uint64_t GS = (uint64_t)scout_group(G, narrow);
        int fit = 0, st = RAMBO_OK;
        const uint64_t key = ((uint64_t)G << 16) | ((uint64_t)tu.seg << 8) | (narrow ? 2u : 1u);
#define RAMBO_SPLIT_BODY_                                                                                    \
    st = narrow ? resident(h, key, k_batch_scout<SEG, G, 1>, 256, 0, &fit)                                   \
                : resident(h, key, k_batch_scout<SEG, G, 0>, 256, 0, &fit)
        RAMBO_DISPATCH_SPLIT(tu.seg, G)
#undef RAMBO_SPLIT_BODY_
        if (st != RAMBO_OK) return st;
        const uint64_t blocks = std::max<uint64_t>(
            1, std::min<uint64_t>((n * GS + 255) / 256, (uint64_t)fit * h->n_cu));
        QueryOpts opt{h->resolve, h->early_exit, h->probe_counter, tu.sched, io.counts,
                      io.counts ? io.noterm : h->d_emptyq};
#define RAMBO_SPLIT_BODY_                                                                                   \
    if (narrow)                                                                                             \
        hipLaunchKernelGGL((k_batch_scout<SEG, G, 1>), dim3((unsigned)blocks), dim3(256), 0, s, ix, bg.in, out,   \
                           bg.bb, opt, hd, own, !apart);                                                             \
    else                                                                                                     \
        hipLaunchKernelGGL((k_batch_scout<SEG, G, 0>), dim3((unsigned)blocks), dim3(256), 0, s, ix, bg.in, out,   \
                           bg.bb, opt, hd, own, !apart)
        RAMBO_DISPATCH_SPLIT(tu.seg, G)
#undef RAMBO_SPLIT_BODY_
        HIP_CHECK(hipGetLastError());
        if (apart) {
            hipLaunchKernelGGL(k_batch_zero, dim3((unsigned)std::min<uint64_t>((n + 31) / 32, (uint64_t)h->n_cu * 8)),
                               dim3(256), 0, s, bg.in, bg.bb.live, out, (uint64_t)h->W);
            HIP_CHECK(hipGetLastError());
        }
    }
    const uint32_t most = (uint32_t)tu.tile;
    const uint32_t least = std::min(most, std::max<uint32_t>(64, 512 / (uint32_t)std::max(1, (int)h->RW / tu.seg)));
    if (one) {
        hipLaunchKernelGGL((k_batch_prep<2, 1024, true>), dim3(1), dim3(1024), 0, s, bg.in, mw, h->RW, least, most,
                           bg.bb, pre ? 1 : 0, bg.parts);
        HIP_CHECK(hipGetLastError());
        return RAMBO_OK;
    }
    // four reads per thread once one per thread would take over eight
    // workgroups per compute unit
    const uint32_t per = (n + 255) / 256 > 8 * (uint64_t)h->n_cu ? 4 : 1;
    const dim3 grid((unsigned)((n + 256 * per - 1) / (256 * per)));
    if (per == 4)
        hipLaunchKernelGGL((k_batch_prep<4, 256, false>), grid, dim3(256), 0, s, bg.in, mw, h->RW, least, most,
                           bg.bb, pre ? 1 : 0, bg.parts);
    else
        hipLaunchKernelGGL((k_batch_prep<1, 256, false>), grid, dim3(256), 0, s, bg.in, mw, h->RW, least, most,
                           bg.bb, pre ? 1 : 0, bg.parts);
    HIP_CHECK(hipGetLastError());
    // the header's first field is the number of reads
    return launch_scan_parts(bg.bb.extra, &bg.in->n, n, bg.bb.extra_off, bg.parts, per, s);
}

static int enqueue_main(rambo_s *h, const Tune &tu, BatchGraph &bg, uint64_t *out, hipStream_t s, const IdsOut &io) {
    const Index ix = make_index(h);
    const uint32_t mw = h->R * h->RW;
    const int G = (int)h->RW / tu.seg;
    const int use_res = seq_lds_result(h->W) ? 1 : 0;
    const size_t lds = (size_t)tu.wpb * wave_lds(mw, h->W, use_res != 0, false).total * 4;
    // the scout schedule has run its scout windows in the scout pass already
    const int ksched = tu.sched == SCHED_SCOUT ? SCHED_PRESCOUT : tu.sched;
    QueryOpts opt{h->resolve, h->early_exit, h->probe_counter, ksched, io.counts,
                  io.counts ? io.noterm : h->d_emptyq, nullptr, io.counts ? io.wm : nullptr};
    // a persistent grid must be resident: never more workgroups than fit
    const uint64_t key = ((uint64_t)lds << 32) | ((uint64_t)G << 16) | ((uint64_t)tu.seg << 8) | (uint64_t)(4 + tu.wpb);
#define RAMBO_SPLIT_BODY_                                                                                  \
    {                                                                                                      \
        int fit = 0;                                                                                       \
        const int st = resident(h, key, k_batch_main<SEG, G>, 64 * tu.wpb, lds, &fit);                     \
        if (st != RAMBO_OK) return st;                                                                     \
        const int per_cu = std::max(1, std::min(fit, tu.waves_per_cu / tu.wpb));                         \
        bg.blocks = (unsigned)(h->n_cu * per_cu);                                                          \
        hipLaunchKernelGGL((k_batch_main<SEG, G>), dim3(bg.blocks), dim3(64 * tu.wpb), lds, s, ix, bg.in, out,  \
                           bg.bb, opt, use_res, (uint32_t)tu.grab);                  \
    }
    RAMBO_DISPATCH_SPLIT(tu.seg, G)
#undef RAMBO_SPLIT_BODY_
    HIP_CHECK(hipGetLastError());
    return RAMBO_OK;
}

BatchEvents::~BatchEvents() {
    for (auto &x : e)
        if (x) (void)hipEventDestroy(x);
}

static int make_events(std::shared_ptr<BatchEvents> &res) {
    auto ev = std::make_shared<BatchEvents>();
    for (auto &x : ev->e) HIP_CHECK(hipEventCreate(&x));
    res = ev;
    return RAMBO_OK;
}

BatchGraph::~BatchGraph() {
    if (exec_prep) (void)hipGraphExecDestroy(exec_prep);
    if (exec_main) (void)hipGraphExecDestroy(exec_main);
    if (graph_prep) (void)hipGraphDestroy(graph_prep);
    if (graph_main) (void)hipGraphDestroy(graph_main);
    if (mem) (void)hipFree(mem);
}

static int capture(rambo_s *h, hipGraph_t *g, hipGraphExec_t *exec, const std::function<int(hipStream_t)> &body) {
    HIP_CHECK(hipStreamBeginCapture(h->aux, hipStreamCaptureModeThreadLocal));
    int st = body(h->aux);
    hipGraph_t gg = nullptr;
    hipError_t e = hipStreamEndCapture(h->aux, &gg);
    if (st != RAMBO_OK) {
        if (gg) (void)hipGraphDestroy(gg);
        return st;
    }
    if (e != hipSuccess) return fail(RAMBO_EDEVICE, "graph capture failed: %s", hipGetErrorString(e));
    *g = gg;
    HIP_CHECK(hipGraphInstantiate(exec, gg, nullptr, nullptr, 0));
    return RAMBO_OK;
}

// Queue position, class counters, work left and tile: a 128-byte line each.
constexpr size_t kHeadBytes = 128 * (1 + 4 + kWorkParts + 1);

// Queue state for up to cap reads; without an external header, one of its own.
static int alloc_state(rambo_s *h, BatchGraph &bg, uint64_t cap, bool batch_bufs, const InputHdr *in_dev) {
    const size_t mw = (size_t)h->R * h->RW;
    auto al = [](size_t x) { return (x + 255) & ~(size_t)255; };
    size_t b_mask = 0, b_done = 0, b_extra = 0, b_off = 0, b_parts = 0, b_order = 0, b_smask = 0, b_live = 0;
    if (batch_bufs) {
        b_smask = al(cap * h->RW * 4);
        b_live = al(cap * 4);
        b_mask = al(cap * mw * 4);
        b_done = al(cap * 8);
        b_extra = al(cap * 8);
        b_off = al((cap + 1) * 8);
        b_parts = al(scan_parts_needed(cap, 1) * 8);
        b_order = al(4 * cap * 4);
    }
    const size_t total = b_mask + b_done + b_extra + b_off + b_parts + b_order + b_smask + b_live + kHeadBytes + 256;
    if (hipMalloc(&bg.mem, total) != hipSuccess) {
        (void)hipGetLastError();
        bg.mem = nullptr;
        return fail(RAMBO_ENOMEM, "cannot allocate %llu bytes for a batch's queue", (unsigned long long)total);
    }
    char *p = (char *)bg.mem;
    bg.bb.smask = b_smask ? (uint32_t *)p : nullptr; p += b_smask;
    bg.bb.live = b_live ? (uint32_t *)p : nullptr; p += b_live;
    bg.parts = (uint64_t *)p; p += b_parts;
    bg.bb.rmask = (uint32_t *)p; p += b_mask;
    bg.bb.done = (unsigned long long *)p; p += b_done;
    bg.bb.extra = (uint64_t *)p; p += b_extra;
    bg.bb.extra_off = (uint64_t *)p; p += b_off;
    bg.bb.order = (uint32_t *)p; p += b_order;
    bg.bb.head = (unsigned long long *)p;  // its own 128-byte line (every wave's queue atomic)
    bg.bb.cls = bg.bb.head + 16;           // class v at cls[16 v]: the next four lines
    bg.bb.work = bg.bb.cls + 4 * 16;       // part v at work[16 v]
    bg.bb.tile = (uint32_t *)(bg.bb.work + kWorkParts * 16);
    p += kHeadBytes;
    bg.bb.cap = cap;
    bg.cap = cap;
    bg.own = in_dev ? nullptr : (InputHdr *)p;
    bg.in = in_dev ? in_dev : bg.own;
    // launches of the query entry point are timed (rambo_last_batch_ms); the
    // server's graphs are not (three fewer operations per batch)
    return in_dev ? RAMBO_OK : make_events(bg.ev);
}

int make_batch_graph(rambo_s *h, const Tune &tu, const InputHdr *in_dev, uint64_t cap, uint64_t *out,
                     std::shared_ptr<BatchGraph> &res) {
    auto bg = std::make_shared<BatchGraph>();
    bg->tune = tu;
    std::lock_guard<std::mutex> g(h->mu);
    int st = alloc_state(h, *bg, cap, true, in_dev);
    if (st != RAMBO_OK) return st;
    hipLaunchKernelGGL(k_batch_reset, dim3(1), dim3(64), 0, h->aux, bg->bb, InputHdr{}, (InputHdr *)nullptr);
    HIP_CHECK(hipGetLastError());
    HIP_CHECK(hipStreamSynchronize(h->aux));
    if (st == RAMBO_OK)
        st = capture(h, &bg->graph_prep, &bg->exec_prep,
                     [&](hipStream_t s) { return enqueue_prep(h, tu, *bg, cap, nullptr, out, IdsOut(), s); });
    if (st == RAMBO_OK)
        st = capture(h, &bg->graph_main, &bg->exec_main,
                     [&](hipStream_t s) { return enqueue_main(h, tu, *bg, out, s, IdsOut()); });
    if (st != RAMBO_OK) return st;
    res = bg;
    return RAMBO_OK;
}

int make_plain_graph(rambo_s *h, const InputHdr *in_dev, uint64_t cap, uint64_t *out,
                     std::shared_ptr<BatchGraph> &res) {
    auto bg = std::make_shared<BatchGraph>();
    int st = alloc_state(h, *bg, cap, false, in_dev);
    if (st == RAMBO_OK)
        st = capture(h, &bg->graph_main, &bg->exec_main, [&](hipStream_t s) {
            return launch_query_seqs_plain(h, nullptr, nullptr, cap, out, s, default_seg(h->RW), bg->in);
        });
    if (st != RAMBO_OK) return st;
    res = bg;
    return RAMBO_OK;
}

int launch_batch_graph(rambo_s *h, BatchGraph &bg, hipStream_t s) {
    (void)h;
    if (bg.exec_prep) HIP_CHECK(hipGraphLaunch(bg.exec_prep, s));
    HIP_CHECK(hipGraphLaunch(bg.exec_main, s));
    return RAMBO_OK;
}

// Queue state for a call of n reads on stream s, from the handle's pool: one
// whose last call was on s (the new call follows it) or has ended, of the fewest
// reads that hold n; otherwise a new one, up to kPool of them (the ended ones
// that are too small are freed first); otherwise, of those that hold n, the one
// whose call was launched first, which s then waits for (or, if none does, the
// first launched of all, replaced by a larger one). Called with h->mu held.
constexpr size_t kPool = 16;
static int take_state(rambo_s *h, uint64_t n, hipStream_t s, std::shared_ptr<BatchGraph> &res) {
    auto &pool = h->batch_pool;
    auto ended = [](const BatchGraph &b) { return hipEventQuery(b.ev->e[2]) == hipSuccess; };
    size_t best = pool.size();
    for (size_t k = 0; k < pool.size(); k++)
        if (pool[k]->cap >= n && (best == pool.size() || pool[k]->cap < pool[best]->cap) &&
            (!pool[k]->used || pool[k]->stream == s || ended(*pool[k])))
            best = k;
    if (best == pool.size()) {
        (void)hipGetLastError();  // (a query that found work still running)
        for (size_t k = 0; k < pool.size();)
            if (pool[k]->cap < n && ended(*pool[k])) pool.erase(pool.begin() + k);
            else k++;
        (void)hipGetLastError();
        uint64_t cap = std::max<uint64_t>(n, 4096);
        if (pool.size() >= kPool) {
            best = 0;
            for (size_t k = 1; k < pool.size(); k++) {
                const bool fits = pool[k]->cap >= n, had = pool[best]->cap >= n;
                if (fits != had ? fits : pool[k]->turn < pool[best]->turn) best = k;
            }
            if (pool[best]->cap < n) {
                HIP_CHECK(hipEventSynchronize(pool[best]->ev->e[2]));
                pool.erase(pool.begin() + best);
                best = pool.size();
                cap = n;
            }
        }
        if (pool.size() < kPool) {
            auto bg = std::make_shared<BatchGraph>();
            int st = alloc_state(h, *bg, cap, true, nullptr);
            if (st == RAMBO_ENOMEM) {
                give_back(h, true);
                bg = std::make_shared<BatchGraph>();
                st = alloc_state(h, *bg, n, true, nullptr);
            }
            if (st != RAMBO_OK) return st;
            pool.push_back(bg);
            best = pool.size() - 1;
        }
    }
    (void)hipGetLastError();
    res = pool[best];
    if (res->used) HIP_CHECK(hipStreamWaitEvent(s, res->ev->e[2], 0));
    return RAMBO_OK;
}

// One batch: its kernels launched directly, whatever buffers it comes in.
static int run_batch(rambo_s *h, const Tune &tu, const uint8_t *seqs, const uint64_t *offs, uint64_t n, uint64_t *out,
                     hipStream_t s, const IdsOut &io = IdsOut(), bool note = true) {
    std::lock_guard<std::mutex> g(h->mu);
    std::shared_ptr<BatchGraph> bg;
    int st = take_state(h, n, s, bg);
    if (st != RAMBO_OK) return st;
    // (the last batched call keeps its times)
    if (!note && h->last_ev == bg->ev && (st = make_events(bg->ev)) != RAMBO_OK) return st;
    const InputHdr val{n, offs, seqs, 0};
    const hipEvent_t *ev = bg->ev->e;
    HIP_CHECK(hipEventRecord(ev[0], s));
    if (!bg->used) {
        hipLaunchKernelGGL(k_batch_reset, dim3(1), dim3(64), 0, s, bg->bb, val, (InputHdr *)nullptr);
        HIP_CHECK(hipGetLastError());
    }
    st = enqueue_prep(h, tu, *bg, n, &val, out, io, s);
    if (st == RAMBO_OK) {
        HIP_CHECK(hipEventRecord(ev[1], s));
        st = enqueue_main(h, tu, *bg, out, s, io);
    }
    HIP_CHECK(hipEventRecord(ev[2], s));
    bg->stream = s;
    bg->used = true;
    bg->turn = ++h->batch_turns;
    if (st == RAMBO_OK && note) {
        h->last_graph = bg;
        h->last_ev = bg->ev;
    }
    return st;
}

void drop_ended_states(rambo_s *h) {
    auto &pool = h->batch_pool;
    for (size_t k = 0; k < pool.size();)
        if (hipEventQuery(pool[k]->ev->e[2]) == hipSuccess) pool.erase(pool.begin() + k);
        else k++;
    (void)hipGetLastError();  // (a query that found work still running)
    h->last_graph.reset();
}

void drop_graphs(rambo_s *h) {
    h->batch_pool.clear();
    h->resident.clear();
    h->last_graph.reset();
    h->last_ev.reset();
}

// ---------------------------------------------------------------------------
// autotuner: coordinate search over the launch shape on the caller's batch
// (every candidate computes the same bits), cached per index shape.
// ---------------------------------------------------------------------------
bool tune_valid(const rambo_s *h, const Tune &t) {
    return (t.seg == 1 || t.seg == 2 || t.seg == 4) && (int)h->RW % t.seg == 0 &&
           split_supported(t.seg, (int)h->RW / t.seg) && t.tile >= 64 && t.tile % 64 == 0 && t.tile <= (1 << 20) &&
           t.waves_per_cu >= 1 && t.waves_per_cu <= 64 && (t.wpb == 1 || t.wpb == 2 || t.wpb == 4) && t.grab >= 1 &&
           t.grab <= 64 && t.sched >= 0 && t.sched <= 2;
}

static std::string tune_key(const rambo_s *h) {
    hipDeviceProp_t prop;
    const char *arch = "gpu";
    if (hipGetDeviceProperties(&prop, h->device) == hipSuccess) arch = prop.gcnArchName;
    char buf[256];
    snprintf(buf, sizeof buf, "%s K=%llu B=%u R=%u eta=%u m=%llu ee=%d", arch, (unsigned long long)h->K, h->B, h->R,
             h->eta, (unsigned long long)h->m, h->early_exit);
    std::string s = buf;
    for (auto &c : s)
        if (c == ':' || c == '|') c = '_';
    return s;
}

static bool tune_cache_load(rambo_s *h) {
    const char *path = getenv("RAMBO_TUNE_CACHE");
    if (!path) return false;
    std::ifstream f(path);
    std::string line, key = tune_key(h);
    while (std::getline(f, line)) {
        const size_t bar = line.find('|');
        if (bar == std::string::npos || line.substr(0, bar) != key) continue;
        Tune t;
        if (sscanf(line.c_str() + bar + 1, "%d %d %d %d %d %d", &t.seg, &t.tile, &t.waves_per_cu, &t.wpb, &t.grab,
                   &t.sched) == 6 &&
            tune_valid(h, t)) {
            h->tune = t;
            return true;
        }
    }
    return false;
}

static void tune_cache_store(const rambo_s *h) {
    const char *path = getenv("RAMBO_TUNE_CACHE");
    if (!path) return;
    std::ofstream f(path, std::ios::app);
    f << tune_key(h) << "|" << h->tune.seg << " " << h->tune.tile << " " << h->tune.waves_per_cu << " "
      << h->tune.wpb << " " << h->tune.grab << " " << h->tune.sched << "\n";
}

static int time_candidate(rambo_s *h, const Tune &tu, const uint8_t *seqs, const uint64_t *offs, uint64_t n,
                          uint64_t *out, hipStream_t s, float &best_ms) {
    hipEvent_t a, b;
    HIP_CHECK(hipEventCreate(&a));
    HIP_CHECK(hipEventCreate(&b));
    int st = run_batch(h, tu, seqs, offs, n, out, s);  // warm-up (and queue state)
    if (st == RAMBO_OK) st = run_batch(h, tu, seqs, offs, n, out, s);
    float best = 1e30f;
    for (int rep = 0; rep < 5 && st == RAMBO_OK; rep++) {
        (void)hipEventRecord(a, s);
        st = run_batch(h, tu, seqs, offs, n, out, s);
        (void)hipEventRecord(b, s);
        if (hipEventSynchronize(b) != hipSuccess) st = fail(RAMBO_EDEVICE, "autotune: run failed");
        float ms = 0;
        if (st == RAMBO_OK) {
            (void)hipEventElapsedTime(&ms, a, b);
            best = std::min(best, ms);
        }
    }
    (void)hipEventDestroy(a);
    (void)hipEventDestroy(b);
    best_ms = best;
    return st;
}

// Windows per item of the last batch (which has ended).
static int last_tile(rambo_s *h, uint32_t *tile) {
    std::lock_guard<std::mutex> g(h->mu);
    *tile = ~0u;
    if (!h->last_graph) return RAMBO_OK;
    HIP_CHECK(hipMemcpy(tile, h->last_graph->bb.tile, sizeof *tile, hipMemcpyDeviceToHost));
    return RAMBO_OK;
}

int autotune(rambo_s *h, const uint8_t *seqs, const uint64_t *offs, uint64_t n, uint64_t *out, hipStream_t s) {
    Tune best = h->tune;
    best.seg = default_seg(h->RW);
    float best_ms = 0;
    int st = time_candidate(h, best, seqs, offs, n, out, s, best_ms);
    if (st != RAMBO_OK) return st;
    const char *vb = getenv("RAMBO_TUNE_VERBOSE");
    const bool verbose = vb && vb[0] == '1';
    if (verbose)
        fprintf(stderr, "rambo autotune: seg=%d tile=%d waves/CU=%d wpb=%d grab=%d sched=%d -> %.3f ms (start)\n",
                best.seg, best.tile, best.waves_per_cu, best.wpb, best.grab, best.sched, best_ms);
    auto consider = [&](Tune t) -> int {
        if (!tune_valid(h, t)) return RAMBO_OK;
        float ms = 0;
        int st2 = time_candidate(h, t, seqs, offs, n, out, s, ms);
        if (st2 != RAMBO_OK) return st2;
        if (verbose)
            fprintf(stderr, "rambo autotune: seg=%d tile=%d waves/CU=%d wpb=%d grab=%d sched=%d -> %.3f ms\n", t.seg,
                    t.tile, t.waves_per_cu, t.wpb, t.grab, t.sched, ms);
        if (ms < best_ms * 0.98f) {
            best = t;
            best_ms = ms;
        }
        return RAMBO_OK;
    };
    // two rounds of coordinate search (the second revisits every axis from
    // the first round's shape); a candidate must beat the best by 2 %
    for (int round = 0; round < 2; round++) {
        int cut = 1 << 30;  // the tile that the batch's larger ones are cut to, once seen
        for (int tile : {128, 256, 512, 1024, 2048, 4096}) {
            Tune t = best; t.tile = tile;
            if (std::min(t.tile, cut) == std::min(best.tile, cut)) continue;
            if ((st = consider(t))) return st;
            uint32_t ran = 0;
            if ((st = last_tile(h, &ran))) return st;
            if ((int)ran < t.tile) cut = (int)ran;
        }
        for (int wpc : {8, 12, 16, 20, 24, 32}) {
            Tune t = best; t.waves_per_cu = wpc;
            if (t.waves_per_cu != best.waves_per_cu && (st = consider(t))) return st;
        }
        for (int seg : {1, 2, 4}) { Tune t = best; t.seg = seg; if (t.seg != best.seg && (st = consider(t))) return st; }
        for (int grab : {1, 2, 4, 16}) {
            Tune t = best; t.grab = grab;
            if (t.grab != best.grab && (st = consider(t))) return st;
        }
        for (int wpb : {1, 2, 4}) { Tune t = best; t.wpb = wpb; if (t.wpb != best.wpb && (st = consider(t))) return st; }
        for (int sched : {0, 1, 2}) {
            Tune t = best; t.sched = sched;
            if (sched != best.sched && (st = consider(t))) return st;
        }
    }
    std::lock_guard<std::mutex> g(h->mu);
    h->tune = best;
    return RAMBO_OK;
}

int query_seqs_batched(rambo_s *h, const uint8_t *seqs, const uint64_t *offs, uint64_t n, uint64_t *out,
                       hipStream_t s, const IdsOut &io) {
    // under capture the plain kernel, which needs no state of the handle
    hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(s, &cap) == hipSuccess && cap != hipStreamCaptureStatusNone)
        return launch_query_seqs_plain(h, seqs, offs, n, out, s, default_seg(h->RW), nullptr, io);
    if (!h->tuned) {
        h->tune.seg = default_seg(h->RW);
        const char *mode = getenv("RAMBO_TUNE");
        const bool off = mode && !strcmp(mode, "off");
        if (!off && !tune_cache_load(h)) {
            int st = autotune(h, seqs, offs, n, out, s);
            if (st != RAMBO_OK) return st;
            tune_cache_store(h);
        }
        h->tuned = true;
    }
    Tune tu;
    {
        std::lock_guard<std::mutex> g(h->mu);
        tu = h->tune;
    }
    return run_batch(h, tu, seqs, offs, n, out, s, io);
}

// Plain-form queries: the plain kernels, or, from the size on where they no
// longer keep the chip busy, the batched form's in their default shape -- a
// long read is one wave's (or one workgroup's) work in the plain kernels, which
// the others' end waits for. Measured, plain kernels against batched launches,
// us: K=10,000 (a lane a term) 1,000 reads 62 / 86, 2,000 109 / 95, 4,000 167 /
// 121, 16,000 554 / 290, 100,000 1,775 / 1,353; K=101,000 (8 lanes) 2,000 63 / 93,
// 4,000 104 / 105, 8,000 203 / 106, 100,000 895 / 588. Under capture, with the
// RAMBO+ tallies and without memory for the queue the plain kernels run.
int query_seqs_plain(rambo_s *h, const uint8_t *seqs, const uint64_t *offs, uint64_t n, uint64_t *out, hipStream_t s,
                     const IdsOut &io) {
    Tune tu;
    tu.seg = default_seg(h->RW);
    tu.sched = h->tune.sched;
    const bool lane_rows = h->RW <= 4;  // a lane holds a whole row
    hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
    if (n > (lane_rows ? 6 : 16) * (uint64_t)h->n_cu && !h->sparse_counter &&
        hipStreamIsCapturing(s, &cap) == hipSuccess && cap == hipStreamCaptureStatusNone) {
        const int st = run_batch(h, tu, seqs, offs, n, out, s, io, false);
        if (st != RAMBO_ENOMEM) return st;
    }
    return launch_query_seqs_plain(h, seqs, offs, n, out, s, tu.seg, nullptr, io);
}

}  // namespace rambo

using namespace rambo;

RAMBO_API int rambo_autotune(rambo_t *h, const uint8_t *seqs, const uint64_t *offsets, uint64_t n, uint64_t *out,
                             void *stream) {
    if (!h || !seqs || !offsets || !out || n == 0) return fail(RAMBO_EINVAL, "rambo_autotune: bad argument");
    int st = autotune(h, seqs, offsets, n, out, (hipStream_t)stream);
    if (st == RAMBO_OK) h->tuned = true;
    return st;
}

RAMBO_API int rambo_last_batch_ms(rambo_t *h, float *graph_ms, float *kernel_ms) {
    if (!h || !graph_ms || !kernel_ms) return fail(RAMBO_EINVAL, "rambo_last_batch_ms: null argument");
    std::shared_ptr<BatchEvents> ev;
    {
        std::lock_guard<std::mutex> g(h->mu);
        ev = h->last_ev;
    }
    if (!ev) return fail(RAMBO_EINVAL, "rambo_last_batch_ms: no batched launch yet");
    HIP_CHECK(hipEventSynchronize(ev->e[2]));
    // (read under the lock: another thread's batch may have taken the state and its
    // events meanwhile; then it is the most recent one, and waited for)
    std::lock_guard<std::mutex> g(h->mu);
    if (h->last_ev) ev = h->last_ev;
    HIP_CHECK(hipEventSynchronize(ev->e[2]));
    HIP_CHECK(hipEventElapsedTime(graph_ms, ev->e[0], ev->e[2]));
    HIP_CHECK(hipEventElapsedTime(kernel_ms, ev->e[1], ev->e[2]));
    return RAMBO_OK;
}

RAMBO_API int rambo_get_tune(const rambo_t *h, rambo_tune_t *t) {
    if (!h || !t) return fail(RAMBO_EINVAL, "rambo_get_tune: null argument");
    t->seg = h->tune.seg;
    t->tile = h->tune.tile;
    t->waves_per_cu = h->tune.waves_per_cu;
    t->wpb = h->tune.wpb;
    t->grab = h->tune.grab;
    t->sched = h->tune.sched;
    t->tuned = h->tuned ? 1 : 0;
    return RAMBO_OK;
}

RAMBO_API int rambo_set_tune(rambo_t *h, const rambo_tune_t *t) {
    if (!h || !t) return fail(RAMBO_EINVAL, "rambo_set_tune: null argument");
    Tune tu;
    tu.seg = t->seg;
    tu.tile = t->tile;
    tu.waves_per_cu = t->waves_per_cu;
    tu.wpb = t->wpb;
    tu.grab = t->grab;
    tu.sched = t->sched;
    if (!tune_valid(h, tu)) return fail(RAMBO_EINVAL, "rambo_set_tune: launch shape out of range");
    std::lock_guard<std::mutex> g(h->mu);
    h->tune = tu;
    h->tuned = true;
    return RAMBO_OK;
}
