// Plain one-batch sequence queries (Algorithm 2, Section 3.3.1) and the
// bitset -> id-list compaction.
//
// Per term: R * eta row reads (one per Bloom hash and repetition), ANDed
// over j into the B-bit mask M_r of positive BFUs of repetition r. A
// sequence ANDs the masks of its terms across the lanes of its wave and
// stops at the first repetition whose mask is empty. The per-document AND
// over repetitions ("resolve") runs on the masks staged in LDS.
#include "rambo_int.h"
#include "scan.h"

namespace rambo {


// -------------------------------------------------------------------------
// sequence queries, plain form: one wave per read, 64 windows per step
// -------------------------------------------------------------------------
template <int SEG, int G, bool RPLUS>
__global__ __launch_bounds__(256) void k_query_seqs_plain(Index ix, const uint8_t *__restrict__ seqs,
                                                          const uint64_t *__restrict__ offs, uint64_t n,
                                                          const InputHdr *hdr, uint64_t *__restrict__ out,
                                                          QueryOpts opt, int use_res) {
    if (hdr) {  // batch described in device memory (graph replays)
        n = hdr->n;
        offs = hdr->offs;
        seqs = hdr->seqs;
    }
    extern __shared__ __align__(16) uint64_t smem64[];
    const uint32_t lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const WaveLds L = wave_lds(ix.R * ix.RW, ix.W, use_res != 0, opt.sched == SCHED_SCOUT);
    uint32_t *M = reinterpret_cast<uint32_t *>(smem64) + wave * L.total;
    uint64_t *res = use_res ? reinterpret_cast<uint64_t *>(M + L.res) : nullptr;
    uint8_t *stage = opt.sched == SCHED_SCOUT ? reinterpret_cast<uint8_t *>(M + L.stage) : nullptr;

    const uint64_t read = (uint64_t)blockIdx.x * (blockDim.x >> 6) + wave;
    if (read >= n) return;
    const uint64_t beg = offs[read];
    uint64_t end = offs[read + 1];
    if (end < beg) end = beg;
    const uint64_t nwin = end - beg >= 31 ? end - beg - 30 : 0;

    init_masks(ix, M, lane);
    const uint64_t issued = probe_windows<SEG, G, RPLUS>(ix, seqs, beg, end, 0, nwin, lane, M, opt.early_exit != 0,
                                                         opt.sched, stage, opt.rplus);
    if (opt.probes && lane == 0 && issued) atomicAdd(opt.probes, (unsigned long long)(issued * ix.eta));
    // every valid window is probed at least in repetition 0 unless a probe
    // has ended the read first, so nothing issued means no valid window
    if (issued == 0 && lane == 0) atomicAdd(opt.emptyq, 1ULL);
    uint64_t *o = out + read * ix.W;
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    answer_read(ix, M, res, o, lane, opt.rmode, opt.counts, read, opt.wm);
}

// As k_query_seqs_plain with a workgroup of up to 16 waves per read, for batches
// too small to fill the chip with one wave per read: the waves share the
// read's windows (each a contiguous part, repetition 0 first) in masks of their
// own, which are then ANDed, and resolve it together. Bound by the chain of
// round trips of the longest read (offsets, bytes, repetition 0's rows, the
// other repetitions' rows, the resolve): with one wave per read a read of
// 1,500 bases took 24 steps of 64 windows one after the other, here two (16
// reads at K=10,000: 53 us a call, now 21).
//
// With early exit the waves first scout (repetition 0 on 64 windows 31 apart, then
// on the rest of those) where the parts take many steps, or where the batch's
// rows are what it waits for (kTeamScout bases, about 8 us of rows): most reads
// that no document holds end there. Without, 4,000 reads of 10 kbp with an error
// in a thousand bases took 789 us at K=101,000, now 60 (55 with one wave per read,
// which scouts), 257 of 1 kbp with one in a hundred 41, now 27. Elsewhere the
// scouts' round trip would only make the reads that live wait (id lists of 257
// reads of median 300: 83 us without, 86 with scouts in the longer reads).
constexpr uint64_t kTeamScout = 3 << 16;
template <int SEG, int G>
__global__ __launch_bounds__(1024) void k_query_seqs_team(Index ix, const uint8_t *__restrict__ seqs,
                                                          const uint64_t *__restrict__ offs, uint64_t n,
                                                          const InputHdr *hdr, uint64_t *__restrict__ out,
                                                          QueryOpts opt, int use_res) {
    if (hdr) {
        n = hdr->n;
        offs = hdr->offs;
        seqs = hdr->seqs;
    }
    const uint64_t read = blockIdx.x;
    if (read >= n) return;
    extern __shared__ __align__(16) uint64_t smem64[];
    __shared__ unsigned long long issued, kept;
    const uint32_t lane = threadIdx.x & 63, wave = threadIdx.x >> 6, waves = blockDim.x >> 6;
    const uint32_t mw = ix.R * ix.RW, pitch = wave_lds(mw, ix.W, false, false).total;
    uint32_t *M0 = reinterpret_cast<uint32_t *>(smem64), *M = M0 + wave * pitch;
    uint64_t *res = use_res ? reinterpret_cast<uint64_t *>(M0 + waves * pitch) : nullptr;
    const uint64_t beg = offs[read];
    uint64_t end = offs[read + 1];
    if (end < beg) end = beg;
    const uint64_t nwin = n_windows(beg, end);
    constexpr uint32_t kGrain = 64 / G;  // terms that the wave's lanes take together
    const uint64_t part = ((nwin + kGrain - 1) / kGrain + waves - 1) / waves * kGrain;  // windows per wave
    const bool ee = opt.early_exit != 0;
    const bool scouts = ee && nwin > 0 && (part > 128 || offs[n] - offs[0] >= kTeamScout);
    // waves that probe anything
    const uint32_t used = scouts ? waves : part ? (uint32_t)((nwin + part - 1) / part) : 0;
    if (threadIdx.x == 0) issued = kept = 0;
    init_masks(ix, M, lane);
    __syncthreads();
    const uint64_t w_lo = min(nwin, wave * part), w_hi = min(nwin, w_lo + part);
    bool live = true;
    uint64_t got = 0;
    uint64_t *o = out + read * ix.W;
    // the AND of the waves' repetition-0 masks is not empty (the same in every wave)
    auto rep0_live = [&]() -> bool {
        uint32_t any = 0;
        for (uint32_t w = lane; w < ix.RW; w += 64) {
            uint32_t v = 0xFFFFFFFFu;
            for (uint32_t k = 0; k < used; k++) v &= M0[k * pitch + w];
            any |= v;
        }
        return __ballot(any != 0) != 0;
    };
    // the answer of a read that repetition 0 has ended
    auto ended = [&]() {
        if (opt.probes && lane == 0 && got) atomicAdd(opt.probes, (unsigned long long)(got * ix.eta));
        if (!opt.counts)
            for (uint32_t w = threadIdx.x; w < ix.W; w += blockDim.x) o[w] = 0;
        else if (threadIdx.x == 0) opt.counts[read] = 0;
    };
    if (scouts) {
        const uint64_t ns = scout_count(0, nwin);
        for (uint64_t s0 = 0, s1; s0 < ns; s0 = s1) {
            s1 = s0 ? ns : min<uint64_t>(ns, 64);
            const uint64_t per = ((s1 - s0 + kGrain - 1) / kGrain + waves - 1) / waves * kGrain;
            const uint64_t hi = min(s1, s0 + (wave + 1) * per);
            for (uint64_t i0 = s0 + wave * per; i0 < hi; i0 += 64) {
                Window wv{0, false};
                if (i0 + lane < hi) {
                    WinBytes wb;
                    load_window_bytes(wb, seqs + beg + scout_pos(0, nwin, i0 + lane));
                    wv = decode_window(wb);
                }
                (void)probe_group<SEG, G, 0, 1>(ix, step_params(ix), wv, wv.valid, lane, M);
                got += (uint64_t)__popcll(__ballot(wv.valid));
            }
            __syncthreads();
            live = rep0_live();
            if (!live) {
                ended();
                return;
            }
            __syncthreads();  // (the masks change again)
        }
    }
    if (w_lo < w_hi)
        got += sweep_rep0<SEG, G>(ix, seqs, beg, end, w_lo, w_hi, lane, M, ee, scouts, 0, nwin, live);
    __syncthreads();
    if (ee && used) {
        // the read ends here if the parts' AND is empty
        live = rep0_live();
        if (!live) {
            ended();
            return;
        }
    }
    if (w_lo < w_hi && ix.R > 1) got += sweep_rest<SEG, G>(ix, seqs, beg, end, w_lo, w_hi, lane, M, ee);
    if (lane == 0 && got) atomicAdd(&issued, (unsigned long long)got);
    __syncthreads();
    for (uint32_t w = threadIdx.x; w < mw; w += blockDim.x) {
        uint32_t v = M0[w];
        for (uint32_t k = 1; k < used; k++) v &= M0[k * pitch + w];
        M0[w] = v;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        if (opt.probes && issued) atomicAdd(opt.probes, issued * ix.eta);
        if (issued == 0) atomicAdd(opt.emptyq, 1ULL);
    }
    if (masks_some_rep_empty(ix, M0, lane)) {
        if (!opt.counts)
            for (uint32_t w = threadIdx.x; w < ix.W; w += blockDim.x) o[w] = 0;
        else if (threadIdx.x == 0) opt.counts[read] = 0;
        return;
    }
    uint64_t *wm = (opt.counts && opt.wm) ? opt.wm + read * ((ix.W + 63) / 64) : nullptr;
    const uint64_t pc = resolve(ix, M0, res, o, lane, opt.rmode, wm, WholeGroup{wave, waves});
    if (opt.counts) {
        if (lane == 0 && pc) atomicAdd(&kept, (unsigned long long)pc);
        __syncthreads();
        if (threadIdx.x == 0) opt.counts[read] = kept;
    }
}

// LDS of a team of waves: their masks and one candidate bitset.
size_t team_lds(const rambo_s *h, uint32_t waves, bool use_res) {
    return (size_t)waves * wave_lds(h->R * h->RW, h->W, false, false).total * 4 + (use_res ? (size_t)h->W * 8 : 0);
}

// Waves per read of a batch of n reads (1: the one-wave kernel): 16 while every
// compute unit holds one such workgroup (and a little past that, where a second one
// waits), then two workgroups of 8, then four a read until one wave per read fills
// the chip. The lines lie where it makes little difference (whole calls, us, with 16
// / 8 / 4 waves): K=10,000 (a lane a term) 256 reads 57 / 59 / 57, 288 58 / 59 / 57,
// 320 58 / 59 / 57, 512 66 / 65 / 62, 768 86 / 79 / 77; K=101,000 (8 lanes a term)
// 256 reads 45 / 42 / 54, 288 46 / 44 / 55, 512 50 / 47 / 58, 768 57 / 50 / 61. With
// one wave 16 reads took 57-86 and 24-100, 257 81-110 and 120-140, 2,000 167-227 and
// 133-176, 8,000 261-272 and 217-241; with 4 2,000 114-135 and 77-85, 8,000 293-315
// and 197-218.
uint32_t team_waves(const rambo_s *h, uint64_t n) {
    const uint64_t cu = (uint64_t)h->n_cu;
    uint32_t t = n <= cu + cu / 8 ? 16 : n <= 2 * cu ? 8 : n <= 16 * cu ? 4 : 1;  // (past that only under capture and the like)
    while (t > 1 && team_lds(h, t, seq_lds_result(h->W)) + 64 > h->lds_max) t /= 2;
    return t;
}

int launch_query_seqs_plain(rambo_s *h, const uint8_t *seqs, const uint64_t *offs, uint64_t n, uint64_t *out,
                            hipStream_t s, int seg, const InputHdr *hdr, const IdsOut &io) {
    // with hdr, the batch is read on the device and n is only its capacity
    const Index ix = make_index(h);
    const int G = (int)h->RW / seg;
    const int WPB = 4;
    const int sched = h->tune.sched;  // (this form scouts inside its kernel)
    const bool stage = sched == SCHED_SCOUT;
    const int use_res = seq_lds_result(h->W) ? 1 : 0;
    const size_t lds = (size_t)WPB * wave_lds(h->R * h->RW, h->W, use_res != 0, stage).total * 4;
    const uint64_t blocks = (n + WPB - 1) / WPB;
    if (blocks > 0x7FFFFFFFULL) return fail(RAMBO_EINVAL, "rambo_query_seqs: batch too large");
    QueryOpts opt{h->resolve, h->early_exit, h->probe_counter, sched, io.counts,
                  io.counts ? io.noterm : h->d_emptyq, h->sparse_counter, io.counts ? io.wm : nullptr};
    const uint32_t team = opt.rplus ? 1 : team_waves(h, n);
    if (team > 1) {
        const size_t tlds = team_lds(h, team, use_res != 0);
#define RAMBO_SPLIT_BODY_                                                                                  \
    hipLaunchKernelGGL((k_query_seqs_team<SEG, G>), dim3((unsigned)n), dim3(64 * team), tlds, s, ix, seqs, offs, n, \
                       hdr, out, opt, use_res)
        RAMBO_DISPATCH_DEFAULT_SPLIT(seg, G)
#undef RAMBO_SPLIT_BODY_
        HIP_CHECK(hipGetLastError());
        return RAMBO_OK;
    }
    // the RAMBO+ tallies have a kernel of their own (measurement only)
#define RAMBO_SPLIT_BODY_                                                                                  \
    if (opt.rplus)                                                                                         \
        hipLaunchKernelGGL((k_query_seqs_plain<SEG, G, true>), dim3((unsigned)blocks), dim3(64 * WPB), lds, s, ix,  \
                           seqs, offs, n, hdr, out, opt, use_res);                                          \
    else                                                                                                   \
        hipLaunchKernelGGL((k_query_seqs_plain<SEG, G, false>), dim3((unsigned)blocks), dim3(64 * WPB), lds, s, ix, \
                           seqs, offs, n, hdr, out, opt, use_res)
    RAMBO_DISPATCH_DEFAULT_SPLIT(seg, G)
#undef RAMBO_SPLIT_BODY_
    HIP_CHECK(hipGetLastError());
    return RAMBO_OK;
}

// -------------------------------------------------------------------------
// bitsets -> ascending id lists
// -------------------------------------------------------------------------
// One read's ids, ascending, from ids[base] on, by one wave. With marks (the
// query's marks of its non-zero bitset words, (W + 63) / 64 words) only the
// marked words are read: per mark word, the lanes take its 64 bitset words, load
// the marked ones, and number their ids by a prefix sum. Without, the whole row
// is read, 64 words a load, eight loads in flight.
__device__ __forceinline__ void place_ids(uint64_t v, uint32_t w, uint32_t lane, uint64_t &base,
                                          uint32_t *__restrict__ ids) {
    const uint32_t pc = (uint32_t)__popcll(v);
    uint32_t incl = pc;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const uint32_t t = __shfl_up(incl, d);
        if ((int)lane >= d) incl += t;
    }
    uint64_t pos = base + incl - pc;
    while (v) {
        ids[pos++] = w * 64 + (uint32_t)__builtin_ctzll(v);
        v &= v - 1;
    }
    base += __shfl(incl, 63);
}
__device__ __forceinline__ void compact_read(const uint64_t *__restrict__ row, const uint64_t *__restrict__ marks,
                                             uint32_t W, uint64_t base, uint32_t lane, uint32_t *__restrict__ ids) {
    if (marks) {
        const uint32_t WM = (W + 63) / 64;
        for (uint32_t m0 = 0; m0 < WM; m0 += 64) {
            const uint64_t mw = m0 + lane < WM ? marks[m0 + lane] : 0;
            uint64_t src = __ballot(mw != 0);
            while (src) {
                const uint32_t j = (uint32_t)__builtin_ctzll(src);
                src &= src - 1;
                // (readlane returns a signed int: widen through uint32_t)
                const uint64_t m = ((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(mw >> 32), (int)j) << 32) |
                                   (uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)mw, (int)j);
                const uint32_t w = (m0 + j) * 64 + lane;
                place_ids((((m >> lane) & 1) && w < W) ? row[w] : 0, w, lane, base, ids);
            }
        }
        return;
    }
    constexpr uint32_t U = 8;
    for (uint32_t c0 = 0; c0 < W; c0 += 64 * U) {
        uint64_t word[U];
#pragma unroll
        for (uint32_t u = 0; u < U; u++) {
            const uint32_t w = c0 + 64 * u + lane;
            word[u] = w < W ? row[w] : 0;
        }
#pragma unroll
        for (uint32_t u = 0; u < U; u++) place_ids(word[u], c0 + 64 * u + lane, lane, base, ids);
    }
}

// What the host waits for: the total and the reads without a term (cleared for
// the next call).
__device__ __forceinline__ void tell_host(uint64_t *host, uint64_t total, unsigned long long *noterm) {
    if (!host) return;
    host[0] = total;
    host[1] = *noterm;
    *noterm = 0;
}

// A wave takes `per` reads (1 to 64): those with ids (a few per cent in id-list
// workloads) are found with one ballot and compacted one after the other;
// empty answers cost nothing more. The total (off[n]) is checked here: over cap,
// nothing is written and the host reports the shortfall after the pass.
__global__ __launch_bounds__(256) void k_compact(const uint64_t *__restrict__ bits, const uint64_t *__restrict__ wm,
                                                 uint64_t n, uint32_t W, const uint64_t *__restrict__ off,
                                                 uint32_t *__restrict__ ids, uint64_t cap, uint32_t per,
                                                 unsigned long long *noterm, uint64_t *host) {
    const uint32_t lane = threadIdx.x & 63, WM = (W + 63) / 64;
    const uint64_t total = off[n];
    if (blockIdx.x == 0 && threadIdx.x == 0) tell_host(host, total, noterm);
    const uint64_t i0 = (((uint64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6) * per;
    if (i0 >= n || total > cap) return;
    const uint64_t mine = i0 + lane;
    uint64_t todo = __ballot(lane < per && mine < n && off[mine + 1] != off[mine]);
    while (todo) {
        const uint64_t i = i0 + (uint64_t)__builtin_ctzll(todo);
        todo &= todo - 1;
        compact_read(bits + i * W, wm ? wm + i * WM : nullptr, W, off[i], lane, ids);
    }
}

// Scan and compaction of a small batch in one launch, a wave per read: each
// adds up the sizes before its own (n / 64 loads a lane).
__global__ __launch_bounds__(256) void k_compact_small(const uint64_t *__restrict__ bits,
                                                       const uint64_t *__restrict__ wm, uint32_t n, uint32_t W,
                                                       const unsigned long long *__restrict__ counts,
                                                       uint64_t *__restrict__ off, uint32_t *__restrict__ ids,
                                                       uint64_t cap, unsigned long long *noterm, uint64_t *host) {
    const uint32_t lane = threadIdx.x & 63, i = (blockIdx.x * blockDim.x + threadIdx.x) >> 6;
    if (i >= n) return;
    uint64_t before = 0, total = 0;
#pragma unroll 4
    for (uint32_t j = lane; j < n; j += 64) {
        const uint64_t c = counts[j];
        total += c;
        before += j < i ? c : 0;
    }
#pragma unroll
    for (int d = 32; d > 0; d >>= 1) {
        total += __shfl_xor(total, d);
        before += __shfl_xor(before, d);
    }
    if (lane == 0) off[i] = before;
    if (i == n - 1 && lane == 0) {
        off[n] = total;
        tell_host(host, total, noterm);
    }
    if (counts[i] == 0 || total > cap) return;
    compact_read(bits + (uint64_t)i * W, wm ? wm + (uint64_t)i * ((W + 63) / 64) : nullptr, W, before, lane, ids);
}

__global__ void k_store_u64(uint64_t *p, uint64_t v) {
    if (threadIdx.x == 0) *p = v;
}

uint64_t ids_aux_words(uint64_t n) { return scan_parts_needed(n) + 1; }

// one-launch id lists up to this many reads: 2,000 sizes are 32 loads a lane
static constexpr uint64_t kSmallIds = 2048;

// total of this thread's last id-list call
static thread_local uint64_t g_ids_total = 0;
void clear_ids_total() { g_ids_total = 0; }

int launch_ids(rambo_s *h, const uint64_t *bits, uint64_t n, uint32_t *ids, uint64_t *id_off, uint64_t ids_cap,
               hipStream_t s, const IdsOut &io, uint64_t *aux, uint64_t *host) {
    const uint32_t W = (uint32_t)h->W;
    uint64_t total = 0;
    if (n == 0) {
        HIP_CHECK(hipMemsetAsync(id_off, 0, 8, s));
        HIP_CHECK(hipStreamSynchronize(s));
        return RAMBO_OK;
    }
    // the compaction checks the total against the capacity itself: no round
    // trip to the host before it
    const uint64_t cap = ids ? ids_cap : 0;
    if (n <= kSmallIds) {
        hipLaunchKernelGGL(k_compact_small, dim3((unsigned)((n + 3) / 4)), dim3(256), 0, s, bits, io.wm, (uint32_t)n, W,
                           io.counts, id_off, ids, cap, io.noterm, host);
    } else {
        uint64_t *parts = aux, *d_n = aux + scan_parts_needed(n);
        hipLaunchKernelGGL(k_store_u64, dim3(1), dim3(64), 0, s, d_n, n);
        HIP_CHECK(hipGetLastError());
        const int sst = launch_exclusive_scan(reinterpret_cast<const uint64_t *>(io.counts), d_n, n, id_off, parts, s);
        if (sst != RAMBO_OK) return sst;
        // reads per wave: as many as leave every place for a wave one
        uint32_t per = 64;
        while (per > 1 && n < (uint64_t)per * h->n_cu * 16) per /= 2;
        const uint64_t waves = (n + per - 1) / per;
        hipLaunchKernelGGL(k_compact, dim3((unsigned)((waves + 3) / 4)), dim3(256), 0, s, bits, io.wm, n, W, id_off, ids,
                           cap, per, io.noterm, host);
    }
    HIP_CHECK(hipGetLastError());
    unsigned long long noterm = 0;
    hipError_t e = hipSuccess;
    if (!host) {
        e = hipMemcpyAsync(&total, id_off + n, 8, hipMemcpyDeviceToHost, s);
        if (e == hipSuccess) e = hipMemcpyAsync(&noterm, io.noterm, 8, hipMemcpyDeviceToHost, s);
    }
    if (e == hipSuccess) e = hipStreamSynchronize(s);
    if (e != hipSuccess) return fail(RAMBO_EDEVICE, "rambo_query_seqs_ids: %s", hipGetErrorString(e));
    if (host) {
        total = host[0];
        noterm = host[1];
    }
    g_ids_total = total;
    if (total > ids_cap)
        return fail(RAMBO_ETRUNC, "rambo_query_seqs_ids: %llu ids do not fit %llu", (unsigned long long)total,
                    (unsigned long long)ids_cap);
    if (total > 0 && !ids) return fail(RAMBO_EINVAL, "rambo_query_seqs_ids: null ids");
    return noterm ? RAMBO_OK_EMPTYQ : RAMBO_OK;
}

int launch_store_u64(uint64_t *p, uint64_t v, hipStream_t s) {
    hipLaunchKernelGGL(k_store_u64, dim3(1), dim3(64), 0, s, p, v);
    HIP_CHECK(hipGetLastError());
    return RAMBO_OK;
}

}  // namespace rambo

using namespace rambo;

RAMBO_API uint64_t rambo_last_ids_total(void) { return g_ids_total; }
