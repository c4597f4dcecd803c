// Construction (Algorithm 1): every term of document d sets, in every
// repetition r and for every Bloom hash j, bit phi_r(d) of row
// (r, h_{r,j}(term)) -- one atomic OR of one bit per (term, r, j). Bits are
// only ever set, so the result is independent of order and of repeats
// (streaming insertion, Section 3.2, is the same kernel on new documents).
#include <algorithm>
#include <cmath>

#include "rambo_int.h"

namespace rambo {

// Set one bit of the rows. Many terms are inserted more than once (documents
// share k-mers; a common word is in every document and many times in each), and
// atomics on one line are performed one after the other, so a bit that a plain
// load shows set already is left alone (bits are only ever set: a stale load
// can only cost an atomic that was not needed). The load also brings the line
// in, so that it costs nothing where the bit was not set: 10^8 random bits over
// 1 GiB, 5.05 ms by atomics alone, 4.16 ms with the load before them, 1.9 ms
// once they are set; over 4 KB 19.5 and 0.1 ms.
// The loads of a group of bits are issued together.
__device__ __forceinline__ uint32_t peek(const uint32_t *p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Term x of the document with cell record cd in repetitions FIRST .. FIRST + COUNT - 1
// (those below R), ETA hashes each.
template <int FIRST, int COUNT, int ETA>
__device__ __forceinline__ void scatter_reps(const Index &ix, uint64_t x, const uint4 &cd) {
    uint32_t *at[COUNT][ETA];
    uint32_t old[COUNT][ETA];
#pragma unroll
    for (int i = 0; i < COUNT; i++) {
        if (FIRST + i >= (int)ix.R) continue;
#pragma unroll
        for (int j = 0; j < ETA; j++) {
            const uint64_t pos = bloom_pos(ix, (uint32_t)(FIRST + i) * ETA + j, x);
            at[i][j] = ix.rows + (((uint64_t)(FIRST + i) * ix.m + pos) << ix.log2RW) + (cell_at(cd, FIRST + i) >> 5);
            old[i][j] = peek(at[i][j]);
        }
    }
#pragma unroll
    for (int i = 0; i < COUNT; i++) {
        if (FIRST + i >= (int)ix.R) continue;
        const uint32_t bit = 1u << (cell_at(cd, FIRST + i) & 31);
#pragma unroll
        for (int j = 0; j < ETA; j++)
            if (~old[i][j] & bit) atomicOr(at[i][j], bit);
    }
}

__device__ __forceinline__ void scatter_term(const Index &ix, uint64_t x, uint64_t d) {
    const uint4 cd = ix.cells[d];
    if (ix.eta == 2) {
        scatter_reps<0, 4, 2>(ix, x, cd);
        if (ix.R > 4) scatter_reps<4, 4, 2>(ix, x, cd);
    } else if (ix.eta == 3) {
        scatter_reps<0, 4, 3>(ix, x, cd);
        if (ix.R > 4) scatter_reps<4, 4, 3>(ix, x, cd);
    } else {
        for (uint32_t r = 0; r < ix.R; r++) {
            const uint32_t b = reinterpret_cast<const uint16_t *>(ix.cells + d)[r], bit = 1u << (b & 31);
            for (uint32_t j = 0; j < ix.eta; j++) {
                const uint64_t pos = bloom_pos(ix, r * ix.eta + j, x);
                uint32_t *p = ix.rows + (((uint64_t)r * ix.m + pos) << ix.log2RW) + (b >> 5);
                if (~peek(p) & bit) atomicOr(p, bit);
            }
        }
    }
}

// largest k in [lo, n) with off[k] <= p (off non-decreasing, off[lo] <= p)
__device__ __forceinline__ uint64_t find_doc(const uint64_t *off, uint64_t lo, uint64_t n, uint64_t p) {
    uint64_t hi = n;
    while (hi - lo > 1) {
        const uint64_t mid = (lo + hi) >> 1;
        if (off[mid] <= p) lo = mid;
        else hi = mid;
    }
    return lo;
}

// The documents of an insertion: off[k] .. off[k + 1] are document ids[k]'s
// k-mer codes (kmers) or bytes (seqs), n of them.
struct Docs {
    const uint64_t *kmers;
    const uint8_t *seqs;
    const uint64_t *off, *ids;
    uint64_t n;
};

// The term at each of the 64 positions p0 .. p0 + 63 (one a lane, those below
// last; the documents end at all) and its document; ok where there is one. k is the document of an earlier
// position of the wave, the place the search for p0's starts from. Values that
// are no k-mers and ids >= K are counted in *invalid if count. All 64 lanes.
struct Term {
    uint64_t x, d;
    bool ok;
};
template <bool SEQS>
__device__ __forceinline__ Term load_term(const Index &ix, const Docs &in, uint64_t p0, uint64_t last, uint64_t all,
                                          uint64_t &k, uint32_t lane, unsigned long long *invalid, bool count) {
    Term t{0, 0, false};
    p0 = uniform64(p0);
    if (p0 >= last) return t;
    if (in.off[k + 1] <= p0)  // the next document, usually
        k = k + 2 <= in.n && in.off[k + 2] > p0 ? k + 1 : uniform64(find_doc(in.off, k + 1, in.n, p0));
    const uint64_t p = p0 + lane, dend = in.off[k + 1];
    if constexpr (SEQS) {
        const uint32_t c0 = p < all ? in.seqs[p] : 0u;
        const uint32_t c1 = (lane < 30 && p + 64 < all) ? in.seqs[p + 64] : 0u;
        const Window w = extract_windows(c0, c1, lane);
        t.x = w.canon;
        t.ok = w.valid && p < last;
        if (p0 + 94 <= dend) {  // the whole step in one document
            t.d = in.ids[k];
        } else if (t.ok) {
            const uint64_t mine = dend <= p ? find_doc(in.off, k + 1, in.n, p) : k;
            t.ok = p + 31 <= in.off[mine + 1];
            t.d = in.ids[mine];
        }
        if (t.ok && t.d >= ix.K) {
            if (count) atomicAdd(invalid, 1ULL);
            t.ok = false;
        }
    } else if (p < last) {
        t.d = in.ids[dend <= p ? find_doc(in.off, k + 1, in.n, p) : k];
        t.x = in.kmers[p];
        t.ok = t.d < ix.K && (ix.opaque || !(t.x >> 62));
        if (!t.ok && count) atomicAdd(invalid, 1ULL);
        if (!ix.opaque) t.x = canonical(t.x);
    }
    return t;
}

// Direct insertion: one bit at a time into the rows. A wave takes a contiguous
// share of the concatenated documents' positions (from the from-th on), 64 per
// step, so that it searches for its document once (11.5 million terms again
// into an index that holds them: 0.36 ms with the waves' steps interleaved and
// a search each, 0.28 now). Bound by the rate of random atomics, 2.0 x 10^10 a
// second over 1 GiB of rows, where bits are new.
template <bool SEQS>
__device__ __forceinline__ void build_share(const Index &ix, const Docs &in, uint64_t first, uint64_t last,
                                            unsigned long long *invalid) {
    if (first >= last) return;
    const uint32_t lane = threadIdx.x & 63;
    const uint64_t waves = ((uint64_t)gridDim.x * blockDim.x) >> 6;
    const uint64_t wave = ((uint64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6;
    const uint64_t share = ((last - first + waves - 1) / waves + 63) & ~63ull;
    const uint64_t lo = first + wave * share;
    if (lo >= last) return;
    const uint64_t hi = min(last, lo + share);
    uint64_t k = 0;
    for (uint64_t p0 = lo; p0 < hi; p0 += 64) {
        const Term t = load_term<SEQS>(ix, in, p0, hi, last, k, lane, invalid, true);
        if (t.ok) scatter_term(ix, t.x, t.d);
    }
}
// All positions of an insertion of fewer than least; those from the from-th on of
// a larger one.
template <bool SEQS>
__global__ __launch_bounds__(256) void k_build(Index ix, Docs in, uint64_t from, uint64_t least,
                                               unsigned long long *invalid) {
    const uint64_t first = in.off[0], last = in.off[in.n];
    if (last <= first) return;
    build_share<SEQS>(ix, in, last - first < least ? first : first + from, last, invalid);
}

// ---------------------------------------------------------------------------
// Partitioned insertion, for batches that set several bits of every line of a
// repetition's rows. Random atomics are performed one 128-byte line at a time
// (37 ps each at best, 50 ps over 1 GiB); here the bits of one repetition
// are first sorted by region of the rows (k_part_scatter), then each region is
// put together in LDS and ORed into the rows in order (k_part_apply), which
// costs 0.8 ms a GiB. 1,000 documents of 200 kbp, R=4, eta=3 into 1 GiB of rows
// (2.4 x 10^9 bits): 116 ms by atomics alone, 79 ms by direct insertion
// as above, 14.0 ms partitioned.
// ---------------------------------------------------------------------------
constexpr uint32_t kBuckets = 1024;    // regions of the scatter, at most
constexpr uint32_t kStage = 32768;     // bits staged by a scatter workgroup (128 KB of LDS), over all buckets
constexpr uint32_t kFlush = 16;        // bits written together (64 bytes)
constexpr uint32_t kGroupAdds = 9;     // bits a thread adds between flushes: nine a bucket of 32 places, with 1,024
                                       // (14.2 ms for the genomes above; 14.7 with 6, 14.4 with 12, which overflow more)
constexpr uint32_t kUnroll = 4;        // positions of a thread whose loads go together
constexpr uint32_t kTileBits = 20;     // an apply tile, at most: 128 KB of rows
constexpr uint32_t kBucketBits = 19;   // a bucket, at least
constexpr uint32_t kApplyGroups = 4096;  // of an apply launch that has one a tile, at most

// Where a partitioned insertion keeps its bits: segment (b, g) holds those of
// bucket b that workgroup g found, at most cap of them (a multiple of 16), as
// bit offsets in the bucket.
struct Parts {
    uint32_t *bits;    // [buckets][groups][cap]
    uint32_t *count;   // [buckets][groups]
    uint32_t cap, groups;
    uint32_t buckets, lg;  // bucket b: rows b << lg .. ((b + 1) << lg) - 1 of the repetition
    uint32_t slots;    // staged bits of a bucket: kStage / buckets, a power of two
    uint64_t chunk;    // positions of the concatenated documents a pass takes
    uint64_t least;    // positions below which the whole insertion is direct
    uint64_t rep;      // words from a repetition's segments to the next one's (0: one set of segments)
};

// Repetition blockIdx.y of a launch that takes several has segments of its own.
__device__ __forceinline__ uint32_t part_rep(Parts &pt, uint32_t r) {
    pt.bits += blockIdx.y * pt.rep;
    pt.count += blockIdx.y * pt.rep;
    return r + blockIdx.y;
}

__device__ __forceinline__ uint32_t *part_base(const Index &ix, const Parts &pt, uint32_t r, uint32_t b) {
    return ix.rows + (((uint64_t)r * ix.m + ((uint64_t)b << pt.lg)) << ix.log2RW);
}

// A bit that has no place in its segment is set directly.
__device__ __forceinline__ void part_direct(uint32_t *base, uint32_t v) {
    uint32_t *p = base + (v >> 5);
    const uint32_t bit = 1u << (v & 31);
    if (~peek(p) & bit) atomicOr(p, bit);
}

// Bits of repetition r of positions [first + pass * chunk, + chunk) into the
// segments. A workgroup a compute unit; it takes a contiguous share of the
// positions and stages bits in LDS, so that they leave 16 of a bucket at a time.
// A bit that finds its bucket's places taken is set directly. An insertion of
// fewer than least positions is left to k_build (the host does not know the number
// of positions).
// Bound by vector instructions (the hashes' 64-bit products; 300 a 64 positions
// and eta = 3): 6.7 x 10^7 positions of one repetition in 0.91 ms.
template <bool SEQS>
__global__ __launch_bounds__(1024) void k_part_scatter(Index ix, Docs in, Parts pt, uint32_t r, uint32_t pass,
                                                       unsigned long long *invalid) {
    extern __shared__ __align__(16) uint32_t smem32[];
    r = part_rep(pt, r);
    uint32_t *stage = smem32;            // [buckets][slots]
    uint32_t *fill = stage + kStage;     // [kBuckets] staged
    uint32_t *sent = fill + kBuckets;    // [kBuckets] written to the segment
    const uint32_t lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const uint64_t first = in.off[0], all = in.off[in.n];
    if (all <= first || all - first < pt.least) return;
    const uint64_t lo = first + (uint64_t)pass * pt.chunk;
    if (lo >= all) return;
    const uint64_t hi = min(all, lo + pt.chunk);
    for (uint32_t b = threadIdx.x; b < kBuckets; b += blockDim.x) fill[b] = sent[b] = 0;
    __syncthreads();
    // this workgroup's share, in steps of 1,024 * kUnroll positions
    const uint64_t share = ((hi - lo + gridDim.x - 1) / gridDim.x + 63) & ~63ull;
    const uint64_t p0 = min(hi, lo + blockIdx.x * share), p1 = min(hi, p0 + share);
    auto flush = [&](bool end) {
        __syncthreads();
        // four lanes a bucket
        for (uint32_t b0 = wave * 16; b0 < pt.buckets; b0 += (blockDim.x >> 6) * 16) {
            const uint32_t b = b0 + (lane >> 2), q = lane & 3;
            if (b >= pt.buckets) continue;
            const uint32_t n = min(fill[b], pt.slots);
            if (n < kFlush && !end) continue;
            const uint32_t done = sent[b];
            uint32_t *st = stage + b * pt.slots;
            uint32_t *seg = pt.bits + ((uint64_t)b * pt.groups + blockIdx.x) * pt.cap;
            uint32_t at = 0;
            for (; at + kFlush <= n; at += kFlush) {
                const uint4 v = *reinterpret_cast<const uint4 *>(st + at + q * 4);
                if (done + at + kFlush <= pt.cap) {
                    *reinterpret_cast<uint4 *>(seg + done + at + q * 4) = v;
                } else {
                    uint32_t *base = part_base(ix, pt, r, b);
                    part_direct(base, v.x); part_direct(base, v.y); part_direct(base, v.z); part_direct(base, v.w);
                }
            }
            uint32_t out = min(done + at, pt.cap);
            if (end) {
                for (uint32_t i = at + q; i < n; i += 4) {
                    if (out + i - at < pt.cap) seg[out + i - at] = st[i];
                    else part_direct(part_base(ix, pt, r, b), st[i]);
                }
                out = min(out + n - at, pt.cap);
                if (q == 0) pt.count[(uint64_t)b * pt.groups + blockIdx.x] = out;
            } else {
                // what is left (fewer than 16) moves to the front
                if (at < n) {
                    const uint4 v = *reinterpret_cast<const uint4 *>(st + at + q * 4);
                    *reinterpret_cast<uint4 *>(st + q * 4) = v;
                }
                if (q == 0) fill[b] = n - at, sent[b] = out;
            }
        }
        __syncthreads();
    };
    uint64_t k = 0;
    uint32_t adds = 0;
    for (uint64_t p = p0; p < p1; p += 1024 * kUnroll) {
        Term t[kUnroll];
        uint32_t c[kUnroll];
#pragma unroll
        for (uint32_t u = 0; u < kUnroll; u++)
            t[u] = load_term<SEQS>(ix, in, p + (wave * kUnroll + u) * 64, p1, all, k, lane, invalid, r == 0);
#pragma unroll
        for (uint32_t u = 0; u < kUnroll; u++)
            c[u] = t[u].ok ? reinterpret_cast<const uint16_t *>(ix.cells + t[u].d)[r] : 0;
#pragma unroll
        for (uint32_t u = 0; u < kUnroll; u++) {
            for (uint32_t j = 0; j < ix.eta; j++) {
                if (adds == kGroupAdds) {
                    flush(false);
                    adds = 0;
                }
                adds++;
                if (!t[u].ok) continue;
                const uint64_t pos = bloom_pos(hash_rec(ix.hp->h, r * ix.eta + j), ix.m, t[u].x);
                const uint32_t b = (uint32_t)(pos >> pt.lg);
                const uint32_t v = (((uint32_t)pos & ((1u << pt.lg) - 1)) << (ix.log2RW + 5)) | c[u];
                const uint32_t i = atomicAdd(&fill[b], 1u);
                if (i < pt.slots) stage[b * pt.slots + i] = v;
                else part_direct(part_base(ix, pt, r, b), v);
            }
        }
    }
    flush(true);
}

// ORs the segments' bits into the rows, tile by tile (128 KB of rows, or a smaller
// bucket): a workgroup collects a tile's in LDS, reading all of its bucket's
// segments, four lanes a segment. A bucket's tiles are eight workgroups apart, so
// they run on one XCD, whose L2 then reads the segments once. The rows are
// changed by atomics (in order, at more than half the rate of plain loads and
// stores), so insertions on other streams may run at the same time.
// Bound by the reads of the bits, each by every tile of its bucket, where there
// are many tiles, and by the atomics where there are few: tiles of 128 KB, one
// workgroup a compute unit, against 64 KB, two: 5 x 10^10 bits at 64 / 128 tiles a
// bucket, scatter included, 1.10 / 1.53 s; 2.4 x 10^9 at 2 / 4, 14.0 / 14.2 ms.
// A workgroup a tile up to kApplyGroups; past that the grid is what is resident and
// strides over the tiles (a launch that finds nothing to do takes 130 us with
// 131,072 workgroups; striding costs 2 % of a launch of a few tiles a workgroup).
// A larger grid that strides would have the resident workgroups leave a bucket
// before its last tiles (K=101,000, 96 GiB, 128 tiles a bucket: 4.8 s to build, 4.1).
__global__ __launch_bounds__(1024) void k_part_apply(Index ix, Docs in, Parts pt, uint32_t r, uint32_t pass,
                                                    uint32_t tiles, uint32_t lgt) {
    extern __shared__ __align__(16) uint32_t smem32[];
    r = part_rep(pt, r);
    const uint64_t first = in.off[0], all = in.off[in.n];
    if (all <= first || first + (uint64_t)pass * pt.chunk >= all || all - first < pt.least) return;
    const uint32_t words = 1u << (lgt - 5), part = threadIdx.x & 3;
    const uint32_t end = ((pt.buckets + 7) / 8) * 8 * tiles;
    for (uint32_t w = blockIdx.x; w < end; w += gridDim.x) {
        const uint32_t b = (w / (8 * tiles)) * 8 + w % 8, tile = (w / 8) % tiles;
        if (b >= pt.buckets) continue;
        // (a thread clears the words that it wrote out itself: no barrier before)
        for (uint32_t i = threadIdx.x; i < words; i += blockDim.x) smem32[i] = 0;
        __syncthreads();
        auto put = [&](uint32_t v) {
            if (v >> lgt == tile) atomicOr(&smem32[(v & ((1u << lgt) - 1)) >> 5], 1u << (v & 31));
        };
        constexpr uint32_t U = 8;  // loads of a lane in flight
        const uint32_t *counts = pt.count + (uint64_t)b * pt.groups;
        const uint32_t g0 = threadIdx.x >> 2, gs = blockDim.x >> 2;
        uint32_t next = g0 < pt.groups ? counts[g0] : 0;
        for (uint32_t g = g0; g < pt.groups; g += gs) {
            const uint32_t n = next;
            next = g + gs < pt.groups ? counts[g + gs] : 0;
            const uint32_t *seg = pt.bits + ((uint64_t)b * pt.groups + g) * pt.cap;
            const uint4 *seg4 = reinterpret_cast<const uint4 *>(seg);
            const uint32_t n4 = n / 4;
            for (uint32_t i0 = part; i0 < n4; i0 += 4 * U) {
                uint4 v[U];
#pragma unroll
                for (uint32_t u = 0; u < U; u++) v[u] = seg4[min(i0 + 4 * u, n4 - 1)];
#pragma unroll
                for (uint32_t u = 0; u < U; u++) {
                    if (i0 + 4 * u >= n4) break;
                    put(v[u].x); put(v[u].y); put(v[u].z); put(v[u].w);
                }
            }
            if (part < n % 4) put(seg[n4 * 4 + part]);
        }
        __syncthreads();
        uint32_t *rows = part_base(ix, pt, r, b) + (uint64_t)tile * words;
        for (uint32_t i = threadIdx.x; i < words; i += blockDim.x) {
            const uint32_t v = smem32[i];
            if (v) atomicOr(rows + i, v);
        }
    }
}

// BFU(r, b) as a plain m-bit filter: lane l of a wave reads row base + l.
__global__ __launch_bounds__(256) void k_dump_bfu(Index ix, uint32_t r, uint32_t b, uint64_t *out) {
    const uint32_t lane = threadIdx.x & 63;
    const uint64_t words = (ix.m + 63) / 64;
    const uint64_t nwaves = ((uint64_t)gridDim.x * blockDim.x) >> 6;
    for (uint64_t w = ((uint64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6; w < words; w += nwaves) {
        const uint64_t p = w * 64 + lane;
        uint32_t bit = 0;
        if (p < ix.m) bit = (ix.rows[(((uint64_t)r * ix.m + p) << ix.log2RW) + (b >> 5)] >> (b & 31)) & 1u;
        const uint64_t word = __ballot(bit);
        if (lane == 0) out[w] = word;
    }
}

static unsigned grid_for(const rambo_s *h, uint64_t work_waves, unsigned per_cu) {
    uint64_t cap = (uint64_t)h->n_cu * per_cu;
    uint64_t blocks = (work_waves + 3) / 4;
    if (blocks > cap) blocks = cap;
    return (unsigned)(blocks ? blocks : 1);
}

// How far the allocation that holds p reaches past it, in bytes (0: not known).
static uint64_t bytes_from(const void *p) {
    hipDeviceptr_t base = nullptr;
    size_t size = 0;
    if (hipMemGetAddressRange(&base, &size, const_cast<void *>(p)) != hipSuccess) {
        (void)hipGetLastError();
        return 0;
    }
    return (uint64_t)((const char *)base + size - (const char *)p);
}

void free_parts(rambo_s *h) {
    std::lock_guard<std::mutex> g(h->parts_mu);
    if (!h->d_parts) return;
    if (h->parts_done) (void)hipEventSynchronize(h->parts_done);
    (void)hipFree(h->d_parts);
    h->d_parts = nullptr;
    h->parts_bytes = 0;
}

// Positions that an insertion of n_docs documents is taken to hold, where the
// buffer does not say: the index's K documents fill its filters to three quarters
// at most (2 m ln 2 / eta terms a filter, B of them for the K documents), or 2^17
// positions a document if that is more. The buffer may be a store of documents,
// of which the call inserts a few: without this bound a document of 100 kbp out
// of 10 GB went through 132 rounds of launches that found nothing to do (17.4 ms,
// K=101,000; 0.04 ms out of a buffer of its own).
static uint64_t likely_positions(const rambo_s *h, uint64_t n_docs) {
    const double full = 2 * 0.6931 * (double)h->m * h->B / h->eta;  // of all K
    const double docs = (double)n_docs * std::max(full / (double)h->K, 131072.0);
    return (uint64_t)std::min(docs, std::max(full, 4194304.0));
}

// The partitioned insertion of at most `most` positions, if it pays; *taken says
// whether it was enqueued. Word terms stay direct: most of a document's bits are
// words that others have set already, and a load shows that sooner than the
// partition (11.5 million terms of 17,618 documents into an index that holds
// others: 0.73 ms direct, 0.73 ms partitioned; again 0.38 and 0.60).
template <bool SEQS>
static int launch_parts(rambo_s *h, const Docs &in, uint64_t most, hipStream_t s, bool *taken) {
    *taken = false;
    const uint64_t rep_bytes = h->m * h->RW * 4;
    // direct 33 to 50 ps a bit, partitioned 5.3 ps a bit, 0.9 ms a GiB of rows and
    // 45 us a repetition: equal near 1.6 million bits and one per 32 bytes of rows
    const uint64_t least_bits = 1600000 + rep_bytes / 32;
    // (more than two million positions: the bound may be an allocation's, and small
    // tensors share one of 2 MB)
    const uint64_t least = std::max<uint64_t>((2 << 20) + 1, (least_bits + h->eta - 1) / h->eta);
    if (h->opaque || most < least) return RAMBO_OK;
    hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(s, &cap) != hipSuccess || cap != hipStreamCaptureStatusNone) return RAMBO_OK;
    Parts pt;
    pt.groups = (uint32_t)h->n_cu;
    // buckets of a tile at least, and not more than there are places for
    pt.lg = kBucketBits - 5 - std::min<uint32_t>(h->log2RW, kBucketBits - 5);
    while ((((h->m - 1) >> pt.lg) + 1) > kBuckets) pt.lg++;
    pt.buckets = (uint32_t)(((h->m - 1) >> pt.lg) + 1);
    pt.slots = kStage / kBuckets;
    while (pt.slots * 2 * pt.buckets <= kStage && pt.slots < 4096) pt.slots *= 2;
    const uint32_t bucket_bits = pt.lg + h->log2RW + 5;
    // (every tile of a bucket reads the bucket's bits: at 64 tiles, a repetition of
    // 8 GiB, 5 x 10^10 bits in 1.10 s, 2.57 directly; at 128, 16 GiB, 1.2 x 10^11
    // bits in 4.1 s, 5.1 directly; at 256 it would take longer)
    if (bucket_bits > kTileBits + 7) return RAMBO_OK;
    // segments of the mean number of bits and eight deviations more, and their counts
    const uint64_t segs = (uint64_t)pt.buckets * pt.groups;
    const uint64_t room = std::max<uint64_t>(256ull << 20, std::min<uint64_t>(h->rows_bytes, 4ull << 30));
    auto seg_cap = [&](uint64_t positions) {
        const double mean = (double)positions * h->eta / (double)segs;
        return ((uint64_t)(mean + 8 * std::sqrt(mean)) + 16 + 15) & ~15ull;
    };
    auto chunk_of = [&](uint64_t passes) { return ((most + passes - 1) / passes + 1023) & ~1023ull; };
    auto words_of = [&](uint64_t chunk) { return (segs * (seg_cap(chunk) + 1) + 3) & ~3ull; };  // of a repetition
    uint64_t passes = 1;
    while (words_of(chunk_of(passes)) * 4 > room && chunk_of(passes) > 1024) passes++;
    pt.chunk = chunk_of(passes);
    pt.cap = (uint32_t)seg_cap(pt.chunk);
    pt.least = least;
    // all repetitions in one launch where their segments fit together (the launches
    // are then few, should the documents turn out to be small)
    const bool together = passes == 1 && h->R * words_of(pt.chunk) * 4 <= room;
    pt.rep = together ? words_of(pt.chunk) : 0;
    const uint64_t need = (together ? h->R : 1) * words_of(pt.chunk) * 4;
    if (need > room) return RAMBO_OK;
    std::lock_guard<std::mutex> g(h->parts_mu);
    if (h->parts_bytes < need) {
        if (h->d_parts) (void)hipFree(h->d_parts);  // (waits for the work that uses it)
        h->d_parts = nullptr;
        h->parts_bytes = 0;
        if (hipMalloc(&h->d_parts, need) != hipSuccess) {
            (void)hipGetLastError();
            h->d_parts = nullptr;
            return RAMBO_OK;
        }
        h->parts_bytes = need;
    }
    if (!h->parts_done) HIP_CHECK(hipEventCreateWithFlags(&h->parts_done, hipEventDisableTiming));
    else HIP_CHECK(hipStreamWaitEvent(s, h->parts_done, 0));
    pt.bits = (uint32_t *)h->d_parts;
    pt.count = pt.bits + segs * pt.cap;
    const Index ix = make_index(h);
    const size_t lds = (size_t)(kStage + kBuckets * 2) * 4;
    const uint32_t lgt = std::min<uint32_t>(bucket_bits, kTileBits), tiles = 1u << (bucket_bits - lgt);
    // (resident: 64 KB of LDS a workgroup of 512 threads, two a compute unit, else one)
    const unsigned resident = ((unsigned)h->n_cu * (lgt > kBucketBits ? 1 : 2) + 7) / 8 * 8;
    unsigned apply = ((pt.buckets + 7) / 8) * 8 * tiles;
    if (apply > kApplyGroups) apply = resident;
    const unsigned reps = together ? h->R : 1;
    for (uint64_t c = 0; c < passes; c++)
        for (uint32_t r = 0; r < h->R; r += reps) {
            hipLaunchKernelGGL(k_part_scatter<SEQS>, dim3(pt.groups, reps), dim3(1024), lds, s, ix, in, pt, r, (uint32_t)c,
                               h->d_invalid);
            hipLaunchKernelGGL(k_part_apply, dim3(apply, reps), dim3(lgt > kBucketBits ? 1024 : 512),
                               (size_t)1 << (lgt - 3), s, ix, in, pt, r, (uint32_t)c, tiles, lgt);
        }
    // an insertion that turns out to be small, or the positions past `most`
    hipLaunchKernelGGL(k_build<SEQS>, dim3((unsigned)h->n_cu * 16), dim3(256), 0, s, ix, in, passes * pt.chunk, least,
                       h->d_invalid);
    HIP_CHECK(hipGetLastError());
    HIP_CHECK(hipEventRecord(h->parts_done, s));
    *taken = true;
    return RAMBO_OK;
}

template <bool SEQS>
static int launch_build(rambo_s *h, const Docs &in, uint64_t most, hipStream_t s) {
    bool taken = false;
    const int st = launch_parts<SEQS>(h, in, most, s, &taken);
    if (st != RAMBO_OK || taken) return st;
    // the grid is persistent (grid-stride); the number of positions is only known on the device
    hipLaunchKernelGGL(k_build<SEQS>, dim3((unsigned)h->n_cu * 16), dim3(256), 0, s, make_index(h), in, (uint64_t)0,
                       (uint64_t)0, h->d_invalid);
    HIP_CHECK(hipGetLastError());
    return RAMBO_OK;
}

int launch_build_kmers(rambo_s *h, const uint64_t *kmers, const uint64_t *koff, const uint64_t *doc_ids,
                       uint64_t n_docs, hipStream_t s, uint64_t positions) {
    const uint64_t most = positions ? positions : std::min(bytes_from(kmers) / 8, likely_positions(h, n_docs));
    return launch_build<false>(h, Docs{kmers, nullptr, koff, doc_ids, n_docs}, most, s);
}

int launch_build_seqs(rambo_s *h, const uint8_t *seqs, const uint64_t *offs, const uint64_t *doc_ids,
                      uint64_t n_docs, hipStream_t s) {
    return launch_build<true>(h, Docs{nullptr, seqs, offs, doc_ids, n_docs},
                              std::min(bytes_from(seqs), likely_positions(h, n_docs)), s);
}

int launch_dump_bfu(rambo_s *h, uint32_t r, uint32_t b, uint64_t *d_out, hipStream_t s) {
    const uint64_t words = (h->m + 63) / 64;
    hipLaunchKernelGGL(k_dump_bfu, dim3(grid_for(h, words, 16)), dim3(256), 0, s, make_index(h), r, b, d_out);
    HIP_CHECK(hipGetLastError());
    return RAMBO_OK;
}

}  // namespace rambo

namespace rambo {

// Folding over (Section 5.3): BFU'(r, b) = BFU(r, b) OR BFU(r, b + B/2) for
// b < B/2. In the bit-sliced layout this is, per row, the OR of the row's low
// B/2 bits with its bits [B/2, B) shifted down by B/2. One thread per output
// word; rows of RWo words (RWo = power of two >= ceil(B/2 / 32)).
__global__ __launch_bounds__(256) void k_fold(const uint32_t *__restrict__ in, uint32_t *__restrict__ out,
                                              uint64_t rows, uint32_t RWi, uint32_t log2RWo, uint32_t half) {
    const uint64_t n = rows << log2RWo;
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    const uint32_t RWo = 1u << log2RWo;
    for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) {
        const uint64_t row = i >> log2RWo;
        const uint32_t w = (uint32_t)(i & (RWo - 1));
        const uint32_t *r = in + row * RWi;
        const uint32_t b0 = w * 32;  // first output bit of this word
        uint32_t keep = 0;           // output bits b0 + k with b0 + k < half
        if (b0 < half) keep = (half - b0 >= 32) ? 0xFFFFFFFFu : ((1u << (half - b0)) - 1u);
        uint32_t v = 0;
        if (keep) {
            const uint32_t lo = (w < RWi) ? r[w] : 0u;
            const uint32_t hb = half + b0, q = hb >> 5, sh = hb & 31;
            uint32_t hi = (q < RWi) ? (r[q] >> sh) : 0u;
            if (sh && q + 1 < RWi) hi |= r[q + 1] << (32 - sh);
            v = (lo | hi) & keep;
        }
        out[i] = v;
    }
}

// Rows of at most 128 bits (B <= 128): one thread per row, which loads the
// row whole, folds it as one 128-bit value, v | (v >> B/2) on the low B/2
// bits, and stores the folded row whole -- one load and one store per row,
// coalesced across the wave.
template <int RWI>
__global__ __launch_bounds__(256) void k_fold_rows(const uint32_t *__restrict__ in, uint32_t *__restrict__ out,
                                                   uint64_t rows, uint32_t RWo, uint32_t half) {
    typedef unsigned __int128 u128;
    const u128 keep = (((u128)1) << half) - 1;  // half <= 64
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    for (uint64_t row = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; row < rows; row += stride) {
        u128 v;
        if constexpr (RWI == 4) {
            const uint4 a = reinterpret_cast<const uint4 *>(in)[row];
            v = (u128)a.x | ((u128)a.y << 32) | ((u128)a.z << 64) | ((u128)a.w << 96);
        } else if constexpr (RWI == 2) {
            const uint2 a = reinterpret_cast<const uint2 *>(in)[row];
            v = (u128)a.x | ((u128)a.y << 32);
        } else {
            v = in[row];
        }
        const u128 f = (v | (v >> half)) & keep;
        if (RWo == 2) {
            reinterpret_cast<uint2 *>(out)[row] = make_uint2((uint32_t)f, (uint32_t)(f >> 32));
        } else {
            out[row] = (uint32_t)f;
        }
    }
}

int launch_fold(rambo_s *h, const uint32_t *in, uint32_t *out, uint32_t RWi, uint32_t log2RWo, uint32_t half,
                hipStream_t s) {
    const uint64_t rows = (uint64_t)h->R * h->m;
    const dim3 grid((unsigned)h->n_cu * 32), block(256);
    const uint32_t RWo = 1u << log2RWo;  // (half <= 64 when RWi <= 4: RWo is 1 or 2)
    if (RWi == 4) hipLaunchKernelGGL(k_fold_rows<4>, grid, block, 0, s, in, out, rows, RWo, half);
    else if (RWi == 2) hipLaunchKernelGGL(k_fold_rows<2>, grid, block, 0, s, in, out, rows, RWo, half);
    else if (RWi == 1) hipLaunchKernelGGL(k_fold_rows<1>, grid, block, 0, s, in, out, rows, RWo, half);
    else hipLaunchKernelGGL(k_fold, grid, block, 0, s, in, out, rows, RWi, log2RWo, half);
    HIP_CHECK(hipGetLastError());
    return RAMBO_OK;
}

// ---------------------------------------------------------------------------
// Checksum of the row array (index files): the sum, mod 2^64, of the
// SplitMix64 output function (Steele, Lea and Flood, OOPSLA 2014) applied to
// (word index << 32 | word) over every 32-bit word. Each term depends on a
// word's value and place, so a changed, moved or missing word changes the sum
// except with probability about 2^-64; the sum is independent of the order of
// accumulation, so the grid adds its partial sums with atomics.
// ---------------------------------------------------------------------------
__device__ __forceinline__ uint64_t mix_word(uint64_t z) {
    z += 0x9E3779B97F4A7C15ull;
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    return z ^ (z >> 31);
}

__global__ __launch_bounds__(256) void k_rows_checksum(const uint32_t *__restrict__ w, uint64_t n,
                                                       unsigned long long *sum) {
    uint64_t acc = 0;
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride)
        acc += mix_word((i << 32) | w[i]);
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) acc += __shfl_xor(acc, off);
    __shared__ unsigned long long part[4];
    if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = acc;
    __syncthreads();
    if (threadIdx.x == 0) atomicAdd(sum, part[0] + part[1] + part[2] + part[3]);
}

int rows_checksum(rambo_s *h, uint64_t *out, hipStream_t s) {
    unsigned long long *d = nullptr;
    HIP_CHECK(hipMallocAsync((void **)&d, 8, s));
    int st = RAMBO_OK;
    if (hipMemsetAsync(d, 0, 8, s) != hipSuccess) st = fail(RAMBO_EDEVICE, "checksum: memset failed");
    if (st == RAMBO_OK) {
        hipLaunchKernelGGL(k_rows_checksum, dim3((unsigned)(h->n_cu * 8)), dim3(256), 0, s, h->rows,
                           h->rows_bytes / 4, d);
        if (hipGetLastError() != hipSuccess ||
            hipMemcpyAsync(out, d, 8, hipMemcpyDeviceToHost, s) != hipSuccess ||
            hipStreamSynchronize(s) != hipSuccess)
            st = fail(RAMBO_EDEVICE, "checksum: launch or copy failed");
    }
    (void)hipFreeAsync(d, s);
    (void)hipStreamSynchronize(s);
    return st;
}

}  // namespace rambo
