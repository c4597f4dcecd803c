// Term queries: single k-mers or word terms, and term sets (Algorithm 2;
// Section 3.3.1 for sets).
//
// A term's answer is R masks of B bits (the rows of its eta hashes ANDed, per
// repetition) and then, per document, the AND of R mask bits. Testing every
// (query, document) pair bit by bit made the resolve the bound (50,000
// documents x 3 repetitions per query). Here a group of 64 queries is
// resolved together, bit-sliced over the queries: the group's masks are
// transposed in LDS into T[r][c], the 64-bit set of the group's queries whose
// repetition-r mask has cell c; the queries of document d are then
// AND_r T[r][phi_r(d)], R LDS reads for all 64 queries, and a 64 x 64 bit
// transpose across the wave turns 64 documents' query sets into one result
// word of every query. What remains per query is its rows and its result row.
#include <algorithm>
#include <type_traits>

#include "rambo_int.h"

namespace rambo {

// The index as the group kernels see it, with the documents' cells in the
// order of their resolve (rambo_s::d_docslot).
struct TermIndex : Index {
    const uint4 *docslot;  // [R][ceil(W / 8)][64]
};

// Lane constants of the 64 x 64 transpose: byte selectors of the stages that
// exchange 16-bit and 8-bit blocks, rotations and keep masks of the 4-, 2- and
// 1-bit ones.
struct Transpose {
    uint32_t sel16, sel8, rot4, keep4, rot2, keep2, rot1, keep1;
    __device__ __forceinline__ explicit Transpose(uint32_t lane) {
        sel16 = lane & 16 ? 0x07060302u : 0x05040100u;
        sel8 = lane & 8 ? 0x03070105u : 0x06020400u;
        rot4 = lane & 4 ? 4u : 28u;
        keep4 = lane & 4 ? 0xF0F0F0F0u : 0x0F0F0F0Fu;
        rot2 = lane & 2 ? 2u : 30u;
        keep2 = lane & 2 ? 0xCCCCCCCCu : 0x33333333u;
        rot1 = lane & 1 ? 1u : 31u;
        keep1 = lane & 1 ? 0xAAAAAAAAu : 0x55555555u;
    }
};

template <int CTRL>
__device__ __forceinline__ uint32_t dpp(uint32_t v) {
    return (uint32_t)__builtin_amdgcn_mov_dpp((int)v, CTRL, 0xF, 0xF, true);
}

// bits of a where the mask is set, of b elsewhere (one bit-field insert)
__device__ __forceinline__ uint32_t pick(uint32_t mask, uint32_t a, uint32_t b) { return ((a ^ b) & mask) ^ b; }

// The five stages inside each 32-bit half: blocks of 16, 8, 4, 2, 1 bits
// exchanged with lane ^ 16 (row swap), ^ 8 (row rotate by 8), ^ 4 (reversed
// quads, mirrored half-row), ^ 2 and ^ 1 (quad permutes).
__device__ __forceinline__ uint32_t transpose32(uint32_t v, const Transpose &t) {
    const auto s = __builtin_amdgcn_permlane16_swap(v, v, false, false);
    v = __builtin_amdgcn_perm(s[1], s[0], t.sel16);
    v = __builtin_amdgcn_perm(dpp<0x128>(v), v, t.sel8);
    uint32_t o = dpp<0x141>(dpp<0x1B>(v));
    v = pick(t.keep4, v, __builtin_amdgcn_alignbit(o, o, t.rot4));
    o = dpp<0x4E>(v);
    v = pick(t.keep2, v, __builtin_amdgcn_alignbit(o, o, t.rot2));
    o = dpp<0xB1>(v);
    return pick(t.keep1, v, __builtin_amdgcn_alignbit(o, o, t.rot1));
}

// 64 x 64 bit transpose across a wave: bit j of lane i's x becomes bit i of
// lane j's result. The 32-bit halves change places with one lane swap; about
// 30 vector instructions and no LDS (the butterfly by lane shuffles takes 12
// LDS permutes and three times the instructions). All 64 lanes.
__device__ __forceinline__ uint64_t transpose64(uint64_t x, const Transpose &t) {
    const auto s = __builtin_amdgcn_permlane32_swap((uint32_t)x, (uint32_t)(x >> 32), false, false);
    return (uint64_t)transpose32(s[0], t) | ((uint64_t)transpose32(s[1], t) << 32);
}

// The group's T in LDS: per repetition, blocks of 64 cells of 65 words (one
// word of padding spreads a query's mask words, one block apart, over the
// banks). Block k of repetition r first holds the queries' mask words (word t:
// bits 64 k .. 64 k + 63 of query t's mask), then, transposed, its cells' query
// sets. ix.docslot holds the documents' cells as slots c + c / 64 of this array.
// A group of 32 queries has words of 32 bits instead: a block first holds the low
// halves of its 32 mask words, then the high halves.
constexpr uint32_t kBlockWords = 65;
__host__ __device__ inline uint32_t t_blocks(uint32_t B) { return (B + 63) / 64; }
__host__ __device__ inline uint32_t t_words(uint32_t R, uint32_t B) { return R * t_blocks(B) * kBlockWords; }

__device__ __forceinline__ void transpose_blocks(uint64_t *T, uint32_t blocks, uint32_t wave, uint32_t waves,
                                                 uint32_t lane, const Transpose &tp) {
    for (uint32_t k = wave; k < blocks; k += waves) {
        const uint64_t x = T[k * kBlockWords + lane];
        if (__ballot(x != 0)) T[k * kBlockWords + lane] = transpose64(x, tp);
    }
}
__device__ __forceinline__ void transpose_blocks(uint32_t *T, uint32_t blocks, uint32_t wave, uint32_t waves,
                                                 uint32_t lane, const Transpose &tp) {
    for (uint32_t k = wave; k < blocks; k += waves) {
        const uint32_t x = T[k * kBlockWords + lane];
        if (__ballot(x != 0)) T[k * kBlockWords + lane] = transpose32(x, tp);
    }
}

// Transpose of 16-byte pieces across each P lanes (P = 4 or 8): piece j of
// lane i becomes piece i of lane j.
template <int P>
__device__ __forceinline__ void transpose_pieces(uint32_t (&w)[4 * P], uint32_t lane) {
#pragma unroll
    for (int d = 1; d < P; d <<= 1) {
        const bool up = lane & d;
#pragma unroll
        for (int p = 0; p < P; p++) {
            if (p & d) continue;
#pragma unroll
            for (int k = 0; k < 4; k++) {
                const uint32_t a = w[4 * p + k], b = w[4 * (p + d) + k];
                const uint32_t v = up ? a : b;  // the one that leaves the lane
                const uint32_t o = d == 1 ? dpp<0xB1>(v) : d == 2 ? dpp<0x4E>(v) : dpp<0x141>(dpp<0x1B>(v));
                w[4 * p + k] = up ? o : a;
                w[4 * (p + d) + k] = up ? b : o;
            }
        }
    }
}

// Result words of 64 N documents (chunk c: words N c .. N c + N - 1, N = 8 or
// 16) for the group's nq queries. Lane t ends with query t's N words; N / 2
// lanes exchange them so that a store writes N * 8 contiguous bytes of a row
// (16 bytes of 64 rows a store made the stores the bound: 10^7 terms at W = 16
// 2.35 ms, 200,000 at W = 782 0.99 ms). Rows are 8-byte aligned.
template <int R, int N>
__device__ __forceinline__ void resolve_chunk(const TermIndex &ix, const uint64_t *T, uint64_t *__restrict__ out,
                                              uint64_t base, uint32_t nq, uint32_t c, uint32_t lane,
                                              const Transpose &tp) {
    const uint32_t records = (ix.W + 7) / 8, stride = t_blocks(ix.B) * kBlockWords;
    uint32_t w[2 * N];
#pragma unroll
    for (int h = 0; h < N / 8; h++) {
        const uint32_t rec = c * (N / 8) + h;
        uint32_t slot[R][4];
#pragma unroll
        for (int r = 0; r < R; r++) {
            const uint4 v = ix.docslot[((uint64_t)r * records + min(rec, records - 1)) * 64 + lane];
            slot[r][0] = v.x; slot[r][1] = v.y; slot[r][2] = v.z; slot[r][3] = v.w;
        }
#pragma unroll
        for (int k = 0; k < 8; k += 2) {
            // (two words at a time, so that only their reads are in registers)
            __builtin_amdgcn_sched_barrier(0);
            if (rec * 8 + k >= ix.W) {  // no such words
                w[16 * h + 2 * k] = w[16 * h + 2 * k + 1] = w[16 * h + 2 * k + 2] = w[16 * h + 2 * k + 3] = 0;
                continue;
            }
#pragma unroll
            for (int j = 0; j < 2; j++) {
                uint64_t q = ~0ULL;
#pragma unroll
                for (int r = 0; r < R; r++) {
                    const uint32_t s = j ? slot[r][k >> 1] >> 16 : slot[r][k >> 1] & 0xFFFFu;
                    q &= T[r * stride + s];
                }
                const uint64_t d = ((uint64_t)rec * 8 + k + j) * 64 + lane;
                if (d >= ix.K) q = 0;  // (the slots past K are 0, a real cell)
                const uint64_t v = transpose64(q, tp);
                w[16 * h + 2 * (k + j)] = (uint32_t)v;
                w[16 * h + 2 * (k + j) + 1] = (uint32_t)(v >> 32);
            }
        }
    }
    constexpr uint32_t P = N / 2;
    transpose_pieces<(int)P>(w, lane);
    const uint32_t k = c * N + 2 * (lane % P);  // this lane's words k, k + 1 of rows q0 .. q0 + P - 1
    const uint32_t q0 = lane & ~(P - 1);
    uint64_t *o = out + (base + q0) * ix.W + k;
#pragma unroll
    for (uint32_t i = 0; i < P; i++) {
        if (q0 + i < nq) {
            if (k + 1 < ix.W) __builtin_memcpy(o + (uint64_t)i * ix.W, w + 4 * i, 16);
            else if (k < ix.W) __builtin_memcpy(o + (uint64_t)i * ix.W, w + 4 * i, 8);
        }
    }
}

// The same for a group of 32 queries and N = 16: the transpose takes word k of both
// halves of the chunk at a time, so that lanes t and 32 + t end with words 0 to 7
// and 8 to 15 of query t; the pieces' exchange has two more stages, which bring
// the halves of a row eight lanes together again.
template <int R, int N>
__device__ __forceinline__ void resolve_chunk(const TermIndex &ix, const uint32_t *T, uint64_t *__restrict__ out,
                                              uint64_t base, uint32_t nq, uint32_t c, uint32_t lane,
                                              const Transpose &tp) {
    static_assert(N == 16, "two records of eight words");
    const uint32_t records = (ix.W + 7) / 8, stride = t_blocks(ix.B) * kBlockWords;
    uint32_t slot[2][R][4], w[16];
#pragma unroll
    for (int h = 0; h < 2; h++)
#pragma unroll
        for (int r = 0; r < R; r++) {
            const uint4 v = ix.docslot[((uint64_t)r * records + min(2 * c + h, records - 1)) * 64 + lane];
            slot[h][r][0] = v.x; slot[h][r][1] = v.y; slot[h][r][2] = v.z; slot[h][r][3] = v.w;
        }
#pragma unroll
    for (int k = 0; k < 8; k++) {
        if (k % 2 == 0) __builtin_amdgcn_sched_barrier(0);
        uint32_t q[2];
#pragma unroll
        for (int h = 0; h < 2; h++) {
            q[h] = ~0u;
#pragma unroll
            for (int r = 0; r < R; r++) {
                const uint32_t s = k % 2 ? slot[h][r][k >> 1] >> 16 : slot[h][r][k >> 1] & 0xFFFFu;
                q[h] &= T[r * stride + s];
            }
            if (((uint64_t)c * 16 + 8 * h + k) * 64 + lane >= ix.K) q[h] = 0;  // (the slots past K are 0, a real cell)
        }
        const uint64_t v = transpose64((uint64_t)q[1] << 32 | q[0], tp);
        w[2 * k] = (uint32_t)v;
        w[2 * k + 1] = (uint32_t)(v >> 32);
    }
    transpose_pieces<4>(w, lane);  // piece i: words 8 h + 2 (lane % 4) of query (lane % 32 & ~3) + i
    // pieces 2, 3 change places with the other half's 0, 1; then 2, 3 with lane ^ 4's 0, 1
    const bool up = lane & 4;
#pragma unroll
    for (int p = 0; p < 2; p++)
#pragma unroll
        for (int k = 0; k < 4; k++) {
            const auto x = __builtin_amdgcn_permlane32_swap(w[4 * p + k], w[4 * (p + 2) + k], false, false);
            const uint32_t a = x[0], b = x[1];
            const uint32_t o = dpp<0x141>(dpp<0x1B>(up ? a : b));
            w[4 * p + k] = up ? o : a;
            w[4 * (p + 2) + k] = up ? b : o;
        }
    const uint32_t k = c * 16 + 2 * (lane & 7);
    const uint32_t q0 = (lane & 24) | (lane >> 5) << 1;
#pragma unroll
    for (uint32_t i = 0; i < 4; i++) {
        const uint32_t q = q0 | (i & 2) << 1 | (i & 1);
        if (q < nq) {
            uint64_t *o = out + (base + q) * ix.W + k;
            if (k + 1 < ix.W) __builtin_memcpy(o, w + 4 * i, 16);
            else if (k < ix.W) __builtin_memcpy(o, w + 4 * i, 8);
        }
    }
}

// The documents of one of the slices, in chunks of N words, every waves-th one
// from the wave-th: a batch of few groups is cut into slices so that it fills
// the chip, each slice probing its group's terms again.
struct Slice {
    uint32_t at, of;
};
template <int R, int N, typename Q>
__device__ __forceinline__ void resolve_chunks(const TermIndex &ix, const Q *T, uint64_t *__restrict__ out,
                                               uint64_t base, uint32_t nq, uint32_t wave, uint32_t waves,
                                               uint32_t lane, const Transpose &tp, Slice sl) {
    const uint32_t chunks = (ix.W + N - 1) / N, per = (chunks + sl.of - 1) / sl.of;
    const uint32_t c0 = min(chunks, sl.at * per), c1 = min(chunks, c0 + per);
    for (uint32_t c = c0 + wave; c < c1; c += waves) resolve_chunk<R, N>(ix, T, out, base, nq, c, lane, tp);
}

template <int N, typename Q>
__device__ __forceinline__ void resolve_group(const TermIndex &ix, const Q *T, uint64_t *__restrict__ out,
                                              uint64_t base, uint32_t nq, uint32_t wave, uint32_t waves,
                                              uint32_t lane, const Transpose &tp, Slice sl) {
    switch (ix.R) {
#define RAMBO_R_(R_) case R_: resolve_chunks<R_, N>(ix, T, out, base, nq, wave, waves, lane, tp, sl); break;
    RAMBO_R_(1) RAMBO_R_(2) RAMBO_R_(3) RAMBO_R_(4) RAMBO_R_(5) RAMBO_R_(6) RAMBO_R_(7) RAMBO_R_(8)
#undef RAMBO_R_
    }
}

// Query t's masks of repetitions FIRST .. FIRST + COUNT - 1 (those below R) into
// the blocks: this lane holds SEG consecutive row words from word seg * SEG.
template <int SEG, int FIRST, int COUNT, typename Q>
__device__ __forceinline__ void store_masks(const Index &ix, const Seg<SEG> (&cm)[COUNT], uint32_t seg, uint32_t t,
                                            Q *T) {
    const uint32_t nb = t_blocks(ix.B);
#pragma unroll
    for (int i = 0; i < COUNT; i++) {
        if (FIRST + i >= (int)ix.R) continue;
#pragma unroll
        for (int s = 0; s < SEG; s += 2) {
            const uint32_t k = (seg * SEG + s) / 2;
            uint64_t v = cm[i].w[s];
            if constexpr (SEG > 1) v |= (uint64_t)cm[i].w[s + 1] << 32;
            if (k >= nb) continue;
            Q *b = T + ((FIRST + i) * nb + k) * kBlockWords + t;
            b[0] = (Q)v;
            if constexpr (sizeof(Q) == 4) b[32] = (Q)(v >> 32);
        }
    }
}

template <int SEG, int COUNT>
__device__ __forceinline__ void fill_masks(Seg<SEG> (&cm)[COUNT], uint32_t v) {
#pragma unroll
    for (int i = 0; i < COUNT; i++)
#pragma unroll
        for (int s = 0; s < SEG; s++) cm[i].w[s] = v;
}

// Rows of at most 4 words (B <= 128): a lane holds a term's whole masks, and
// a wave resolves its own 64 terms, with T in its own LDS area.
// Bound by random row reads (one 128-byte line each): repetition 0's rows are
// read first, then repetition 1's, then the others', and a term that no document
// of the index holds (half of a typical batch) mostly stops early: with B = 32
// three quarters of those have no positive cell left after each. K=1,000 (B=32, R=4, eta=3, rows of 1 GiB), 10^7
// terms: 3.17 ms with all 12 rows read at once, one ballot per cell and 8-byte
// stores; 2.35 ms in this form with 16-byte stores 128 bytes apart; 2.02 ms with
// 64-byte, 1.83 ms with 128-byte stores (1.44 ms with none: the 1.28 GB of
// results and the row reads share HBM); 1.76 ms with repetition 1 apart.
template <int SEG>
__global__ __launch_bounds__(256) void k_terms_lane(TermIndex ix, const uint64_t *__restrict__ terms, uint64_t n,
                                                    uint64_t *__restrict__ out, unsigned long long *invalid) {
    extern __shared__ uint64_t smem64[];
    const uint32_t lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    uint64_t *T = smem64 + wave * t_words(ix.R, ix.B);
    const uint64_t base = ((uint64_t)blockIdx.x * (blockDim.x >> 6) + wave) * 64;
    if (base >= n) return;
    const Transpose tp(lane);
    Seg<SEG> acc[MAXR];
    set_ones(acc);
    auto some = [&](int r) {
        uint32_t o = 0;
#pragma unroll
        for (int s = 0; s < SEG; s++) o |= acc[r].w[s];
        return o != 0;
    };
    bool go = base + lane < n;
    uint64_t x = go ? terms[base + lane] : 0;
    if (go && !ix.opaque) {
        if (x >> 62) {
            if (blockIdx.y == 0) atomicAdd(invalid, 1ULL);
            go = false;
        } else {
            x = canonical(x);
        }
    }
    if (go) {
        probe_reps<SEG, 0, 1>(ix, ix.hp->h, x, 0, acc);
        go = some(0);
        if (go) probe_reps<SEG, 1, 1, 1>(ix, ix.hp->h, x, 0, acc);
        go = go && some(1);
        if (go) probe_reps<SEG, 2, 3, 2>(ix, ix.hp->h, x, 0, acc);
        if (go && ix.R > 5) probe_reps<SEG, 5, MAXR - 5, 5>(ix, ix.hp->h, x, 0, acc);
    } else {
#pragma unroll
        for (int s = 0; s < SEG; s++) acc[0].w[s] = 0;
    }
    const uint32_t nq = (uint32_t)min<uint64_t>(64, n - base);
    bool live = go;
#pragma unroll
    for (int r = 2; r < MAXR; r++)
        if (r < (int)ix.R) live = live && some(r);
    if (__ballot(live) == 0) {
        // no document for any of the terms (one k-mer that no document holds,
        // K=10,000: 23 us through the resolve, 21 without)
        const uint32_t words = ((ix.W + 15) / 16 + gridDim.y - 1) / gridDim.y * 16;
        const uint32_t w0 = min(ix.W, blockIdx.y * words), w1 = min(ix.W, w0 + words);
        for (uint32_t q = 0; q < nq; q++)
            for (uint32_t w = w0 + lane; w < w1; w += 64) out[(base + q) * ix.W + w] = 0;
        return;
    }
    const uint32_t nb = t_blocks(ix.B);
#pragma unroll
    for (int r = 0; r < MAXR; r++) {
        if (r >= (int)ix.R) continue;
#pragma unroll
        for (int s = 0; s < SEG; s += 2) {
            if ((uint32_t)s / 2 >= nb) continue;
            uint64_t v = acc[r].w[s];
            if constexpr (SEG > 1) v |= (uint64_t)acc[r].w[s + 1] << 32;
            T[(r * nb + s / 2) * kBlockWords + lane] = transpose64(v, tp);
        }
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    resolve_group<16>(ix, T, out, base, nq, 0, 1, lane, tp, Slice{blockIdx.y, gridDim.y});
}

// Wider rows: G = 2^lg lanes share a term's row (4 words each) and a workgroup
// resolves 64 or 32 terms (of the type Q: a bit a term); all rows of up to four
// repetitions are in flight at once.
// Bound by the result stores and the resolve's LDS reads where the index is cached
// (ClueWeb-like, 50,000 documents, R=3, B=5,000, 200,000 terms, 1.25 GB of
// results: 14.7 ms with a candidate resolve per term; 0.64 ms in groups of 64,
// whose T of 123 KB leaves one workgroup a CU, 0.45 ms of it without the stores,
// the probes 0.13 ms; 0.55 ms in groups of 32, two workgroups a CU, one of which
// probes while the other stores; 0.58 ms with 24 waves a CU instead of 16, for
// which registers are spilled).
template <typename Q>
__global__ __launch_bounds__(1024) void k_terms_group(TermIndex ix, const uint64_t *__restrict__ terms, uint64_t n,
                                                      uint64_t *__restrict__ out, unsigned long long *invalid,
                                                      uint32_t lg) {
    extern __shared__ uint64_t smem64[];
    constexpr uint32_t kQ = 8 * sizeof(Q);  // queries of a group
    Q *T = (Q *)smem64;
    const uint32_t lane = threadIdx.x & 63, wave = threadIdx.x >> 6, waves = blockDim.x >> 6;
    const uint64_t base = (uint64_t)blockIdx.x * kQ;
    const Transpose tp(lane);
    const uint32_t per = 64u >> lg, g = lane >> lg, seg = lane & ((1u << lg) - 1);
    uint64_t mine = 0;  // term base + lane
    bool mine_ok = lane < kQ && base + lane < n;
    if (mine_ok) mine = terms[base + lane];
    if (mine_ok && !ix.opaque && (mine >> 62)) {
        mine_ok = false;
        if (wave == 0 && blockIdx.y == 0) atomicAdd(invalid, 1ULL);
    }
    if (!ix.opaque) mine = canonical(mine);
    const uint64_t oks = __ballot(mine_ok);
    for (uint32_t t0 = wave * per; t0 < kQ; t0 += waves * per) {
        const uint32_t t = t0 + g;
        const uint64_t x = __shfl(mine, (int)t);
        // (lanes past the last cell's word have nothing to read: at B=5,000 24 of 64)
        const bool ok = ((oks >> t) & 1) && seg * 128 < ix.B;
        {
            Seg<4> cm[4];
            fill_masks(cm, ok ? 0xFFFFFFFFu : 0u);
            if (ok) probe_reps<4, 0, 4>(ix, ix.hp->h, x, seg, cm);
            store_masks<4, 0, 4>(ix, cm, seg, t, T);
        }
        if (ix.R > 4) {
            Seg<4> cm[4];
            fill_masks(cm, ok ? 0xFFFFFFFFu : 0u);
            if (ok) probe_reps<4, 4, 4>(ix, ix.hp->h, x, seg, cm);
            store_masks<4, 4, 4>(ix, cm, seg, t, T);
        }
    }
    __syncthreads();
    transpose_blocks(T, ix.R * t_blocks(ix.B), wave, waves, lane, tp);
    __syncthreads();
    resolve_group<16>(ix, T, out, base, (uint32_t)min<uint64_t>(kQ, n - base), wave, waves, lane, tp,
                      Slice{blockIdx.y, gridDim.y});
}

// Rows of U terms in repetitions FIRST .. FIRST + COUNT - 1 (those below R), all
// loads before any use; a term that there is not reads row 0 of the repetition.
template <int SEG, int FIRST, int COUNT, int U, int ETA>
__device__ __forceinline__ void probe_steps_eta(const Index &ix, const HashRec *hp, const uint64_t (&x)[U],
                                                const bool (&has)[U], uint32_t seg, Seg<SEG> (&cm)[U][COUNT]) {
    Seg<SEG> v[U][COUNT][ETA];
#pragma unroll
    for (int u = 0; u < U; u++)
#pragma unroll
        for (int k = 0; k < COUNT; k++)
            if (FIRST + k < (int)ix.R)
#pragma unroll
                for (int j = 0; j < ETA; j++) {
                    const uint64_t pos = has[u] ? bloom_pos(hash_rec(hp, (FIRST + k) * ETA + j), ix.m, x[u]) : 0;
                    v[u][k][j] = load_seg<SEG>(row_ptr(ix, FIRST + k, pos) + seg * SEG);
                }
#pragma unroll
    for (int u = 0; u < U; u++)
#pragma unroll
        for (int k = 0; k < COUNT; k++)
            if (FIRST + k < (int)ix.R)
#pragma unroll
                for (int j = 0; j < ETA; j++)
#pragma unroll
                    for (int s = 0; s < SEG; s++) cm[u][k].w[s] &= v[u][k][j].w[s];
}
template <int SEG, int FIRST, int COUNT, int U>
__device__ __forceinline__ void probe_steps(const Index &ix, const HashRec *hp, const uint64_t (&x)[U],
                                            const bool (&has)[U], uint32_t seg, Seg<SEG> (&cm)[U][COUNT]) {
    if (ix.eta == 2) probe_steps_eta<SEG, FIRST, COUNT, U, 2>(ix, hp, x, has, seg, cm);
    else if (ix.eta == 1) probe_steps_eta<SEG, FIRST, COUNT, U, 1>(ix, hp, x, has, seg, cm);
    else
#pragma unroll
        for (int u = 0; u < U; u++)
            if (has[u]) probe_reps<SEG, FIRST, COUNT>(ix, hp, x[u], seg, cm[u]);
}

// A group's term sets on their way through the repetitions: lane t of every wave
// holds set t (terms[beg .. beg + len)), alive the sets that no mask has ended.
struct SetGroup {
    const uint64_t *terms;
    uint64_t beg, len, alive;
    uint64_t *T;
    uint32_t lane, wave, waves, lg;  // 2^lg lanes share a row
    bool early_exit;
    uint64_t issued;  // probes of the group
};

// ANDs repetitions FIRST .. FIRST + COUNT - 1 of the rows of the group's sets
// into their masks in T. The sets' terms are taken in rounds, of up to 64 of
// each set at first and twice as many (to 1,024) each time; a round's terms are
// one flat list, 64 >> lg of them a wave at a time and U such steps in flight, so
// that sets of a few terms keep every wave's loads in flight. After a round
// (with early exit) a set one of whose masks is empty is done. Called by the whole
// workgroup.
template <int SEG, int FIRST, int COUNT, int U>
__device__ __forceinline__ void and_sets(const Index &ix, SetGroup &g) {
    const uint32_t lane = g.lane, per = 64u >> g.lg, in = lane >> g.lg, seg = lane & ((1u << g.lg) - 1);
    const uint32_t nb = t_blocks(ix.B), reps = min(ix.R - FIRST, (uint32_t)COUNT);
    uint32_t step = 64;
    for (uint64_t at = 0;; at += step, step = min(2 * step, 1024u)) {
        const uint32_t cnt = ((g.alive >> lane) & 1) && g.len > at ? (uint32_t)min<uint64_t>(step, g.len - at) : 0;
        const uint32_t incl = wave_inclusive(cnt, lane);
        const uint32_t total = __shfl(incl, 63);
        if (total == 0) return;
        const uint64_t src = g.beg + at - (incl - cnt);  // item i of this lane's set is terms[src + i]
        for (uint32_t i0 = g.wave * per; i0 < total; i0 += U * g.waves * per) {
            uint32_t own[U];
            uint64_t x[U];
            bool has[U];
#pragma unroll
            for (int u = 0; u < U; u++) {
                const uint32_t i = i0 + u * g.waves * per + in;
                uint32_t t = 0;  // owner of item i: the number of sets whose inclusive sum is <= i
#pragma unroll
                for (uint32_t st = 32; st; st >>= 1)
                    if (__shfl(incl, (int)(t + st - 1)) <= i) t += st;
                own[u] = t;
                const uint64_t from = __shfl(src, (int)(t & 63));
                has[u] = i < total && seg * (SEG * 32) < ix.B;
                x[u] = has[u] ? g.terms[from + i] : 0;
            }
            Seg<SEG> cm[U][COUNT];
#pragma unroll
            for (int u = 0; u < U; u++) {
                if (!ix.opaque) x[u] = canonical(x[u]);
                fill_masks(cm[u], 0xFFFFFFFFu);
            }
            if constexpr (U == 1) {
                if (has[0]) probe_reps<SEG, FIRST, COUNT>(ix, step_params(ix), x[0], seg, cm[0]);
            } else {
                // (rows of terms that there are not: row 0, in range, unused)
                probe_steps<SEG, FIRST, COUNT, U>(ix, step_params(ix), x, has, seg, cm);
            }
#pragma unroll
            for (int u = 0; u < U; u++) {
                if (!has[u]) continue;
#pragma unroll
                for (int r = 0; r < COUNT; r++) {
                    if (FIRST + r >= (int)ix.R) continue;
#pragma unroll
                    for (int s = 0; s < SEG; s += 2) {
                        const uint32_t k = (seg * SEG + s) / 2;
                        uint64_t v = cm[u][r].w[s];
                        if constexpr (SEG > 1) v |= (uint64_t)cm[u][r].w[s + 1] << 32;
                        if (k < nb)
                            __hip_atomic_fetch_and(&g.T[((FIRST + r) * nb + k) * kBlockWords + own[u]], v,
                                                   __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                    }
                }
            }
        }
        g.issued += (uint64_t)total * reps;
        __syncthreads();
        if (g.early_exit) {
            bool live = (g.alive >> lane) & 1;
            for (uint32_t r = FIRST; r < FIRST + reps; r++) {
                uint64_t o = 0;
                for (uint32_t k = 0; k < nb; k++) o |= g.T[(r * nb + k) * kBlockWords + lane];
                live = live && o != 0;
            }
            g.alive = __ballot(live);
            __syncthreads();
        }
    }
}

// The answers of a group with few positive cells, a wave a set: the sets that
// have ended get zeros, the others are resolved from their own masks (in M; only
// the first mwaves waves have room for them).
__device__ __forceinline__ void resolve_sets(const TermIndex &ix, const SetGroup &g, uint64_t *__restrict__ out,
                                             uint64_t base, uint32_t nq, uint32_t *M, uint32_t mwaves, int rmode,
                                             Slice sl) {
    const uint32_t lane = g.lane, nb = t_blocks(ix.B);
    uint32_t live = 0, ended = 0;
    for (uint32_t t = 0; t < nq; t++) {
        uint64_t *o = out + (base + t) * ix.W;
        if (!((g.alive >> t) & 1)) {
            if (ended++ % (g.waves * sl.of) == g.wave * sl.of + sl.at) write_zeros(o, ix.W, lane);
            continue;
        }
        if (live++ % (mwaves * sl.of) != g.wave * sl.of + sl.at) continue;
        for (uint32_t w = lane; w < ix.R * ix.RW; w += 64) {
            const uint32_t r = w / ix.RW, k = (w % ix.RW) / 2;
            const uint64_t v = k < nb ? g.T[(r * nb + k) * kBlockWords + t] : 0;
            M[w] = (uint32_t)(w % ix.RW & 1 ? v >> 32 : v);
        }
        OneWave().sync();
        (void)resolve(ix, M, nullptr, o, lane, rmode);
        OneWave().sync();
    }
}

// Groups of term sets that are short on average (up to kShortSet terms) take
// k_sets_group, the others k_sets_long, which both find out from the offsets: a
// batch launches both. Past that the flat list's LDS atomic a term costs more than
// a wave a set (ClueWeb-like, 30,000 sets of 64 words 1.73 ms flat, 0.99 a wave
// each; of 4 words 0.43 and 1.85).
constexpr uint32_t kShortSet = 16;
__device__ __forceinline__ bool short_sets(uint64_t len, uint32_t nq) {
#pragma unroll
    for (int d = 32; d > 0; d >>= 1) len += __shfl_xor(len, d);
    return len <= (uint64_t)kShortSet * nq;
}

// Term sets: a workgroup answers tq <= 64 sets, repetition 0 over all their
// terms first, then the others (Section 3.3.1). Bound by round trips: the
// offsets, the terms, two rounds of rows, and the result stores (Wiki-like,
// 17,618 documents, R=2, B=1,000, 100,000 sets of 2 to 8 terms, 0.22 GB of
// results: 1.44 ms with a wave and a resolve per set, 0.21 ms with a wave per
// set and the group's resolve, 0.14 ms with the flat list of terms).
// The group's resolve costs the same whatever its masks hold (K=101,000, 8 sets:
// 75 us). Where the sets' own resolves are estimated to take fewer round trips (512
// documents, or kSlotsAhead slots of 64) they are resolved one by one, and those
// that have ended cost their zeros (30,000 sets of 4 random 31-mers at K=101,000:
// 440 us with the group's resolve, 118 without).
template <int SEG>
__global__ __launch_bounds__(1024) void k_sets_group(TermIndex ix, const uint64_t *__restrict__ terms,
                                                     const uint64_t *__restrict__ offs, uint64_t n,
                                                     uint64_t *__restrict__ out, QueryOpts opt,
                                                     unsigned long long *invalid, uint32_t lg, uint32_t tq,
                                                     uint32_t mwaves) {
    extern __shared__ uint64_t smem64[];
    __shared__ unsigned long long bad_sets;
    const uint32_t lane = threadIdx.x & 63, wave = threadIdx.x >> 6, waves = blockDim.x >> 6;
    const uint64_t base = (uint64_t)blockIdx.x * tq;
    const uint32_t nq = (uint32_t)min<uint64_t>(tq, n - base);
    const Slice sl{blockIdx.y, gridDim.y};
    SetGroup g;
    g.terms = terms;
    g.T = smem64;
    g.lane = lane; g.wave = wave; g.waves = waves; g.lg = lg;
    g.early_exit = opt.early_exit != 0;
    g.beg = g.len = g.issued = 0;
    if (lane < nq) {
        g.beg = offs[base + lane];
        const uint64_t end = offs[base + lane + 1];
        g.len = end > g.beg ? end - g.beg : 0;
    }
    if (!short_sets(g.len, nq)) return;
    const bool counts = sl.at == 0 && wave == 0;  // once per set, whatever the slices
    if (counts && lane < nq && g.len == 0) atomicAdd(opt.emptyq, 1ULL);
    g.alive = __ballot(lane < nq);
    if (!ix.opaque) {
        // a k-mer index takes 31-mer codes only: a set holding another value
        // answers no document
        if (threadIdx.x == 0) bad_sets = 0;
        __syncthreads();
        for (uint32_t t = wave; t < nq; t += waves) {
            const uint64_t b = __shfl(g.beg, (int)t), l = __shfl(g.len, (int)t);
            bool bad = false;
            for (uint64_t w = 0; w < l && !bad; w += 64)
                bad = __ballot(w + lane < l && (terms[b + w + lane] >> 62)) != 0;
            if (bad && lane == 0) atomicOr(&bad_sets, 1ULL << t);
        }
        __syncthreads();
        const uint64_t bad = bad_sets;
        if (counts && lane == 0 && bad) atomicAdd(invalid, (unsigned long long)__popcll(bad));
        g.alive &= ~bad;
    }
    const uint32_t nb = t_blocks(ix.B), blocks = ix.R * nb;
    for (uint32_t k = wave; k < blocks; k += waves) g.T[k * kBlockWords + lane] = (g.alive >> lane) & 1 ? ~0ULL : 0;
    __syncthreads();
    // (few repetitions: several steps in flight instead)
    and_sets<SEG, 0, 1, 4>(ix, g);
    if (ix.R == 2) and_sets<SEG, 1, 1, 4>(ix, g);
    else if (ix.R == 3) and_sets<SEG, 1, 2, 2>(ix, g);
    else if (ix.R > 3) and_sets<SEG, 1, 4, 1>(ix, g);
    if (ix.R > 5) and_sets<SEG, 5, 3, 1>(ix, g);
    if (opt.probes && wave == 0 && lane == 0 && g.issued) atomicAdd(opt.probes, (unsigned long long)(g.issued * ix.eta));
    const uint32_t live = (uint32_t)__popcll(g.alive);
    uint64_t cells = 0;  // positive repetition-0 cells of the sets alive
    if (live) {
        for (uint32_t k = 0; k < nb; k++) cells += (uint32_t)__popcll(g.T[k * kBlockWords + lane]);
        if (!((g.alive >> lane) & 1)) cells = 0;
#pragma unroll
        for (int d = 32; d > 0; d >>= 1) cells += __shfl_xor(cells, d);
    }
    const uint64_t slots = cells * (((ix.K + ix.B - 1) / ix.B + 63) / 64);
    const uint64_t own = (slots / kSlotsAhead + 2 * live) / max(1u, min(live, mwaves * sl.of));
    if (live == 0 || own < (ix.W + 7) / 8 / (waves * sl.of)) {
        uint32_t *M = reinterpret_cast<uint32_t *>(g.T + t_words(ix.R, ix.B)) + wave * ix.R * ix.RW;
        resolve_sets(ix, g, out, base, nq, M, mwaves, opt.rmode, sl);
        return;
    }
    const Transpose tp(lane);
    __syncthreads();  // (every wave has read T for its choice)
    transpose_blocks(g.T, blocks, wave, waves, lane, tp);
    __syncthreads();
    resolve_group<8>(ix, g.T, out, base, nq, wave, waves, lane, tp, sl);
}

// A small batch of term sets of any length: a workgroup of up to 16 waves per set,
// as k_query_seqs_team for reads, the waves sharing the set's terms. Bound by the
// chain of round trips. One launch: two would cost the smallest batches 4 us of 20.
template <int SEG, int G>
__global__ __launch_bounds__(1024) void k_sets_team(Index ix, const uint64_t *__restrict__ terms,
                                                    const uint64_t *__restrict__ offs, uint64_t *__restrict__ out,
                                                    QueryOpts opt, unsigned long long *invalid, int use_res) {
    extern __shared__ __align__(16) uint64_t smem64[];
    __shared__ unsigned long long issued;
    __shared__ uint32_t bad;
    const uint32_t lane = threadIdx.x & 63, wave = threadIdx.x >> 6, waves = blockDim.x >> 6;
    const uint32_t mw = ix.R * ix.RW, pitch = wave_lds(mw, ix.W, false, false).total;
    uint32_t *M0 = reinterpret_cast<uint32_t *>(smem64), *M = M0 + wave * pitch;
    uint64_t *res = use_res ? reinterpret_cast<uint64_t *>(M0 + waves * pitch) : nullptr;
    const uint64_t beg = offs[blockIdx.x], end = offs[blockIdx.x + 1], len = end > beg ? end - beg : 0;
    constexpr uint32_t kGrain = 64 / G;
    const uint64_t part = ((len + kGrain - 1) / kGrain + waves - 1) / waves * kGrain;  // terms per wave
    const uint32_t used = part ? (uint32_t)((len + part - 1) / part) : 0;            // waves that have any
    const uint64_t lo = min(len, wave * part), hi = min(len, lo + part);
    const bool ee = opt.early_exit != 0;
    uint64_t *o = out + (uint64_t)blockIdx.x * ix.W;
    if (threadIdx.x == 0) {
        issued = 0;
        bad = 0;
        if (len == 0) atomicAdd(opt.emptyq, 1ULL);
    }
    init_masks(ix, M, lane);
    __syncthreads();
    auto load = [&](uint64_t w) -> Window {
        Window wv;
        wv.valid = w + lane < hi;
        wv.canon = wv.valid ? terms[beg + w + lane] : 0;
        return wv;
    };
    uint64_t got = 0;
    bool odd = false;  // a value that is no 31-mer: the set answers no document
    bool alive = true;
    for (uint64_t w = lo; w < hi; w += 64) {
        Window wv = load(w);
        if (!ix.opaque) {
            odd |= (wv.canon >> 62) != 0;
            wv.canon = canonical(wv.canon & MASK62);
        }
        if (ee && !alive) continue;  // (the rest is looked through for such values)
        alive = probe_group<SEG, G, 0, 1>(ix, step_params(ix), wv, wv.valid, lane, M, (uint32_t)min<uint64_t>(64, hi - w));
        got += min<uint64_t>(64, hi - w);
        if (ee && !alive && ix.opaque) break;
    }
    if (odd) bad = 1;
    if (opt.probes && lane == 0 && got) atomicAdd(&issued, (unsigned long long)got);
    __syncthreads();
    uint32_t any = 0;  // the parts' AND in repetition 0
    for (uint32_t w = lane; w < ix.RW; w += 64) {
        uint32_t v = 0xFFFFFFFFu;
        for (uint32_t k = 0; k < used; k++) v &= M0[k * pitch + w];
        any |= v;
    }
    const bool live = !bad && (!ee || __ballot(any != 0) != 0);
    if (bad && threadIdx.x == 0) atomicAdd(invalid, 1ULL);
    if (live && ix.R > 1) {
        got = 0;
        for (uint64_t w = lo; w < hi; w += 64) {
            Window wv = load(w);
            if (!ix.opaque) wv.canon = canonical(wv.canon);
            const uint32_t nv = (uint32_t)min<uint64_t>(64, hi - w);
            alive = probe_group<SEG, G, 1, 4>(ix, step_params(ix), wv, wv.valid, lane, M, nv);
            got += nv * (min(ix.R, 5u) - 1);
            if ((int)ix.R > 5 && (alive || !ee)) {
                alive &= probe_group<SEG, G, 5, MAXR - 5>(ix, step_params(ix), wv, wv.valid, lane, M, nv);
                got += nv * (ix.R - 5);
            }
            if (ee && !alive) break;
        }
        if (opt.probes && lane == 0 && got) atomicAdd(&issued, (unsigned long long)got);
    }
    if (live) __syncthreads();
    if (opt.probes && threadIdx.x == 0 && issued) atomicAdd(opt.probes, issued * ix.eta);
    if (live) {
        for (uint32_t w = threadIdx.x; w < mw; w += blockDim.x) {
            uint32_t v = M0[w];
            for (uint32_t k = 1; k < used; k++) v &= M0[k * pitch + w];
            M0[w] = v;
        }
        __syncthreads();
    }
    if (!live || masks_some_rep_empty(ix, M0, lane)) {
        for (uint32_t w = threadIdx.x; w < ix.W; w += blockDim.x) o[w] = 0;
        return;
    }
    // Candidates where twice their steps (kSlotsAhead slots of 64 documents) are fewer
    // than the steps over all documents: sets of 5 words that a document holds have tens
    // to hundreds of positive cells, sets of 200 a few, and a step of candidates takes
    // about two (64 sets, 16 / 8 / 4 waves, candidates against all documents: Wiki-like,
    // 5 words 16.5 / 18.3 / 22.5 us against 12.8 / 13.4 / 17.0, 200 words 13.4 / 12.5 /
    // 14.1 against 15.0 / 15.7 / 21.1; K=101,000, 5 words 21 / 23 / 28 against 49 / 58 / 82).
    const WholeGroup who{wave, waves};
    const SetCells cells(ix, M0, lane);
    const uint64_t slots = (uint64_t)cells.total * (((ix.K + ix.B - 1) / ix.B + 63) / 64);
    if (opt.rmode == 2 || (opt.rmode == 0 && 2 * slots / kSlotsAhead + 1 < (ix.W + 7) / 8))
        (void)resolve_candidates(ix, M0, cells, res, o, lane, nullptr, who);
    else
        (void)resolve_dense(ix, M0, o, lane, nullptr, who);
}

// ---------------------------------------------------------------------------
// The general path, one resolve per term: for the candidate strategy when it
// is asked for, and for indexes whose T does not fit LDS.
// ---------------------------------------------------------------------------
template <int SEG, int G>
__global__ __launch_bounds__(256) void k_query_kmers(Index ix, const uint64_t *__restrict__ kmers, uint64_t n,
                                                     uint64_t *__restrict__ out, unsigned long long *invalid,
                                                     int rmode, int use_res) {
    constexpr int KPW = 64 / G;
    extern __shared__ uint64_t smem64[];
    const uint32_t lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const uint32_t mwords = ((KPW * ix.R * ix.RW) + 1) & ~1u;
    const uint32_t per_wave = mwords + (use_res ? 2 * ix.W : 0);
    uint32_t *M = reinterpret_cast<uint32_t *>(smem64) + wave * per_wave;
    uint64_t *res = use_res ? reinterpret_cast<uint64_t *>(M + mwords) : nullptr;

    const uint64_t base = ((uint64_t)blockIdx.x * (blockDim.x >> 6) + wave) * KPW;
    if (base >= n) return;
    const uint32_t g = lane / G, seg = lane % G;
    const uint64_t q = base + g;

    Seg<SEG> acc[MAXR];
    set_ones(acc);
    if (q < n) {
        const uint64_t x = kmers[q];
        if (!ix.opaque && (x >> 62)) {
            if (seg == 0) atomicAdd(invalid, 1ULL);
#pragma unroll
            for (int r = 0; r < MAXR; r++)
#pragma unroll
                for (int s = 0; s < SEG; s++) acc[r].w[s] = 0;
        } else {
            probe_and<SEG>(ix, ix.opaque ? x : canonical(x), seg, acc);
        }
    }
    // stage every term's masks; alive = no repetition mask is empty
    uint64_t alive = ~0ULL;
    const uint64_t gm = (G >= 64) ? ~0ULL : ((1ULL << G) - 1);
#pragma unroll
    for (int r = 0; r < MAXR; r++) {
        if (r < (int)ix.R) {
            uint32_t o = 0;
#pragma unroll
            for (int s = 0; s < SEG; s++) {
                M[(g * ix.R + r) * ix.RW + seg * SEG + s] = acc[r].w[s];
                o |= acc[r].w[s];
            }
            const uint64_t bal = __ballot(o != 0);
            uint64_t a = 0;
#pragma unroll
            for (int t = 0; t < KPW; t++) a |= (uint64_t)(((bal >> (t * G)) & gm) != 0) << t;
            alive &= a;
        }
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    for (int t = 0; t < KPW; t++) {
        const uint64_t row = base + t;
        if (row >= n) break;
        uint64_t *o = out + row * ix.W;
        if (!((alive >> t) & 1)) write_zeros(o, ix.W, lane);
        else resolve(ix, M + t * ix.R * ix.RW, res, o, lane, rmode);
    }
}

// One term set by one wave (M: its masks in LDS; res: LDS bitset of W words, or
// null), 64 terms per step; repetition 0 over every term first, then the other
// repetitions (Section 3.3.1 order).
template <int SEG, int G>
__device__ __forceinline__ void answer_set(const Index &ix, const uint64_t *__restrict__ terms,
                                           const uint64_t *__restrict__ offs, uint64_t q, uint64_t *__restrict__ out,
                                           const QueryOpts &opt, uint32_t *M, uint64_t *res,
                                           unsigned long long *invalid, uint32_t lane) {
    const uint64_t beg = offs[q];
    uint64_t end = offs[q + 1];
    if (end < beg) end = beg;
    const uint64_t len = end - beg;
    uint64_t *o = out + q * ix.W;
    if (len == 0 && lane == 0) atomicAdd(opt.emptyq, 1ULL);

    // a k-mer index takes 31-mer codes only: a set holding another value
    // answers no document
    bool bad = false;
    if (!ix.opaque)
        for (uint64_t w = 0; w < len && !bad; w += 64)
            bad = __ballot(w + lane < len && (terms[beg + w + lane] >> 62)) != 0;
    if (bad) {
        if (lane == 0) atomicAdd(invalid, 1ULL);
        write_zeros(o, ix.W, lane);
        return;
    }
    init_masks(ix, M, lane);
    uint64_t issued = 0;
    bool ended = false;
    for (int pass = 0; pass < 2 && !ended; pass++) {
        if (pass == 1 && ix.R == 1) break;
        for (uint64_t w = 0; w < len; w += 64) {
            const bool valid = w + lane < len;
            const uint64_t x = valid ? terms[beg + w + lane] : 0;
            Window wv;
            wv.canon = ix.opaque ? x : canonical(x);
            wv.valid = valid;
            const uint32_t nv = (uint32_t)min<uint64_t>(64, len - w);
            bool alive;
            if (pass == 0) {
                alive = probe_group<SEG, G, 0, 1>(ix, step_params(ix), wv, valid, lane, M, nv);
                issued += nv;
            } else {
                alive = probe_group<SEG, G, 1, 4>(ix, step_params(ix), wv, valid, lane, M, nv);
                issued += nv * (min(ix.R, 5u) - 1);
                if ((int)ix.R > 5 && (alive || !opt.early_exit)) {
                    alive &= probe_group<SEG, G, 5, MAXR - 5>(ix, step_params(ix), wv, valid, lane, M, nv);
                    issued += nv * (ix.R - 5);
                }
            }
            if (opt.early_exit && !alive) {
                ended = true;
                break;
            }
        }
    }
    if (opt.probes && lane == 0 && issued) atomicAdd(opt.probes, (unsigned long long)(issued * ix.eta));
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    if (masks_some_rep_empty(ix, M, lane)) {
        write_zeros(o, ix.W, lane);
        return;
    }
    resolve(ix, M, res, o, lane, opt.rmode);
}

// A wave takes `take` consecutive sets. With tq (a multiple of take), only the sets
// of groups of tq that k_sets_group leaves (short_sets): the grid is then one of
// 64 to 128 waves a compute unit, so that a batch without such groups costs a launch
// and one look at the offsets (a wave a set: 14 us for 100,000 sets).
template <int SEG, int G>
__global__ __launch_bounds__(256) void k_sets_long(Index ix, const uint64_t *__restrict__ terms,
                                                   const uint64_t *__restrict__ offs, uint64_t n,
                                                   uint64_t *__restrict__ out, QueryOpts opt, int use_res,
                                                   unsigned long long *invalid, uint32_t tq, uint32_t take) {
    extern __shared__ __align__(16) uint64_t smem64[];
    const uint32_t lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const WaveLds L = wave_lds(ix.R * ix.RW, ix.W, use_res != 0, false);
    uint32_t *M = reinterpret_cast<uint32_t *>(smem64) + wave * L.total;
    uint64_t *res = use_res ? reinterpret_cast<uint64_t *>(M + L.res) : nullptr;

    const uint64_t q0 = ((uint64_t)blockIdx.x * (blockDim.x >> 6) + wave) * take;
    if (q0 >= n) return;
    if (tq) {
        const uint64_t base = q0 - q0 % tq;
        const uint32_t nq = (uint32_t)min<uint64_t>(tq, n - base);
        uint64_t l = 0;
        if (lane < nq) {
            const uint64_t b = offs[base + lane], e = offs[base + lane + 1];
            l = e > b ? e - b : 0;
        }
        if (short_sets(l, nq)) return;
    }
    for (uint64_t q = q0; q < min(n, q0 + take); q++) {
        answer_set<SEG, G>(ix, terms, offs, q, out, opt, M, res, invalid, lane);
        OneWave().sync();
    }
}

static constexpr uint32_t kMaxLds = 64 * 1024;  // of the general path

static TermIndex term_index(const rambo_s *h) {
    TermIndex ix;
    static_cast<Index &>(ix) = make_index(h);
    ix.docslot = h->d_docslot;
    return ix;
}

// Launch shape of the group kernels: waves of a workgroup and slices of the
// documents, for groups of tq queries, chunks of `chunk` result words and words of
// `word` bytes in T.
struct GroupShape {
    uint32_t lds, waves, groups, slices;
};

// Whether a batch takes the group kernels: the candidate strategy has its own
// path, and T must fit the LDS of a workgroup (R * B up to about 19,600 cells
// in 160 KB).
static bool group_resolve(const rambo_s *h) {
    return h->resolve != RAMBO_RESOLVE_CANDIDATE && (uint64_t)t_words(h->R, h->B) * 8 + 64 <= h->lds_max;
}

// T larger than half the LDS leaves one workgroup a compute unit, which then
// takes the unit's 16 waves; smaller ones share it. Few groups are cut into
// slices of the documents until the chip has a workgroup of its own for each
// place, down to one chunk of result words a wave.
static GroupShape group_shape(const rambo_s *h, uint64_t n, uint32_t tq, uint32_t chunk, uint32_t word) {
    GroupShape g;
    g.lds = t_words(h->R, h->B) * word;
    g.waves = g.lds > h->lds_max / 2 ? 16 : g.lds > h->lds_max / 4 ? 8 : 4;
    const uint64_t groups = (n + tq - 1) / tq, places = (uint64_t)h->n_cu * (16 / g.waves);
    const uint64_t chunks = (h->W + chunk - 1) / chunk, most = (chunks + g.waves - 1) / g.waves;
    g.groups = (uint32_t)std::min<uint64_t>(groups, 0x80000000ull);
    g.slices = (uint32_t)std::max<uint64_t>(1, std::min<uint64_t>({places / std::max<uint64_t>(1, groups), most, 65535}));
    return g;
}

static int general_query_kmers(rambo_s *h, const uint64_t *kmers, uint64_t n, uint64_t *out, hipStream_t s) {
    const Index ix = make_index(h);
    const int seg = default_seg(h->RW), G = (int)h->RW / seg;
    const int KPW = 64 / G, WPB = 4;
    const uint32_t mwords = ((KPW * h->R * h->RW) + 1) & ~1u;
    int use_res = 1;
    size_t lds = (size_t)WPB * (mwords + 2 * h->W) * 4;
    if (lds > kMaxLds) {
        use_res = 0;
        lds = (size_t)WPB * mwords * 4;
    }
    const uint64_t waves = (n + KPW - 1) / KPW;
    const uint64_t blocks = (waves + WPB - 1) / WPB;
    if (blocks > 0x7FFFFFFFULL) return fail(RAMBO_EINVAL, "rambo_query_kmers: batch too large");
#define RAMBO_SPLIT_BODY_                                                                                  \
    hipLaunchKernelGGL((k_query_kmers<SEG, G>), dim3((unsigned)blocks), dim3(64 * WPB), lds, s, ix, kmers, n, out, \
                       h->d_invalid, h->resolve, use_res)
    RAMBO_DISPATCH_DEFAULT_SPLIT(seg, G)
#undef RAMBO_SPLIT_BODY_
    HIP_CHECK(hipGetLastError());
    return RAMBO_OK;
}

int launch_query_kmers(rambo_s *h, const uint64_t *kmers, uint64_t n, uint64_t *out, hipStream_t s) {
    if (!group_resolve(h)) return general_query_kmers(h, kmers, n, out, s);
    const TermIndex ix = term_index(h);
    if (h->RW <= 4) {
        // one wave per 64 terms; small batches as single waves, cut into
        // slices of the documents, up to eight waves a compute unit
        const uint64_t groups = (n + 63) / 64, fill = (uint64_t)h->n_cu * 8, chunks = (h->W + 15) / 16;
        const uint32_t wpb = groups >= fill ? 4 : 1;
        const uint64_t blocks = (groups + wpb - 1) / wpb;
        if (blocks > 0x7FFFFFFFULL) return fail(RAMBO_EINVAL, "rambo_query_kmers: batch too large");
        const uint64_t slices = std::max<uint64_t>(1, std::min<uint64_t>({fill / groups, chunks, 65535}));
        const dim3 grid((unsigned)blocks, (unsigned)slices), block(64 * wpb);
        const size_t lds = (size_t)wpb * t_words(h->R, h->B) * 8;
        if (h->RW == 1) hipLaunchKernelGGL(k_terms_lane<1>, grid, block, lds, s, ix, kmers, n, out, h->d_invalid);
        else if (h->RW == 2) hipLaunchKernelGGL(k_terms_lane<2>, grid, block, lds, s, ix, kmers, n, out, h->d_invalid);
        else hipLaunchKernelGGL(k_terms_lane<4>, grid, block, lds, s, ix, kmers, n, out, h->d_invalid);
        HIP_CHECK(hipGetLastError());
        return RAMBO_OK;
    }
    // where a T of 64 terms would take more than half the LDS, and so leave one
    // workgroup a compute unit, groups of 32 (0.64 -> 0.55 ms, see the kernel);
    // elsewhere they would only read the documents' cells twice as often
    const bool half = t_words(h->R, h->B) * 8 > h->lds_max / 2;
    const uint32_t tq = half ? 32 : 64;
    // (a launch has fewer than 2^32 threads: 4 to 16 of them a term)
    const uint64_t most = 0xFFFFFFFFull / (64 * 16) * tq;
    for (uint64_t at = 0; at < n; at += most) {
        const uint64_t m = std::min(n - at, most);
        const GroupShape g = group_shape(h, m, tq, 16, half ? 4 : 8);
        const dim3 grid(g.groups, g.slices), block(64 * g.waves);
        if (half)
            hipLaunchKernelGGL(k_terms_group<uint32_t>, grid, block, g.lds, s, ix, kmers + at, m, out + at * h->W,
                               h->d_invalid, h->log2RW - 2);
        else
            hipLaunchKernelGGL(k_terms_group<uint64_t>, grid, block, g.lds, s, ix, kmers + at, m, out + at * h->W,
                               h->d_invalid, h->log2RW - 2);
        HIP_CHECK(hipGetLastError());
    }
    return RAMBO_OK;
}

// A wave a set: all sets, or those of long groups of tq.
static int launch_sets_long(rambo_s *h, const uint64_t *terms, const uint64_t *offs, uint64_t n, uint64_t *out,
                            hipStream_t s, const QueryOpts &opt, uint32_t tq) {
    const Index ix = make_index(h);
    const int seg = default_seg(h->RW), G = (int)h->RW / seg;
    const int WPB = 4;
    int use_res = 1;
    size_t lds = (size_t)WPB * wave_lds(h->R * h->RW, h->W, true, false).total * 4;
    if (lds > kMaxLds) {
        use_res = 0;
        lds = (size_t)WPB * wave_lds(h->R * h->RW, h->W, false, false).total * 4;
    }
    uint32_t take = 1;
    while (2 * take <= tq && n > (uint64_t)take * h->n_cu * 128) take *= 2;
    const uint64_t blocks = (n + (uint64_t)WPB * take - 1) / ((uint64_t)WPB * take);
    if (blocks > 0x7FFFFFFFULL) return fail(RAMBO_EINVAL, "rambo_query_term_sets: batch too large");
#define RAMBO_SPLIT_BODY_                                                                                  \
    hipLaunchKernelGGL((k_sets_long<SEG, G>), dim3((unsigned)blocks), dim3(64 * WPB), lds, s, ix, terms, offs, n, out, \
                       opt, use_res, h->d_invalid, tq, take)
    RAMBO_DISPATCH_DEFAULT_SPLIT(seg, G)
#undef RAMBO_SPLIT_BODY_
    HIP_CHECK(hipGetLastError());
    return RAMBO_OK;
}

// A workgroup a set up to four a compute unit (3,000 sets of 64 words, Wiki-like: 54
// us, 38 with a wave each; 1,000 30 and 32), then groups of sets, short and long
// ones; a wave a set for the candidate strategy and for indexes whose T does not fit
// LDS.
int launch_query_termsets(rambo_s *h, const uint64_t *terms, const uint64_t *offs, uint64_t n, uint64_t *out,
                          hipStream_t s) {
    const QueryOpts opt{h->resolve, h->early_exit, h->probe_counter, SCHED_SWEEP, nullptr, h->d_emptyq};
    const uint32_t team = n <= 4 * (uint64_t)h->n_cu ? team_waves(h, n) : 1;
    if (team > 1) {
        const Index ix = make_index(h);
        const int seg = default_seg(h->RW), G = (int)h->RW / seg, use_res = seq_lds_result(h->W) ? 1 : 0;
        const size_t lds = team_lds(h, team, use_res != 0);
#define RAMBO_SPLIT_BODY_                                                                                  \
    hipLaunchKernelGGL((k_sets_team<SEG, G>), dim3((unsigned)n), dim3(64 * team), lds, s, ix, terms, offs, out, opt,   \
                       h->d_invalid, use_res)
        RAMBO_DISPATCH_DEFAULT_SPLIT(seg, G)
#undef RAMBO_SPLIT_BODY_
        HIP_CHECK(hipGetLastError());
        return RAMBO_OK;
    }
    // a wave a set where the resolve is short (W <= 16) and the chip not yet full: the
    // second launch costs more than the groups save (5,000 sets of 4 terms at K=100
    // 27 us, 33 in groups; 30,000 65 and 44)
    const bool few = h->W <= 16 && n <= 32 * (uint64_t)h->n_cu;
    // T and the masks of four waves at least
    const size_t tbytes = (size_t)t_words(h->R, h->B) * 8, mbytes = (size_t)h->R * h->RW * 4;
    if (few || !group_resolve(h) || tbytes + 4 * mbytes + 64 > h->lds_max)
        return launch_sets_long(h, terms, offs, n, out, s, opt, 0);
    const TermIndex ix = term_index(h);
    // sets of a group: 64, or fewer (to 4) where that would leave half of the
    // chip's places for workgroups without one (100,000 sets: 0.14 ms in groups of
    // 64, 0.23 in groups of 16, whose transposes are as many each)
    uint32_t tq = 64;
    const uint64_t places = (uint64_t)h->n_cu * (16 / group_shape(h, n, tq, 8, 8).waves);
    while (tq > 4 && n <= places * tq / 2) tq >>= 1;
    const GroupShape g = group_shape(h, n, tq, 8, 8);
    if (g.groups > 0x7FFFFFFFu) return fail(RAMBO_EINVAL, "rambo_query_term_sets: batch too large");
    const uint32_t mwaves = (uint32_t)std::min<size_t>(g.waves, (h->lds_max - 64 - tbytes) / mbytes);
    const size_t lds = tbytes + mwaves * mbytes;
    const dim3 grid(g.groups, g.slices), block(64 * g.waves);
    if (h->RW == 1)
        hipLaunchKernelGGL(k_sets_group<1>, grid, block, lds, s, ix, terms, offs, n, out, opt, h->d_invalid, 0u, tq, mwaves);
    else if (h->RW == 2)
        hipLaunchKernelGGL(k_sets_group<2>, grid, block, lds, s, ix, terms, offs, n, out, opt, h->d_invalid, 0u, tq, mwaves);
    else
        hipLaunchKernelGGL(k_sets_group<4>, grid, block, lds, s, ix, terms, offs, n, out, opt, h->d_invalid,
                           h->log2RW - 2, tq, mwaves);
    HIP_CHECK(hipGetLastError());
    return launch_sets_long(h, terms, offs, n, out, s, opt, tq);
}

}  // namespace rambo
