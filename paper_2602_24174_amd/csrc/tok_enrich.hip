// Counting core of the paper's tokenizer enrichment ("Enriching the Tokenizer": merge reward
// f_merge(t^n) = freq(t^n) (n - 1) and the loop of the algorithm "Tokenizer Enrichment"), without the
// prefix-collision filter, which needs token strings: every step counts the n-grams (2 <= n <= n_max) of the corpus
// as currently tokenised with the table builder's counting stage, picks the n-gram with the largest reward
// (ties: shorter, then smallest token tuple), gives it the next free token id and re-tokenises the corpus on the
// device (left to right, without overlap, inside each output).
//
// What bounds a merge on a small corpus is its launches and whoever waits for them, so the steps of a merge follow each other
// without the host: what one finds out (the n-gram, the new length, that nothing is left to merge) the next ones read from
// device memory, and the host looks at it once per kBatch merges.  1.0 M tokens, eight merges, orders 2 to 4: 1.1 ms (4.4
// with counting tables in memory, some 35 launches a merge and two looks from the host).
#include <algorithm>
#include <string.h>
#include <vector>

#include "tasc_internal.h"

namespace {
constexpr int kThreads = 256;
constexpr int kItems = 4;                            // positions of a thread
constexpr int kBlock = kThreads * kItems;            // 1024
constexpr int kBatch = 16;
constexpr size_t kMostRecords = (size_t)2 << 30;

struct Merge {           // one line of the result, as the caller's arrays have it
    int32_t row[1 + TASC_MAX_ORDER];
    u32 freq;
};
struct State {
    u32 merges, done;    // merges so far; 1: nothing left to merge: every later step does nothing
    u32 bad;             // a token outside the vocabulary
    u32 n, overlaps;     // the running merge: its n-gram, and whether two occurrences of it can overlap
    int32_t t[TASC_MAX_ORDER], new_id;
};

// st->bad = 1 if a token lies outside [0, vocab)
__global__ __launch_bounds__(kThreads) void k_check_tokens(const int32_t* __restrict__ tok, u64 T, int vocab, State* st) {
    bool bad = false;
    for (u64 i = (u64)blockIdx.x * kThreads + threadIdx.x; i < T; i += (u64)gridDim.x * kThreads) bad = bad || tok[i] < 0 || tok[i] >= vocab;
    if (bad) st->bad = 1;
}

// the best of the partitions' candidates becomes merge number st->merges
constexpr int kPickThreads = 1024;
__global__ __launch_bounds__(kPickThreads) void k_pick(const TascGram* __restrict__ cands, u32 count, int bits, int vocab, State* st, Merge* merges) {
    if (st->done) return;
    TascGram best{0, 0, 0, 0};
    for (u32 i = threadIdx.x; i < count; i += kPickThreads)
        if (tasc_gram_before(cands[i], best, bits)) best = cands[i];
    __shared__ TascGram s_c[kPickThreads];
    s_c[threadIdx.x] = best;
    __syncthreads();
    for (int w = kPickThreads / 2; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w && tasc_gram_before(s_c[threadIdx.x + w], s_c[threadIdx.x], bits)) s_c[threadIdx.x] = s_c[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x != 0) return;
    best = s_c[0];
    if (best.count == 0) {
        st->done = 1;
        return;
    }
    const u32 m = st->merges;
    Merge out;
    out.freq = best.count;
    out.row[0] = (int32_t)best.n;
    for (int j = 0; j < TASC_MAX_ORDER; ++j) {
        const bool in = j < (int)best.n;
        st->t[j] = in ? (int32_t)tasc_key_get(best.lo, best.hi, j, bits) : 0;
        out.row[1 + j] = in ? st->t[j] : -1;
    }
    merges[m] = out;
    bool overlaps = false;
    for (u32 s = 1; s < best.n; ++s) {                       // shifted by s, the n-gram agrees with itself
        bool same = true;
        for (u32 j = 0; j + s < best.n; ++j) same = same && out.row[1 + j] == out.row[1 + j + s];
        overlaps = overlaps || same;
    }
    st->n = best.n;
    st->overlaps = overlaps;
    st->new_id = vocab + (int32_t)m;
    st->merges = m + 1;
}

struct Gram {            // the running merge, in registers
    u32 n, overlaps, merges;
    int32_t t[TASC_MAX_ORDER], new_id;
};
__device__ __forceinline__ Gram running(const State* __restrict__ st) {
    Gram g{st->n, st->overlaps, st->merges, {}, st->new_id};
#pragma unroll
    for (int j = 0; j < TASC_MAX_ORDER; ++j) g.t[j] = st->t[j];
    return g;
}
// the n-gram starts at i and lies inside one output; tok[0] is position i's token
__device__ __forceinline__ bool matches(const int32_t* tok, const uint8_t* __restrict__ last, u64 T, u64 i, const Gram& g) {
    if (tok[0] != g.t[0] || i + g.n > T || last[i]) return false;
    bool ok = true;
#pragma unroll
    for (int j = 1; j < TASC_MAX_ORDER; ++j)
        if (j < (int)g.n) ok = ok && tok[j] == g.t[j] && (j + 1 == (int)g.n || !last[i + j]);
    return ok;
}

// Left-to-right choice among occurrences that can overlap (the others are all taken, and found where they are needed): sel[i] =
// number of the merge.  An occurrence with none in the n - 1 positions before it ("head") is always taken; from it, one lane
// walks the run of occurrences that overlap each other, taking the first at or after the end of the last taken one, and stops when
// that one is a head itself (its own lane takes it) or lies beyond the reach of an overlap.  A walk is a chain of dependent loads, and
// a long run of one token is one walk: after kLaneSteps steps the wave takes it over, 64 positions at a time, and the steps among them
// are a few instructions (200,000 equal tokens, four merges of two: 176 ms with the lane alone; 61 with a byte per
// position to read instead of the tokens; 16 so).  The walk ends at the latest at the end of the corpus.
constexpr unsigned kSelectBlocks = 1024;
constexpr int kLaneSteps = 8;
__global__ __launch_bounds__(kThreads) void k_select(const int32_t* __restrict__ tok, const uint8_t* __restrict__ last, const u64* __restrict__ len,
                                                     const State* __restrict__ st, u32* sel) {
    if (st->done || !st->overlaps) return;
    const u64 T = *len;
    const Gram g = running(st);
    const int n = (int)g.n, lane = threadIdx.x & 63;
    auto is_head = [&](u64 p) {
        for (int j = 1; j < n; ++j)
            if (p >= (u64)j && matches(tok + (p - j), last, T, p - j, g)) return false;
        return true;
    };
    // bit l: an occurrence starts at p + l
    auto starts = [&](u64 p) {
        const u64 i = p + lane;
        bool ok = i + n <= T;
        const u64 at = ok ? i : 0;                           // (all of a lane's loads at once)
#pragma unroll
        for (int j = 0; j < TASC_MAX_ORDER; ++j)
            if (j < n) {
                const int32_t t = tok[at + j];
                const uint8_t e = last[at + j];
                ok = ok & (t == g.t[j]) & (j + 1 == n || !e);
            }
        return __ballot(ok);
    };
    for (u64 i0 = (u64)blockIdx.x * kThreads + threadIdx.x - lane; i0 < T; i0 += (u64)gridDim.x * kThreads) {
        const u64 i = i0 + lane;
        u64 cur = i;
        bool walking = i < T && matches(tok + i, last, T, i, g) && is_head(i);
        for (int s = 0; walking && s < kLaneSteps; ++s) {
            sel[cur] = st->merges;
            u64 next = T;
            for (u64 p = cur + n; p < cur + 2 * (u64)n - 1 && p < T; ++p)
                if (matches(tok + p, last, T, p, g)) { next = p; break; }
            walking = next < T && !is_head(next);
            cur = next;
        }
        // (the last step's `next` of a lane that is still walking is an occurrence that has to be taken)
        for (u64 todo = __ballot(walking); todo != 0; todo &= todo - 1) {
            u64 at = __shfl(cur, __ffsll(todo) - 1);         // taken; the next one lies n to 2 n - 2 positions on
            if (lane == 0) sel[at] = g.merges;
            for (bool on = true; on;) {
                const u64 base = at + 1, here = starts(base);
                u64 taken = 0;
                int c = -1;                                  // the last taken one, from base
                while (c + 2 * n - 2 < 64) {
                    const u64 reach = ((here >> (c + n)) & ((1ull << (n - 1)) - 1)) << (c + n);
                    const int next = __ffsll(reach) - 1;
                    // none, or a head: no occurrence between the last taken one and it
                    if (next < 0 || (here & ((1ull << next) - 1) & (~0ull << (next - n + 1))) == 0) { on = false; break; }
                    taken |= 1ull << next;
                    c = next;
                }
                if ((taken >> lane) & 1) sel[base + lane] = g.merges;
                at = base + c;
            }
        }
    }
}

// What a block of kBlock positions does with the merge: its tokens, 8 more on either side, come to LDS, and from them (or from the
// choice made above) where occurrences start.  keep: of the kItems positions of a thread, those that no taken
// occurrence swallows; starts: those where one begins.
struct BlockTokens {
    int32_t tok[kBlock + 16];
    __attribute__((aligned(16))) uint8_t start[kBlock + 16];
};
__device__ inline void block_keep(BlockTokens& s, const int32_t* __restrict__ tok, const uint8_t* __restrict__ last, const u32* __restrict__ sel,
                                  u64 T, const Gram& g, u32& keep, u32& starts) {
    const int64_t base = (int64_t)blockIdx.x * kBlock - 8;
    for (int q = threadIdx.x; q < kBlock + 16; q += kThreads) s.tok[q] = base + q >= 0 && base + q < (int64_t)T ? tok[base + q] : -1;
    __syncthreads();
    for (int q = threadIdx.x; q < kBlock + 8; q += kThreads) {
        const int64_t p = base + q;
        s.start[q] = p >= 0 && p < (int64_t)T && (g.overlaps ? sel[p] == g.merges : matches(s.tok + q, last, T, (u64)p, g)) ? 1 : 0;
    }
    __syncthreads();
    u32 f = 0;                                               // bit 8 + e: an occurrence starts at the thread's position e
    const uint8_t* at = s.start + kItems * threadIdx.x;
#pragma unroll
    for (int q = 0; q < 8 + kItems; ++q) f |= (u32)(at[q] & 1) << q;
    u32 gone = 0;
    for (u32 j = 1; j < g.n; ++j) gone |= f << j;
    const int64_t left = (int64_t)T - (base + 8) - kItems * (int64_t)threadIdx.x;
    const u32 mine = left >= kItems ? (1u << kItems) - 1 : left > 0 ? (1u << left) - 1 : 0;
    starts = (f >> 8) & mine;
    keep = ~(gone >> 8) & mine;
}

__device__ inline u32 block_scan(u32 v, u32* s_wave, u32* total) {      // exclusive
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    u32 at = v;
    for (int o = 1; o < 64; o <<= 1) {
        const u32 u = __shfl_up(at, o);
        if (lane >= o) at += u;
    }
    if (lane == 63) s_wave[wave] = at;
    __syncthreads();
    u32 before = 0, all = 0;
    for (int w = 0; w < kThreads / 64; ++w) {
        if (w < wave) before += s_wave[w];
        all += s_wave[w];
    }
    __syncthreads();
    *total = all;
    return before + at - v;
}

// records that stay in the blocks before this one, from the blocks' sums, or their scan where there are many
constexpr u32 kScanFrom = 4096;
__device__ __forceinline__ u32 blocks_before(const u32* __restrict__ bsum, u32* s_wave) {
    if (gridDim.x > kScanFrom) return bsum[blockIdx.x];
    u32 n = 0, all;
#pragma unroll 4
    for (u32 b = threadIdx.x; b < blockIdx.x; b += kThreads) n += bsum[b];
    block_scan(n, s_wave, &all);
    return all;
}
__global__ __launch_bounds__(kThreads) void k_scan(u32* bsum, u32 n) {      // in place, exclusive, one workgroup
    __shared__ u32 s_wave[kThreads / 64];
    u32 carry = 0;
    for (u32 b0 = 0; b0 < n; b0 += kThreads * 4) {
        u32 v[4], own = 0, all;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const u32 b = b0 + threadIdx.x * 4 + u;
            v[u] = b < n ? bsum[b] : 0;
            own += v[u];
        }
        u32 at = carry + block_scan(own, s_wave, &all);
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const u32 b = b0 + threadIdx.x * 4 + u;
            if (b < n) bsum[b] = at;
            at += v[u];
        }
        carry += all;
    }
}

__global__ __launch_bounds__(kThreads) void k_sums(const int32_t* __restrict__ tok, const uint8_t* __restrict__ last, const u32* __restrict__ sel,
                                                   const u64* __restrict__ len, const State* __restrict__ st, u32* bsum) {
    __shared__ BlockTokens s;
    __shared__ u32 s_wave[kThreads / 64];
    if (st->done) return;
    u32 keep, starts, sum;
    block_keep(s, tok, last, sel, len[0], running(st), keep, starts);
    block_scan(__popc(keep), s_wave, &sum);
    if (threadIdx.x == 0) bsum[blockIdx.x] = sum;
}
// len[0] = the corpus' length before the merge, len[1] after it
__global__ __launch_bounds__(kThreads) void k_apply(const int32_t* __restrict__ tok, const uint8_t* __restrict__ last, const u32* __restrict__ sel,
                                                    u64* len, const State* __restrict__ st, const u32* __restrict__ bsum,
                                                    int32_t* __restrict__ out, uint8_t* __restrict__ last_out) {
    __shared__ BlockTokens s;
    __shared__ u32 s_wave[kThreads / 64];
    if (st->done) return;
    const Gram g = running(st);
    u32 keep, starts, sum;
    block_keep(s, tok, last, sel, len[0], g, keep, starts);
    const u32 base = blocks_before(bsum, s_wave);
    u32 to = base + block_scan(__popc(keep), s_wave, &sum);
    if (blockIdx.x == gridDim.x - 1 && threadIdx.x == 0) len[1] = base + sum;
    const u64 first = (u64)blockIdx.x * kBlock + kItems * threadIdx.x;
    for (u32 k = keep; k != 0; k &= k - 1, ++to) {
        const int e = __ffs((int)k) - 1;
        const bool merged = (starts >> e) & 1;
        out[to] = merged ? g.new_id : s.tok[8 + kItems * threadIdx.x + e];
        last_out[to] = last[first + e + (merged ? g.n - 1 : 0)];
    }
}

// where the outputs end, in order
__device__ __forceinline__ u32 ends_here(const uint8_t* __restrict__ last, u64 T) {
    const u64 first = (u64)blockIdx.x * kBlock + kItems * threadIdx.x;
    u32 f = 0;
#pragma unroll
    for (int e = 0; e < kItems; ++e) f |= first + e < T && last[first + e] ? 1u << e : 0;
    return f;
}
__global__ __launch_bounds__(kThreads) void k_end_sums(const uint8_t* __restrict__ last, u64 T, u32* bsum) {
    __shared__ u32 s_wave[kThreads / 64];
    u32 sum;
    block_scan(__popc(ends_here(last, T)), s_wave, &sum);
    if (threadIdx.x == 0) bsum[blockIdx.x] = sum;
}
__global__ __launch_bounds__(kThreads) void k_ends(const uint8_t* __restrict__ last, u64 T, const u32* __restrict__ bsum, u32* ends) {
    __shared__ u32 s_wave[kThreads / 64];
    u32 sum;
    const u32 here = ends_here(last, T);
    u32 to = blocks_before(bsum, s_wave) + block_scan(__popc(here), s_wave, &sum);
    for (u32 k = here; k != 0; k &= k - 1) ends[to++] = blockIdx.x * kBlock + kItems * threadIdx.x + __ffs((int)k);
}

struct Arena : TascScratch {
    size_t used = 0;
    size_t carve(size_t bytes) { const size_t at = used; used += (bytes + 255) / 256 * 256; return at; }
};
}  // namespace

#define TOK_TRY(expr) do { tasc_status _rc = (expr); if (_rc != TASC_OK) return _rc; } while (0)

extern "C" tasc_status tasc_tok_enrich(const int32_t* tokens, const int64_t* doc_offsets, int64_t n_docs, int32_t vocab, int32_t n_max,
                                       int32_t budget, tasc_mem where, void* stream, int32_t* merges, int64_t* merge_freq,
                                       int64_t* corpus_len, int32_t* out_tokens, int64_t* out_offsets, int32_t* n_merges) {
    TASC_REQUIRE(doc_offsets && merges && merge_freq && corpus_len && out_offsets && n_merges, "tok_enrich: null argument");
    TASC_REQUIRE(n_docs >= 0 && vocab >= 1 && budget >= 0, "tok_enrich: n_docs %lld, vocab %d, budget %d", (long long)n_docs, vocab, budget);
    TASC_REQUIRE(n_max >= 2 && n_max <= TASC_MAX_ORDER, "tok_enrich: n_max %d outside [2, %d]", n_max, TASC_MAX_ORDER);
    TASC_REQUIRE(where == TASC_MEM_HOST || where == TASC_MEM_DEVICE, "tok_enrich: bad memory kind");
    TASC_REQUIRE((int64_t)vocab + budget <= 0x7FFFFFFF, "tok_enrich: vocab + budget overflows int32");
    const int32_t vocab_all = vocab + budget;               // one key width for every step
    int bits = 1;
    while ((1ll << bits) < vocab_all) ++bits;
    TASC_REQUIRE(n_max * bits <= 128, "tok_enrich: n_max %d x %d bits per token exceeds the 128-bit key", n_max, bits);
    TASC_REQUIRE(doc_offsets[0] == 0, "tok_enrich: doc_offsets[0] != 0");
    for (int64_t d = 0; d < n_docs; ++d)
        TASC_REQUIRE(doc_offsets[d + 1] >= doc_offsets[d], "tok_enrich: doc_offsets decrease at %lld", (long long)d);
    const u64 T0 = (u64)doc_offsets[n_docs];
    TASC_REQUIRE(T0 < 0xFFFFFFFFull, "tok_enrich: corpus of %llu tokens is too large", (unsigned long long)T0);
    TASC_REQUIRE(T0 == 0 || (tokens && out_tokens), "tok_enrich: null tokens");
    hipStream_t st = (hipStream_t)stream;

    // Nothing of the device is looked at before the first kBatch merges are on their way, a token outside the vocabulary included.
    u64 windows = 0;                                         // of order 2, the most of any
    std::vector<uint8_t> empty((size_t)n_docs);              // (out_offsets may be doc_offsets: looked at before anything is written)
    for (int64_t d = 0; d < n_docs; ++d) {
        const int64_t n = doc_offsets[d + 1] - doc_offsets[d];
        windows += (u64)std::max<int64_t>(0, n - 1);
        empty[d] = n == 0;
    }
    const int orders = n_max - 1;
    const TascCountPlan plan = tasc_count_plan(T0, windows, n_max * bits > 64, false);
    const bool run = budget > 0 && T0 > 0;
    Arena ar;
    const size_t at_state = ar.carve(sizeof(State)), at_len = ar.carve(((size_t)budget + 1) * sizeof(u64));
    const size_t at_sel = ar.carve(T0 * sizeof(u32)), zeroed = ar.used;
    const size_t at_tok[2] = {ar.carve(T0 * sizeof(int32_t)), ar.carve(T0 * sizeof(int32_t))}, at_last[2] = {ar.carve(T0), ar.carve(T0)};
    const size_t at_off = ar.carve(((size_t)n_docs + 1) * sizeof(int64_t)), at_ends = ar.carve((size_t)n_docs * sizeof(u32));
    const size_t at_bsum = ar.carve((T0 + kBlock - 1) / kBlock * sizeof(u32)), at_merges = ar.carve((size_t)budget * sizeof(Merge));
    const size_t at_best = ar.carve(run ? (size_t)orders * plan.parts * sizeof(TascGram) : 0);
    // As many orders counted together as kMostRecords hold records of (one order's are always held).  With few chunks an order alone
    // leaves the chip idle (ms, one at a time | together, n_max 6, eight merges: 1.0 M tokens 2.23 | 1.80, 4 M 5.33 | 4.66); many do not need
    // the others (16 M 19.0 | 18.3, 64 M 112.1 | 111.1).
    const size_t most = std::min(kMostRecords, (size_t)g_tasc_config.build_list_kib << 10);
    const int together = (int)std::clamp<size_t>(most / std::max<size_t>(1, plan.rec_bytes + plan.offs_bytes), 1, orders);
    const size_t at_rec = ar.carve(run ? together * plan.rec_bytes : 0), at_roff = ar.carve(run ? together * plan.offs_bytes : 0);
    const size_t at_deal = ar.carve(run ? plan.deal_bytes : 0);
    TOK_TRY(ar.get(ar.used));
    State* const state = (State*)(ar.p + at_state);
    u64* const len = (u64*)(ar.p + at_len);
    int32_t* const tok[2] = {(int32_t*)(ar.p + at_tok[0]), (int32_t*)(ar.p + at_tok[1])};
    uint8_t *const last[2] = {(uint8_t*)(ar.p + at_last[0]), (uint8_t*)(ar.p + at_last[1])};
    int64_t* const d_off = (int64_t*)(ar.p + at_off);
    u32 *const bsum = (u32*)(ar.p + at_bsum), *const sel = (u32*)(ar.p + at_sel), *const ends = (u32*)(ar.p + at_ends);
    Merge* const d_merges = (Merge*)(ar.p + at_merges);
    TascGram* const best = (TascGram*)(ar.p + at_best);
    const TascCountBufs bufs{(u64*)(ar.p + at_rec), (uint16_t*)(ar.p + at_roff), (u64*)(ar.p + at_deal)};

    TASC_HIP(hipMemsetAsync(ar.p, 0, zeroed, st));
    TASC_HIP(hipMemcpyAsync(len, &T0, sizeof T0, hipMemcpyHostToDevice, st));
    if (T0) {
        TASC_HIP(hipMemcpyAsync(tok[0], tokens, T0 * sizeof(int32_t), where == TASC_MEM_HOST ? hipMemcpyHostToDevice : hipMemcpyDeviceToDevice, st));
        TASC_HIP(hipMemcpyAsync(d_off, doc_offsets, (size_t)(n_docs + 1) * sizeof(int64_t), hipMemcpyHostToDevice, st));
        TOK_TRY(tasc_mark_ends(d_off, n_docs, T0, last[0], st));
    }
    if (run) {
        k_check_tokens<<<dim3(1024), dim3(kThreads), 0, st>>>(tok[0], T0, vocab_all, state);
        TASC_LAUNCH_CHECK();
    }
    State h;
    memset(&h, 0, sizeof h);
    std::vector<u64> lens((size_t)budget + 1, 0);
    lens[0] = T0;
    u64 T = T0;                                              // the corpus is no longer than this
    for (int done = 0; run && done < budget && !h.done; ) {
        const int end = std::min(budget, done + kBatch), begin = done;
        TascCountPlan p = plan;                              // (the records' strides are those of the whole corpus)
        p.chunks = (u32)((T + p.chunk - 1) / p.chunk);
        const dim3 grid1((unsigned)std::min<u64>((T + kThreads - 1) / kThreads, kSelectBlocks)), grid2((unsigned)((T + kBlock - 1) / kBlock));
        for (; done < end; ++done) {
            int32_t* const cur = tok[done & 1];
            const uint8_t* const cur_last = last[done & 1];
            for (int n0 = 2; n0 <= n_max; n0 += together) {
                const int here = std::min(together, n_max + 1 - n0);
                TOK_TRY(tasc_count_partition(p, cur, cur_last, T, len + done, n0, here, bits, bufs, nullptr, nullptr, st));
                TOK_TRY(tasc_count_best(p, len + done, n0, here, bits, bufs, best + (size_t)(n0 - 2) * p.parts, st));
            }
            k_pick<<<dim3(1), dim3(kPickThreads), 0, st>>>(best, (u32)orders * p.parts, bits, vocab, state, d_merges);
            k_select<<<grid1, dim3(kThreads), 0, st>>>(cur, cur_last, len + done, state, sel);
            k_sums<<<grid2, dim3(kThreads), 0, st>>>(cur, cur_last, sel, len + done, state, bsum);
            if (grid2.x > kScanFrom) k_scan<<<dim3(1), dim3(kThreads), 0, st>>>(bsum, grid2.x);
            k_apply<<<grid2, dim3(kThreads), 0, st>>>(cur, cur_last, sel, len + done, state, bsum, tok[(done + 1) & 1], last[(done + 1) & 1]);
            TASC_LAUNCH_CHECK();
        }
        TASC_HIP(hipMemcpyAsync(&h, state, sizeof h, hipMemcpyDeviceToHost, st));
        TASC_HIP(hipMemcpyAsync(&lens[begin + 1], len + begin + 1, (size_t)(end - begin) * sizeof(u64), hipMemcpyDeviceToHost, st));
        TASC_HIP(hipStreamSynchronize(st));
        TASC_REQUIRE(h.bad == 0, "tok_enrich: corpus holds a token outside [0, %d)", vocab_all);
        T = lens[h.merges];
    }
    const int n_done = (int)h.merges;
    T = lens[n_done];
    std::vector<Merge> rows(n_done);
    std::vector<u32> h_ends(n_docs);
    if (n_done) TASC_HIP(hipMemcpyAsync(rows.data(), d_merges, rows.size() * sizeof(Merge), hipMemcpyDeviceToHost, st));
    if (T) {
        const dim3 grid2((unsigned)((T + kBlock - 1) / kBlock));
        k_end_sums<<<grid2, dim3(kThreads), 0, st>>>(last[n_done & 1], T, bsum);
        if (grid2.x > kScanFrom) k_scan<<<dim3(1), dim3(kThreads), 0, st>>>(bsum, grid2.x);
        k_ends<<<grid2, dim3(kThreads), 0, st>>>(last[n_done & 1], T, bsum, ends);
        TASC_LAUNCH_CHECK();
        TASC_HIP(hipMemcpyAsync(h_ends.data(), ends, h_ends.size() * sizeof(u32), hipMemcpyDeviceToHost, st));
        TASC_HIP(hipMemcpyAsync(out_tokens, tok[n_done & 1], T * sizeof(int32_t), where == TASC_MEM_HOST ? hipMemcpyDeviceToHost : hipMemcpyDeviceToDevice, st));
    }
    TASC_HIP(hipStreamSynchronize(st));
    ar.keep();
    *n_merges = n_done;
    for (int i = 0; i < n_done; ++i) {
        memcpy(merges + (size_t)i * (1 + TASC_MAX_ORDER), rows[i].row, sizeof rows[i].row);
        merge_freq[i] = (int64_t)rows[i].freq;
    }
    for (int i = 0; i <= n_done; ++i) corpus_len[i] = (int64_t)lens[i];
    out_offsets[0] = 0;
    for (int64_t d = 0, e = 0; d < n_docs; ++d)              // (an output that had tokens keeps at least one)
        out_offsets[d + 1] = empty[d] ? out_offsets[d] : (int64_t)h_ends[e++];
    return TASC_OK;
}
