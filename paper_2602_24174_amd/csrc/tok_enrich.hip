// Counting core of the paper's tokenizer enrichment ("Enriching the Tokenizer": merge reward
// f_merge(t^n) = freq(t^n) (n - 1) and the loop of the algorithm "Tokenizer Enrichment"), without the
// prefix-collision filter, which needs token strings: every step finds the n-gram (2 <= n <= n_max) with the largest reward in the corpus
// as currently tokenised (ties: shorter, then smallest token tuple), gives it the next free token id and re-tokenises the corpus on the
// device (left to right, without overlap, inside each output).
//
// What bounds a merge on a small corpus is its launches and whoever waits for them, so the steps of a merge follow each other
// without the host: what one finds out (the n-gram, the new length, that nothing is left to merge) the next ones read from
// device memory, and the host looks at it once per kBatch merges.  And most n-grams cannot win, which a count of pairs by hash shows (the sieve,
// below): four launches a merge (five above kTellBlocks blocks), some 42 us at 1.0 M tokens, of chains of round trips.  ms, every n-gram of every merge
// counted | so, n_max 4, in turn: 1.0 M tokens of phrases, eight merges 0.92 | 0.48, 64 merges 6.25 | 4.1, 256 merges 22.3 | 19.1 (from some 50 on
// nearly all are counted in full); 20,000 tokens, eight merges 0.66 | 0.39, 2000 merges 148.5 | 149; 16 M tokens, eight merges 8.5 | 3.6.  Where every pair is as
// frequent as any other the sieve only costs, a tenth to a seventh of a call of eight merges, most of it the launches behind the one that gives up: 1.0 M
// random tokens 1.39 | 1.53, of forty kinds 1.02 | 1.19, one token alone 0.60 | 0.70; 64 merges of random tokens 10.0 | 10.5.
#include <algorithm>
#include <string.h>
#include <vector>

#include "tasc_internal.h"

namespace {
constexpr int kThreads = 1024;
constexpr int kItems = 4;                            // positions of a thread
constexpr int kBlock = kThreads * kItems;            // 4096
constexpr int kFirst = 8, kBatch = 16;              // merges that the host launches before it looks: at first, and at most
constexpr size_t kMostRecords = (size_t)2 << 30;

struct Merge {           // one line of the result, as the caller's arrays have it
    int32_t row[1 + TASC_MAX_ORDER];
    u32 freq;
};
// Workgroups of one launch start at different times, and so do the waves of a workgroup: a field that a kernel returns early on is written in
// that launch by no one, or only after all have read it (k_gather's last workgroup).
struct State {
    u32 merges, done;    // merges so far; 1: nothing left to merge: every later step does nothing
    u32 stuck;           // 1: the sieve cannot tell the next merge (see below): every later step does nothing until the host has seen it
    u32 bad, foreign;    // a token outside the vocabulary, the new ids included: nothing is done; one of the new ids: the sieve is not used
    u32 gave_up;         // k_sift's: its lists or tables are full, or most buckets pass; k_gather makes `stuck` of it
    u32 undo, late;      // k_apply's: the last merge was the wrong one; it was left unfinished.  As `stuck` for later steps
    u64 length;          // of the corpus after the last merge, the wrong one included
    u32 arrived;         // workgroups of k_gather that are done with the running merge
    u32 top, taken;      // the fullest bucket of pairs; 1: there is a running merge
    u64 reward, want;    // of the last merge; what the next one is looked for from: a guess, or (retry) the best n-gram that the guess found
    u32 retry;
    u32 n, overlaps;     // the running merge: its n-gram, its windows, and whether two of them can overlap
    u32 freq, seen;      // (seen: counted again, where they can overlap)
    int32_t t[TASC_MAX_ORDER], new_id;
};

__device__ __forceinline__ bool idle(const State* st) { return (st->done | st->stuck | st->bad | st->undo | st->late) != 0; }
__device__ __forceinline__ bool no_merge(const State* st) { return !st->taken; }      // (after an idle k_sift or k_pick, too)

// st->bad = 1 if a token lies outside [0, vocab_all), st->foreign = 1 if outside [0, vocab); and the corpus' length where the steps look for it
__global__ __launch_bounds__(kThreads) void k_check_tokens(const int32_t* __restrict__ tok, u64 T, int vocab, int vocab_all, State* st, u64* len) {
    if (blockIdx.x == 0 && threadIdx.x == 0) len[0] = st->length = T;
    bool bad = false, foreign = false;
    for (u64 i = (u64)blockIdx.x * kThreads + threadIdx.x; i < T; i += (u64)gridDim.x * kThreads) {
        bad = bad || (u32)tok[i] >= (u32)vocab_all;
        foreign = foreign || (u32)tok[i] >= (u32)vocab;
    }
    if (bad) st->bad = 1;
    if (foreign) st->foreign = st->stuck = 1;
}

// The corpus: an even number of merges leaves it in the first of the two places, an odd one in the second.  The steps look for the number in
// `State`: whether the one before it found a merge is not known when a step is launched.
struct Corpus {
    int32_t* tok[2];
    uint8_t* last[2];            // 1: the output's last token
    u64* len;                    // by merges
};
// Of the tokens made since the sieve's pairs were counted: the first and the last token of then
struct Ends {
    int32_t *first, *last;       // [budget]
    int32_t vocab, base, budget; // tokens below `base` were there
    __device__ __forceinline__ int32_t first_of(int32_t t) const { return t < base ? t : first[t - vocab]; }
    __device__ __forceinline__ int32_t last_of(int32_t t) const { return t < base ? t : last[t - vocab]; }
};

// `best` becomes merge number st->merges (one thread)
__device__ void take_merge(const TascGram& best, int bits, const Ends& ends, State* st, Merge* merges) {
    if (best.count == 0) {
        st->done = 1;
        st->taken = 0;
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
    ends.first[m] = ends.first_of(out.row[1]);
    ends.last[m] = ends.last_of(out.row[best.n]);
    bool overlaps = false;
    for (u32 s = 1; s < best.n; ++s) {                       // shifted by s, the n-gram agrees with itself
        bool same = true;
        for (u32 j = 0; j + s < best.n; ++j) same = same && out.row[1 + j] == out.row[1 + j + s];
        overlaps = overlaps || same;
    }
    // few merges are worth less than two fifths of the one before, but where they fall fast they tend to go on falling
    const u64 before = st->reward, reward = (u64)best.count * (best.n - 1);
    st->want = reward * 2 / 5;
    if (before > reward) st->want = min(st->want, (u64)((double)reward / before * reward / 2));
    st->reward = reward;
    st->retry = 0;
    st->taken = 1;
    st->n = best.n;
    st->freq = best.count;
    st->seen = 0;
    st->overlaps = overlaps;
    st->new_id = ends.vocab + (int32_t)m;
    st->merges = m + 1;
    if (m + 1 == (u32)ends.budget) st->done = 1;
}
__device__ __forceinline__ TascGram best_of_wave(TascGram best, int bits) {
    // first by {reward, shorter}; the tokens are looked at where that leaves more than one
    const u64 rank = best.count ? (u64)best.count * (best.n - 1) << 4 | (15 - best.n) : 0;
    u64 most = rank;
    for (int o = 32; o > 0; o >>= 1) most = max(most, (u64)__shfl_xor((long long)most, o));
    const u64 equals = __ballot(rank == most);
    if (most == 0 || __popcll(equals) == 1) {
        const int l = __builtin_ctzll(equals);
        return TascGram{(u64)__shfl((long long)best.lo, l), (u64)__shfl((long long)best.hi, l), (u32)__shfl((int)best.count, l), (u32)__shfl((int)best.n, l)};
    }
    for (int o = 32; o > 0; o >>= 1) {
        const TascGram g{(u64)__shfl_xor((long long)best.lo, o), (u64)__shfl_xor((long long)best.hi, o), (u32)__shfl_xor((int)best.count, o), (u32)__shfl_xor((int)best.n, o)};
        if (tasc_gram_before(g, best, bits)) best = g;
    }
    return best;
}

// the best of the partitions' candidates
__global__ __launch_bounds__(kThreads) void k_pick(const TascGram* __restrict__ cands, u32 count, int bits, Ends ends, State* st, Merge* merges) {
    if (idle(st)) {
        if (threadIdx.x == 0) st->taken = 0;
        return;
    }
    TascGram best{0, 0, 0, 0};
    for (u32 i = threadIdx.x; i < count; i += kThreads)
        if (tasc_gram_before(cands[i], best, bits)) best = cands[i];
    __shared__ TascGram s_best[kThreads / 64];
    best = best_of_wave(best, bits);
    if ((threadIdx.x & 63) == 0) s_best[threadIdx.x >> 6] = best;
    __syncthreads();
    if (threadIdx.x != 0) return;
    for (int w = 1; w < kThreads / 64; ++w)
        if (tasc_gram_before(s_best[w], best, bits)) best = s_best[w];
    take_merge(best, bits, ends, st, merges);
}

// ---- The sieve: the next merge without counting every n-gram.  Most n-grams cannot win: the reward of a window of n <= n_max tokens is at most
// (n_max - 1) times the count of any pair of neighbours in it.
//   * k_pairs counts the pairs of neighbours in kBuckets buckets by hash, a table per workgroup in LDS, and k_pair_sums adds the tables up: no pair
//     is more frequent than its bucket says.  Once for a batch of merges: a pair with a token made since occurs wherever the token's last (or
//     first) old one had the same neighbour, so that pair's bucket bounds it.
//   * k_sift counts the windows all of whose pairs lie in buckets of at least `least` (least_count): those of a block of positions in LDS, by n and
//     a hash of 60 bits, and lists what it found by ranges of the hash;
//   * k_gather adds up what the blocks listed, a range a workgroup, and the last workgroup to end takes the best.
// What was not counted occurs less than `least` times, so a reward above (n_max - 1) (least - 1) is the best of all.  A count by hash is never too
// small, so if the windows of the n-gram taken are as many as its count (k_apply looks), no other n-gram has more: the result is exact.  Where
// the latter fails, or the lists or tables are full, the host has the next merges counted in full (tasc_count_best) and comes back.
// No atomics on memory but one a block and range: with a table there for all blocks these waited for each other at the frequent n-grams (k_sift 40 to 55 us).
// Latency bounds all of it; 1.0 M tokens of phrases, n_max 4: a quarter of the positions begin a window, some hundred n-grams are counted.
constexpr int kBucketBits = 14, kBuckets = 1 << kBucketBits;          // 64 KB of counters
constexpr int kPairThreads = 1024, kPairSpan = 16 * kPairThreads;
constexpr u32 kPairWgs = 256;
constexpr int kSumThreads = 256, kSumWgs = kBuckets / 64;
constexpr int kSiftThreads = 1024, kSiftSpan = 4096, kSiftSlots = 4096, kSiftWindows = 8192;
constexpr u32 kListed = 1024;                                         // n-grams of a block that there is room for, on average
constexpr int kGatherThreads = 1024, kGatherSlots = 4096, kProbes = 64;
constexpr u32 kGatherWgs = 32, kGatherMost = 256;                     // at least, at most

__device__ __forceinline__ u32 bucket_of(u32 a, u32 b) {
    u32 h = a * 0x9E3779B1u + b * 0x85EBCA77u;
    h ^= h >> 16;
    return (h * 0xC2B2AE3Du) >> (32 - kBucketBits);
}

// part[workgroup][bucket]; a workgroup takes `span` positions (a multiple of kPairSpan)
__global__ __launch_bounds__(kPairThreads) void k_pairs(Corpus corpus, State* st, u64 span, u32* __restrict__ part) {
    __shared__ __attribute__((aligned(16))) u32 s_n[kBuckets];
    if (idle(st)) return;
    const u32 merges = st->merges;
    const int32_t* __restrict__ const tok = corpus.tok[merges & 1];
    const uint8_t* __restrict__ const last = corpus.last[merges & 1];
    if (blockIdx.x == 0 && threadIdx.x == 0) st->top = 0;    // (k_pair_sums')
    const u64 T = corpus.len[merges], end = min(T, (blockIdx.x + 1) * span);
    for (int i = threadIdx.x; i < kBuckets / 4; i += kPairThreads) reinterpret_cast<uint4*>(s_n)[i] = make_uint4(0, 0, 0, 0);
    __syncthreads();
    for (u64 p0 = blockIdx.x * span; p0 < end; p0 += kPairSpan) {
        int4 t[4];                                           // 16 positions of a thread, all loads at once (up to 3 past the end, inside the
        int32_t then[4];                                     // call's memory)
        u32 e[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const u64 p = p0 + 4 * (u * kPairThreads + threadIdx.x), at = p < end ? p : 0;
            t[u] = *reinterpret_cast<const int4*>(tok + at);
            e[u] = *reinterpret_cast<const u32*>(last + at);
            then[u] = tok[p + 4 < T ? p + 4 : 0];
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const u64 p = p0 + 4 * (u * kPairThreads + threadIdx.x);
            const u32 v[5] = {(u32)t[u].x, (u32)t[u].y, (u32)t[u].z, (u32)t[u].w, (u32)then[u]};
#pragma unroll
            for (int q = 0; q < 4; ++q)
                if (p + q < end && ((e[u] >> (8 * q)) & 0xFF) == 0) atomicAdd(&s_n[bucket_of(v[q], v[q + 1])], 1u);
        }
    }
    __syncthreads();
    for (int i = threadIdx.x; i < kBuckets / 4; i += kPairThreads)
        reinterpret_cast<uint4*>(part)[(size_t)blockIdx.x * (kBuckets / 4) + i] = reinterpret_cast<const uint4*>(s_n)[i];
}
// sums[bucket] of 64 buckets, a quarter of the tables a wave, and st->top
__global__ __launch_bounds__(kSumThreads) void k_pair_sums(const u32* __restrict__ part, u32 parts, State* st, u32* __restrict__ sums) {
    __shared__ u32 s_n[kSumThreads];
    if (idle(st)) return;
    const u32 lane = threadIdx.x & 63, b = blockIdx.x * 64 + lane;
    u32 n = 0;
#pragma unroll 16
    for (u32 g = threadIdx.x / 64; g < parts; g += kSumThreads / 64) n += part[(size_t)g * kBuckets + b];
    s_n[threadIdx.x] = n;
    __syncthreads();
    if (threadIdx.x >= 64) return;
    n = (s_n[lane] + s_n[lane + 64]) + (s_n[lane + 128] + s_n[lane + 192]);
    sums[b] = n;
    for (int o = 32; o > 0; o >>= 1) n = max(n, (u32)__shfl_xor((int)n, o));
    if (lane == 0) atomicMax(&st->top, n);
}
// The least count of a bucket whose pairs are looked at.  (n_max - 1) times it has to stay below the best reward, which no pair's count exceeds
// (fresh: the pairs are those of the corpus as it stands), nor, as a rule, what the merges before let expect (take_merge).  If that was
// too much, the best of what was counted is a bound that holds.
__device__ __forceinline__ u32 least_count(const State* __restrict__ st, bool fresh, int n_max) {
    const u64 want = st->retry ? st->want : max(fresh ? (u64)st->top * 3 / 5 : 0, st->want);
    return max(1u, (u32)(want / (u64)(n_max - 1)));
}

struct __attribute__((aligned(16))) Found {      // of a block of positions: an n-gram by its hash {60, n : 4}, one of its places, its windows there
    u64 hash;
    u32 at, count;
};

struct Lists {           // [ranges][most] and how many there are
    Found* found;
    u32* listed;
    u32 ranges, most;
};

__global__ __launch_bounds__(kSiftThreads) void k_sift(Corpus corpus, State* st, const u32* __restrict__ sums, Ends ends, bool fresh, int n_max,
                                                       Lists lists) {
    constexpr int W = kSiftSpan / kSiftThreads, S = kSiftSlots / kSiftThreads;
    __shared__ __attribute__((aligned(16))) int32_t s_tok[kSiftSpan + 8];
    __shared__ u32 s_pass[kBuckets / 32];
    __shared__ u64 s_ok[kSiftSpan / 64 + 1];                      // a bit per position: it and the next one are a pair that passes
    __shared__ u64 s_key[kSiftSlots];                             // 0 = free
    __shared__ u32 s_val[kSiftSlots];                             // {count : 13, one of its places : 12}, the place of whoever counted first
    __shared__ u32 s_full, s_windows, s_total, s_open, s_listed[kGatherMost];              // of a range: how many, then where they go
    __shared__ uint16_t s_window[kSiftWindows];                   // {place : 12, n - 1 : 4}
    if (blockIdx.x == 0 && threadIdx.x == 0) st->taken = 0;
    if (idle(st)) return;
    const u32 merges = st->merges;
    const int32_t* __restrict__ const tok = corpus.tok[merges & 1];
    const uint8_t* __restrict__ const last = corpus.last[merges & 1];
    const u64 T = corpus.len[merges], base = (u64)blockIdx.x * kSiftSpan;
    if (base >= T) return;
    const int tid = threadIdx.x, lane = tid & 63;
    int32_t t[W];
    bool inside[W];                                          // of positions w kSiftThreads + tid: the next token is of the same output
#pragma unroll
    for (int w = 0; w < W; ++w) {
        const u64 p = base + w * kSiftThreads + tid, q = p < T ? p : 0;
        t[w] = tok[q];
        inside[w] = last[q] == 0 && p < T;
    }
    int32_t t8 = -1;
    bool beyond = false;
    if (tid < 8 && base + kSiftSpan + tid < T) {
        t8 = tok[base + kSiftSpan + tid];
        beyond = !last[base + kSiftSpan + tid];
    }
    const u32 least = least_count(st, fresh, n_max);
    u32 n_of[kBuckets / kSiftThreads], open = 0;
    if (tid == 0) s_open = 0;
#pragma unroll
    for (int w = 0; w < kBuckets / kSiftThreads; ++w) n_of[w] = sums[w * kSiftThreads + tid];
#pragma unroll
    for (int w = 0; w < W; ++w) s_tok[w * kSiftThreads + tid] = t[w];
    __syncthreads();
    if (tid < 8) s_tok[kSiftSpan + tid] = t8;
#pragma unroll
    for (int w = 0; w < kBuckets / kSiftThreads; ++w) {
        const u64 bits = __ballot(n_of[w] >= least);
        if (lane == 0) reinterpret_cast<u64*>(s_pass)[(w * kSiftThreads + tid) / 64] = bits;
        open += (u32)__popcll(bits);
    }
    if (lane == 0) atomicAdd(&s_open, open);
#pragma unroll
    for (int u = 0; u < S; ++u) {
        s_key[u * kSiftThreads + tid] = 0;
        s_val[u * kSiftThreads + tid] = 0;
    }
    if (tid < (int)kGatherMost) s_listed[tid] = 0;
    if (tid == 0) s_full = s_windows = s_total = 0;
    __syncthreads();
    if (s_open > kBuckets / 4) {                             // (nor is this)
        if (tid == 0) st->gave_up = 1;
        return;
    }
    auto passes = [&](int i) {
        const u32 b = bucket_of((u32)ends.last_of(s_tok[i]), (u32)ends.first_of(s_tok[i + 1]));
        return (s_pass[b >> 5] >> (b & 31)) & 1;
    };
#pragma unroll
    for (int w = 0; w < W; ++w) {
        const int i = w * kSiftThreads + tid;
        const u64 ok = __ballot(inside[w] && passes(i));
        if (lane == 0) s_ok[i / 64] = ok;
    }
    if (tid < 64) {                                          // the pairs that windows of the last positions reach
        const u64 ok = __ballot(tid < 7 && beyond && passes(kSiftSpan + tid));
        if (tid == 0) s_ok[kSiftSpan / 64] = ok;
    }
    __syncthreads();
    auto count = [&](int i, int n) {
        u32 v[TASC_MAX_ORDER], h0 = (u32)n, h1 = 0x1234567u;
#pragma unroll
        for (int j = 0; j < TASC_MAX_ORDER; ++j) v[j] = (u32)s_tok[i + j < kSiftSpan + 8 ? i + j : i];
#pragma unroll
        for (int j = 0; j < TASC_MAX_ORDER; ++j)
            if (j < n) {
                h0 = (h0 ^ v[j]) * 0x9E3779B1u;
                h0 ^= h0 >> 15;
                h1 = (h1 + v[j]) * 0x85EBCA77u;
                h1 ^= h1 >> 13;
            }
        h0 *= 0xC2B2AE3Du;
        const u64 key = ((u64)h0 << 32) | (h1 & ~15u) | (u32)n;      // (never 0; of equal keys the n-grams are equally long)
        u32 idx = h0 >> 20;
        for (int probe = 0; probe < kProbes; ++probe, idx = (idx + 1) & (kSiftSlots - 1)) {
            const u64 old = atomicCAS((unsigned long long*)&s_key[idx], 0ull, (unsigned long long)key);
            if (old == 0) {
                atomicAdd(&s_val[idx], 1u << 12 | (u32)i);
                return;
            }
            if (old == key) {
                atomicAdd(&s_val[idx], 1u << 12);
                return;
            }
        }
        s_full = 1;
    };
    // Few positions have a window, and a window is a chain of LDS round trips: listed first, so that all lanes have one (a position a
    // lane, k_sift took 35 us); those of a quarter of the positions at a time where the list does not hold them all.
    int longest[W];
    u32 all[W], total = 0;                                   // of the wave
#pragma unroll
    for (int w = 0; w < W; ++w) {
        const int i = w * kSiftThreads + tid;
        const u64 ok = (s_ok[i / 64] >> lane) | (lane ? s_ok[i / 64 + 1] << (64 - lane) : 0);
        longest[w] = min(n_max, __builtin_ctz((u32)~ok | 1u << (TASC_MAX_ORDER - 1)) + 1);
        all[w] = 0;
        for (int n = 2; n <= n_max; ++n) all[w] += (u32)__popcll(__ballot(longest[w] >= n));
        total += all[w];
    }
    if (lane == 0 && total) atomicAdd(&s_total, total);
    __syncthreads();
    const bool at_once = s_total <= (u32)kSiftWindows;
#pragma unroll
    for (int w = 0; w < W; ++w) {
        if (all[w] != 0) {
            const int i = w * kSiftThreads + tid;
            u32 at = lane == 0 ? atomicAdd(&s_windows, all[w]) : 0;
            at = (u32)__builtin_amdgcn_readfirstlane((int)at);
            for (int n = 2; n <= n_max; ++n) {
                const u64 have = __ballot(longest[w] >= n);
                if (longest[w] >= n) s_window[at + (u32)__popcll(have & ((1ull << lane) - 1))] = (uint16_t)(i << 4 | (n - 1));
                at += (u32)__popcll(have);
            }
        }
        if (at_once && w + 1 < W) continue;
        __syncthreads();
        const u32 windows = s_windows;
        for (u32 e = tid; e < windows && !*(volatile u32*)&s_full; e += kSiftThreads) count(s_window[e] >> 4, (s_window[e] & 15) + 1);
        __syncthreads();
        if (tid == 0) s_windows = 0;
        __syncthreads();
    }
    static_assert(kSiftWindows >= kSiftThreads * (TASC_MAX_ORDER - 1), "windows of a quarter of the positions");
    if (s_full) {
        if (tid == 0) st->gave_up = 1;
        return;
    }
    u64 key[S];
    u32 at[S], range[S];
#pragma unroll
    for (int u = 0; u < S; ++u) {
        key[u] = s_key[u * kSiftThreads + tid];
        range[u] = __umulhi((u32)(key[u] >> 32), lists.ranges);
        at[u] = key[u] ? atomicAdd(&s_listed[range[u]], 1u) : 0;
    }
    __syncthreads();
    if (tid < (int)lists.ranges) {
        const u32 n = s_listed[tid], to = n ? atomicAdd(&lists.listed[tid], n) : 0;
        if (to + n > lists.most) st->gave_up = 1;
        s_listed[tid] = to + n > lists.most ? lists.most : to;
    }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < S; ++u) {
        const u32 to = s_listed[range[u]] + at[u];
        if (key[u] == 0 || to >= lists.most) continue;
        const u32 v = s_val[u * kSiftThreads + tid];
        lists.found[(size_t)range[u] * lists.most + to] = Found{key[u], (u32)base + (v & (kSiftSpan - 1)), v >> 12};
    }
}
static_assert(kSiftSpan == 1 << 12 && TASC_MAX_ORDER < 16 && kSiftSlots == 1 << 12, "fields of a slot and of a window; bits of the hash");

// the best among equals in rank, by the tokens: of one wave's candidates, those with `mine`
__device__ __forceinline__ TascGram smallest(bool mine, TascGram g, const int32_t* __restrict__ tok, u32 at, int bits) {
    int32_t t[TASC_MAX_ORDER];
#pragma unroll
    for (int j = 0; j < TASC_MAX_ORDER; ++j) t[j] = tok[mine ? at + j : 0];      // (past the n-gram's end: inside the call's memory)
#pragma unroll
    for (int j = 0; j < TASC_MAX_ORDER; ++j)
        if (j < (int)g.n) tasc_key_put(g.lo, g.hi, j, bits, (u32)t[j]);
    if (!mine) g = TascGram{0, 0, 0, 0};
    return best_of_wave(g, bits);
}

__global__ __launch_bounds__(kGatherThreads) void k_gather(Corpus corpus, Lists lists, Ends ends, bool fresh, int n_max, int bits,
                                                           State* st, Merge* merges, TascGram* best_of) {
    __shared__ u64 s_key[kGatherSlots];                           // 0 = free
    __shared__ u32 s_count[kGatherSlots], s_at[kGatherSlots];
    __shared__ u64 s_most[kGatherThreads / 64];
    __shared__ u32 s_full, s_equals, s_equal[64];
    if (idle(st)) return;
    const bool gave_up = st->gave_up != 0;                   // (what is listed is not all, and may be more than there is room for)
    const u32 all = gave_up ? 0 : lists.listed[blockIdx.x], lane = threadIdx.x & 63, wave = threadIdx.x / 64;
    const Found* __restrict__ const found = lists.found + (size_t)blockIdx.x * lists.most;
    for (int i = threadIdx.x; i < kGatherSlots; i += kGatherThreads) {
        s_key[i] = 0;
        s_count[i] = 0;
    }
    if (threadIdx.x == 0) s_full = s_equals = 0;
    const int32_t* __restrict__ const tok = corpus.tok[st->merges & 1];
    __syncthreads();
    for (u32 e = threadIdx.x; e < all; e += kGatherThreads) {
        const Found f = found[e];
        u32 idx = ((u32)f.hash * 0x9E3779B1u) >> 20;
        bool mine = false;
        for (int probe = 0; probe < kProbes && !mine; ++probe) {
            const u64 old = atomicCAS((unsigned long long*)&s_key[idx], 0ull, (unsigned long long)f.hash);
            if (old == 0) s_at[idx] = f.at;
            mine = old == 0 || old == f.hash;
            if (mine) atomicAdd(&s_count[idx], f.count);
            idx = (idx + 1) & (kGatherSlots - 1);
        }
        if (!mine) s_full = 1;
    }
    __syncthreads();
    // the largest reward of the range, then the shortest and smallest n-gram that has it: only those are read from the corpus
    constexpr int S = kGatherSlots / kGatherThreads;
    u64 rank[S], most = 0;                                   // {reward, 15 - n}
#pragma unroll
    for (int u = 0; u < S; ++u) {
        const int i = u * kGatherThreads + threadIdx.x;
        const u32 n = (u32)s_key[i] & 15;
        rank[u] = n ? ((u64)s_count[i] * (n - 1)) << 4 | (15 - n) : 0;
        most = max(most, rank[u]);
    }
    for (int o = 32; o > 0; o >>= 1) most = max(most, (u64)__shfl_xor((long long)most, o));
    if (lane == 0) s_most[wave] = most;
    __syncthreads();
    most = s_most[lane & (kGatherThreads / 64 - 1)];
    for (int o = kGatherThreads / 128; o > 0; o >>= 1) most = max(most, (u64)__shfl_xor((long long)most, o));
#pragma unroll
    for (int u = 0; u < S; ++u)
        if (most != 0 && rank[u] == most) {
            const u32 q = atomicAdd(&s_equals, 1u);
            if (q < 64) s_equal[q] = u * kGatherThreads + threadIdx.x;
            else s_full = 1;
        }
    __syncthreads();
    if (wave != 0) return;
    {
        const bool mine = lane < s_equals;
        const u32 i = mine ? s_equal[lane] : 0;
        TascGram best = smallest(mine, TascGram{0, 0, s_count[i], (u32)s_key[i] & 15}, tok, mine ? s_at[i] : 0, bits);
        u32 before = 0;
        if (lane == 0) {
            if (s_full) best.n = ~0u;
            best_of[blockIdx.x] = best;
            lists.listed[blockIdx.x] = 0;                    // (for the next merge)
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
            before = __hip_atomic_fetch_add(&st->arrived, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        if ((u32)__builtin_amdgcn_readfirstlane((int)before) + 1 != gridDim.x) return;
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
    }
    const u32 least = least_count(st, fresh, n_max);
    TascGram best{0, 0, 0, 0};
    bool full = false;
    for (u32 i = lane; i < gridDim.x; i += 64) {
        const TascGram g = best_of[i];
        full = full || g.n == ~0u;
        if (g.n != ~0u && tasc_gram_before(g, best, bits)) best = g;
    }
    full = __ballot(full) != 0;
    best = best_of_wave(best, bits);
    if (lane != 0) return;
    const u64 reward = (u64)best.count * (best.n - 1);
    st->arrived = 0;
    if (full || gave_up) {
        st->stuck = 1;
    } else if (best.count != 0 && reward > (u64)(n_max - 1) * (least - 1)) {
        take_merge(best, bits, ends, st, merges);
    } else if (!st->retry) {
        st->want = reward;                                   // (nothing found: every pair is looked at)
        st->retry = 1;
    } else if (best.count == 0 && least == 1) {
        take_merge(best, bits, ends, st, merges);            // nothing left
    } else {
        st->stuck = 1;
    }
}

struct Gram {            // the running merge, in registers
    u32 n, overlaps, merges, freq;               // merges: this one included
    int32_t t[TASC_MAX_ORDER], new_id;
};
__device__ __forceinline__ Gram running(const State* __restrict__ st) {
    Gram g{st->n, st->overlaps, st->merges, st->freq, {}, st->new_id};
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

// Left-to-right choice among occurrences that can overlap (the others are all taken, and found where they are needed): sel[i] = number
// of the step, which no other one has (a merge's number comes again if it is taken back, and its marks stay).  An occurrence with none
// in the n - 1 positions before it ("head") is always taken; from it, one lane walks the run of occurrences that overlap each other,
// taking the first at or after the end of the last taken one, and stops when that one is a head itself (its own lane takes it) or lies
// beyond the reach of an overlap.  A walk is a chain of dependent loads, and a long run of one token is one walk: after kLaneSteps
// steps the wave takes it over, 64 positions at a time, and the steps among them are a few instructions (200,000 equal tokens, four
// merges of two: 176 ms with the lane alone; 61 with a byte per position to read instead of the tokens; 16 so).  The walk ends at the
// latest at the end of the corpus.
constexpr unsigned kSelectBlocks = 256, kSelectThreads = 256;
constexpr int kLaneSteps = 8;
__global__ __launch_bounds__(kSelectThreads) void k_select(Corpus corpus, State* st, u32* sel, u32 step) {
    __shared__ u32 s_seen;
    if (no_merge(st) || !st->overlaps) return;
    const Gram g = running(st);
    const int32_t* __restrict__ const tok = corpus.tok[(g.merges - 1) & 1];
    const uint8_t* __restrict__ const last = corpus.last[(g.merges - 1) & 1];
    const u64 T = corpus.len[g.merges - 1];
    const int n = (int)g.n, lane = threadIdx.x & 63;
    u32 seen = 0;
    if (threadIdx.x == 0) s_seen = 0;
    __syncthreads();
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
    for (u64 i0 = (u64)blockIdx.x * kSelectThreads + threadIdx.x - lane; i0 < T; i0 += (u64)gridDim.x * kSelectThreads) {
        const u64 i = i0 + lane;
        u64 cur = i;
        const bool here = i < T && matches(tok + i, last, T, i, g);
        seen += (u32)__popcll(__ballot(here));
        bool walking = here && is_head(i);
        for (int s = 0; walking && s < kLaneSteps; ++s) {
            sel[cur] = step;
            u64 next = T;
            for (u64 p = cur + n; p < cur + 2 * (u64)n - 1 && p < T; ++p)
                if (matches(tok + p, last, T, p, g)) { next = p; break; }
            walking = next < T && !is_head(next);
            cur = next;
        }
        // (the last step's `next` of a lane that is still walking is an occurrence that has to be taken)
        for (u64 todo = __ballot(walking); todo != 0; todo &= todo - 1) {
            u64 at = __shfl(cur, __ffsll(todo) - 1);         // taken; the next one lies n to 2 n - 2 positions on
            if (lane == 0) sel[at] = step;
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
                if ((taken >> lane) & 1) sel[base + lane] = step;
                at = base + c;
            }
        }
    }
    if (lane == 0 && seen) atomicAdd(&s_seen, seen);
    __syncthreads();
    if (threadIdx.x == 0 && s_seen) atomicAdd(&st->seen, s_seen);
}

// What a block of kBlock positions does with the merge: its tokens, 8 more on either side, come to LDS, and from them (or from the
// choice made above) where occurrences start.  keep: of the kItems positions of a thread, those that no taken
// occurrence swallows; starts: those where one begins.
struct BlockTokens {
    int32_t tok[kBlock + 16];
    __attribute__((aligned(16))) uint8_t start[kBlock + 16];
};
__device__ inline void block_keep(BlockTokens& s, const int32_t* __restrict__ tok, const uint8_t* __restrict__ last, const u32* __restrict__ sel,
                                  u32 step, u64 T, const Gram& g, u32& keep, u32& starts) {
    const int64_t base = (int64_t)blockIdx.x * kBlock - 8;
    for (int q = threadIdx.x; q < kBlock + 16; q += kThreads) s.tok[q] = base + q >= 0 && base + q < (int64_t)T ? tok[base + q] : -1;
    __syncthreads();
    for (int q = threadIdx.x; q < kBlock + 8; q += kThreads) {
        const int64_t p = base + q;
        s.start[q] = p >= 0 && p < (int64_t)T && (g.overlaps ? sel[p] == step : matches(s.tok + q, last, T, (u64)p, g)) ? 1 : 0;
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

__global__ __launch_bounds__(kThreads) void k_sums(Corpus corpus, const u32* __restrict__ sel, u32 step, const State* __restrict__ st, u32* bsum) {
    __shared__ BlockTokens s;
    __shared__ u32 s_wave[kThreads / 64];
    if (no_merge(st)) return;
    const Gram g = running(st);
    const u32 from = (g.merges - 1) & 1;
    u32 keep, starts, sum;
    block_keep(s, corpus.tok[from], corpus.last[from], sel, step, corpus.len[g.merges - 1], g, keep, starts);
    block_scan(__popc(keep), s_wave, &sum);
    if (threadIdx.x == 0) bsum[blockIdx.x] = sum;
}
// bsum (nullable): k_sums' ; without, a block tells the others its own sum, as {step, sum}, and waits for those before it.  Every die starts its
// blocks in order, so the first block that has not started waits only for room that started ones take up, and none of those waits for it.  A launch
// and another look at the corpus less, but every block reads every sum before its own: up to kTellBlocks of them.  A block that does not hear from
// another in `wait` looks gives up (the GPU may be shared): the call makes the merge again, with k_sums.
constexpr u32 kTellBlocks = 1024;
__global__ __launch_bounds__(kThreads) void k_apply(Corpus corpus, const u32* __restrict__ sel, u32 step, State* st, const u32* __restrict__ bsum, u64* told,
                                                    u32 wait) {
    __shared__ BlockTokens s;
    __shared__ u32 s_wave[kThreads / 64];
    if (no_merge(st)) return;
    const Gram g = running(st);
    const int32_t* __restrict__ const tok = corpus.tok[(g.merges - 1) & 1];
    const uint8_t* __restrict__ const last = corpus.last[(g.merges - 1) & 1];
    int32_t* __restrict__ const out = corpus.tok[g.merges & 1];
    uint8_t* __restrict__ const last_out = corpus.last[g.merges & 1];
    const u64 T = corpus.len[g.merges - 1], first = (u64)blockIdx.x * kBlock + kItems * threadIdx.x;
    static_assert(kItems == 4, "a word of ends");
    const u32 ends = *reinterpret_cast<const u32*>(last + (first < T ? first : 0));
    u32 keep, starts, sum, base;
    block_keep(s, tok, last, sel, step, T, g, keep, starts);
    u32 to = block_scan(__popc(keep), s_wave, &sum);
    if (bsum) {
        base = blocks_before(bsum, s_wave);
    } else {
        if (threadIdx.x == 0) __hip_atomic_store(&told[blockIdx.x], (u64)step << 32 | sum, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        u32 n = 0;
        if (threadIdx.x < blockIdx.x) {
            bool heard = false;
            for (u32 looks = 0; !heard && looks < wait; ++looks) {
                const u64 v = __hip_atomic_load(&told[threadIdx.x], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                heard = (u32)(v >> 32) == step;
                n = heard ? (u32)v : 0;
            }
            if (!heard) st->late = 1;                        // (what follows lands too far in front, and is not used)
        }
        block_scan(n, s_wave, &base);
    }
    to += base;
    if (blockIdx.x == gridDim.x - 1 && threadIdx.x == 0) {
        corpus.len[g.merges] = st->length = base + sum;
        // (of an n-gram that does not overlap itself every window is merged)
        if (g.overlaps ? st->seen != g.freq : T - (base + sum) != (u64)g.freq * (g.n - 1)) st->undo = 1;
    }
    for (u32 k = keep; k != 0; k &= k - 1, ++to) {
        const int e = __ffs((int)k) - 1;
        const bool merged = (starts >> e) & 1;
        out[to] = merged ? g.new_id : s.tok[8 + kItems * threadIdx.x + e];
        last_out[to] = merged ? last[first + e + g.n - 1] : (uint8_t)(ends >> (8 * e));
    }
}
static_assert(kTellBlocks <= kThreads, "a thread per block before");

// What the merges so far leave: where the outputs end, in order, and the tokens; of a merge that is taken back, what it began with
__device__ __forceinline__ u32 standing(const State* __restrict__ st) { return st->merges - ((st->undo | st->late) != 0 ? 1 : 0); }
__device__ __forceinline__ u32 ends_here(const Corpus& c, u32 merges) {
    const u64 first = (u64)blockIdx.x * kBlock + kItems * threadIdx.x, T = c.len[merges];
    const uint8_t* __restrict__ const last = c.last[merges & 1];
    u32 f = 0;
#pragma unroll
    for (int e = 0; e < kItems; ++e) f |= first + e < T && last[first + e] ? 1u << e : 0;
    return f;
}
__global__ __launch_bounds__(kThreads) void k_end_sums(Corpus c, const State* __restrict__ st, u32* bsum) {
    __shared__ u32 s_wave[kThreads / 64];
    u32 sum;
    block_scan(__popc(ends_here(c, standing(st))), s_wave, &sum);
    if (threadIdx.x == 0) bsum[blockIdx.x] = sum;
}
__global__ __launch_bounds__(kThreads) void k_ends(Corpus c, const State* __restrict__ st, const u32* __restrict__ bsum, u32* ends, int32_t* out) {
    __shared__ u32 s_wave[kThreads / 64];
    u32 sum;
    const u32 merges = standing(st);
    const u64 T = c.len[merges];
    if (out && !st->bad)
        for (u32 e = threadIdx.x; e < kBlock; e += kThreads) {
            const u64 p = (u64)blockIdx.x * kBlock + e;
            if (p < T) out[p] = c.tok[merges & 1][p];
        }
    const u32 here = ends_here(c, merges);
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
    const bool run = budget > 0 && T0 > 0;
    Arena ar, counting;                                      // counting: for full counts, taken with the first of them
    // what the host looks at comes first, in one piece
    const size_t at_state = ar.carve(sizeof(State)), at_len = ar.carve(((size_t)budget + 1) * sizeof(u64)), at_merges = ar.carve((size_t)budget * sizeof(Merge));
    const size_t at_ends = ar.carve((size_t)n_docs * sizeof(u32));
    const size_t at_told = ar.carve((T0 + kBlock - 1) / kBlock * sizeof(u64)), at_listed = ar.carve(kGatherMost * sizeof(u32)), at_sel = ar.carve(T0 * sizeof(u32)), zeroed = ar.used;
    const size_t at_tok[2] = {ar.carve(T0 * sizeof(int32_t)), ar.carve(T0 * sizeof(int32_t))}, at_last[2] = {ar.carve(T0), ar.carve(T0)};
    const size_t at_off = ar.carve(((size_t)n_docs + 1) * sizeof(int64_t)), at_bsum = ar.carve((T0 + kBlock - 1) / kBlock * sizeof(u32));
    const u64 span = std::max<u64>(1, (T0 + (u64)kPairWgs * kPairSpan - 1) / ((u64)kPairWgs * kPairSpan)) * kPairSpan;
    const size_t at_pairs = ar.carve(run ? (T0 + span - 1) / span * kBuckets * sizeof(u32) : 0), at_sums = ar.carve(kBuckets * sizeof(u32));
    const u32 sift_blocks = run ? (u32)((T0 + kSiftSpan - 1) / kSiftSpan) : 0, gather_wgs = std::clamp(sift_blocks / 16, kGatherWgs, kGatherMost);
    const u32 most_listed = (u32)(((u64)sift_blocks * kListed + gather_wgs - 1) / gather_wgs);
    const size_t at_found = ar.carve((size_t)gather_wgs * most_listed * sizeof(Found)), at_sifted = ar.carve(gather_wgs * sizeof(TascGram));
    const size_t at_first = ar.carve((size_t)budget * sizeof(int32_t)), at_last_of = ar.carve((size_t)budget * sizeof(int32_t));
    TOK_TRY(ar.get(ar.used));
    State* const state = (State*)(ar.p + at_state);
    u64* const len = (u64*)(ar.p + at_len);
    int32_t* const tok[2] = {(int32_t*)(ar.p + at_tok[0]), (int32_t*)(ar.p + at_tok[1])};
    uint8_t *const last[2] = {(uint8_t*)(ar.p + at_last[0]), (uint8_t*)(ar.p + at_last[1])};
    int64_t* const d_off = (int64_t*)(ar.p + at_off);
    u32 *const bsum = (u32*)(ar.p + at_bsum), *const sel = (u32*)(ar.p + at_sel), *const ends = (u32*)(ar.p + at_ends);
    u64* const told = (u64*)(ar.p + at_told);
    u32 *const pairs = (u32*)(ar.p + at_pairs), *const sums = (u32*)(ar.p + at_sums);
    Merge* const d_merges = (Merge*)(ar.p + at_merges);
    const Lists lists{(Found*)(ar.p + at_found), (u32*)(ar.p + at_listed), gather_wgs, most_listed};
    TascGram* const sifted = (TascGram*)(ar.p + at_sifted);
    const Corpus corpus{{tok[0], tok[1]}, {last[0], last[1]}, len};

    // Full counts: as many orders together as kMostRecords hold records of (one order's are always held).  With few chunks an order alone
    // leaves the chip idle (ms, one at a time | together, n_max 6, eight merges: 1.0 M tokens 2.23 | 1.80, 4 M 5.33 | 4.66); many do not need
    // the others (16 M 19.0 | 18.3, 64 M 112.1 | 111.1).
    const TascCountPlan plan = tasc_count_plan(T0, windows, n_max * bits > 64, false);
    const size_t most = std::min(kMostRecords, (size_t)g_tasc_config.build_list_kib << 10);
    const int together = (int)std::clamp<size_t>(most / std::max<size_t>(1, plan.rec_bytes + plan.offs_bytes), 1, orders);
    TascGram* best = nullptr;
    TascCountBufs bufs{};
    auto full_counts = [&]() -> tasc_status {
        if (best) return TASC_OK;
        const size_t at_best = counting.carve((size_t)orders * plan.parts * sizeof(TascGram)), at_rec = counting.carve(together * plan.rec_bytes);
        const size_t at_roff = counting.carve(together * plan.offs_bytes), at_deal = counting.carve(plan.deal_bytes);
        // in what is left of the call's first block; or else in one that, if it is kept, holds all of the next call
        char* p = ar.p + ar.used;
        if (ar.bytes < ar.used + counting.used) {
            const size_t all = ar.used + counting.used;
            if (!tasc_scratch_kept(all) || counting.get(all) != TASC_OK) TOK_TRY(counting.get(counting.used));
            p = counting.p;
        }
        best = (TascGram*)(p + at_best);
        bufs = TascCountBufs{(u64*)(p + at_rec), (uint16_t*)(p + at_roff), (u64*)(p + at_deal)};
        return TASC_OK;
    };

    TASC_HIP(hipMemsetAsync(ar.p, 0, zeroed, st));
    if (T0) {
        TASC_HIP(hipMemcpyAsync(tok[0], tokens, T0 * sizeof(int32_t), where == TASC_MEM_HOST ? hipMemcpyHostToDevice : hipMemcpyDeviceToDevice, st));
        TASC_HIP(hipMemcpyAsync(d_off, doc_offsets, (size_t)(n_docs + 1) * sizeof(int64_t), hipMemcpyHostToDevice, st));
        TOK_TRY(tasc_mark_ends(d_off, n_docs, T0, last[0], st));
        // (without a merge to make, nothing looks at the tokens)
        k_check_tokens<<<dim3(run ? 256 : 1), dim3(kThreads), 0, st>>>(tok[0], run ? T0 : 0, vocab, vocab_all, state, len);
        if (!run) TASC_HIP(hipMemcpyAsync(len, &T0, sizeof T0, hipMemcpyHostToDevice, st));
        TASC_LAUNCH_CHECK();
    }
    std::vector<char> report(at_ends + (size_t)n_docs * sizeof(u32), 0);
    State h;
    memset(&h, 0, sizeof h);
    const u64* const lens = reinterpret_cast<const u64*>(report.data() + at_len);
    u64 T = T0;                                              // the corpus is no longer than this
    // The host's look at the state, and, where the merges may have come to their end, at all that the caller gets; nothing waits for the host in between.
    bool whole = false;
    auto look = [&](bool all) -> tasc_status {
        whole = all;
        if (!all) {
            TASC_HIP(hipMemcpyAsync(&h, state, sizeof h, hipMemcpyDeviceToHost, st));
            TASC_HIP(hipStreamSynchronize(st));
            return TASC_OK;
        }
        const dim3 grid((unsigned)((T + kBlock - 1) / kBlock));
        k_end_sums<<<grid, dim3(kThreads), 0, st>>>(corpus, state, bsum);
        if (grid.x > kScanFrom) k_scan<<<dim3(1), dim3(kThreads), 0, st>>>(bsum, grid.x);
        k_ends<<<grid, dim3(kThreads), 0, st>>>(corpus, state, bsum, ends, where == TASC_MEM_DEVICE ? out_tokens : nullptr);
        TASC_LAUNCH_CHECK();
        TASC_HIP(hipMemcpyAsync(report.data(), ar.p, report.size(), hipMemcpyDeviceToHost, st));
        TASC_HIP(hipStreamSynchronize(st));
        memcpy(&h, report.data() + at_state, sizeof h);
        return TASC_OK;
    };
    u32 step = 0;
    bool tell = true;
    // Merges that are still counted in full, and how many the next time that the sieve gives up; merges that it has made since the last time.  A try
    // that fails costs as much as it saves on some three merges, and what it does not settle tends to come one after the other: so the next one is
    // short, and comes after twice as many merges unless there was something to gain.
    u32 full = 0, next_full = kFirst, sieved = 0;
    for (int done = 0, batch = kFirst; run && done < budget && (!h.done || h.stuck || h.undo || h.late);) {
        const int begin = done, end = std::min(budget, done + (full ? (int)std::min<u32>(full, kBatch) : batch));
        if (full) TOK_TRY(full_counts());
        TascCountPlan p = plan;                              // (the records' strides are those of the whole corpus)
        p.chunks = (u32)((T + p.chunk - 1) / p.chunk);
        const dim3 grid1((unsigned)std::min<u64>((T + kSelectThreads - 1) / kSelectThreads, kSelectBlocks)), grid2((unsigned)((T + kBlock - 1) / kBlock));
        const dim3 grid_p((unsigned)((T + span - 1) / span)), grid_s((unsigned)((T + kSiftSpan - 1) / kSiftSpan));
        const Ends since{(int32_t*)(ar.p + at_first), (int32_t*)(ar.p + at_last_of), vocab, vocab + begin, budget};
        const bool told_all = tell && grid2.x <= kTellBlocks;
        if (!full) {
            k_pairs<<<grid_p, dim3(kPairThreads), 0, st>>>(corpus, state, span, pairs);
            k_pair_sums<<<dim3(kSumWgs), dim3(kSumThreads), 0, st>>>(pairs, grid_p.x, state, sums);
        }
        // (a try more than merges: one that has to be made again leaves the others in this look)
        for (int i = begin; i < end + (full ? 0 : 1); ++i) {
            if (full) {
                for (int n0 = 2; n0 <= n_max; n0 += together) {
                    const int here = std::min(together, n_max + 1 - n0);
                    TOK_TRY(tasc_count_partition(p, tok[i & 1], last[i & 1], false, T, len + i, n0, here, bits, bufs, nullptr, nullptr, st));
                    TOK_TRY(tasc_count_best(p, len + i, n0, here, bits, bufs, best + (size_t)(n0 - 2) * p.parts, st));
                }
                k_pick<<<dim3(1), dim3(kThreads), 0, st>>>(best, (u32)orders * p.parts, bits, since, state, d_merges);
            } else {
                k_sift<<<grid_s, dim3(kSiftThreads), 0, st>>>(corpus, state, sums, since, i == begin, n_max, lists);
                k_gather<<<dim3(gather_wgs), dim3(kGatherThreads), 0, st>>>(corpus, lists, since, i == begin, n_max, bits, state, d_merges, sifted);
            }
            k_select<<<grid1, dim3(kSelectThreads), 0, st>>>(corpus, state, sel, ++step);
            if (!told_all) k_sums<<<grid2, dim3(kThreads), 0, st>>>(corpus, sel, step, state, bsum);
            if (grid2.x > kScanFrom) k_scan<<<dim3(1), dim3(kThreads), 0, st>>>(bsum, grid2.x);
            k_apply<<<grid2, dim3(kThreads), 0, st>>>(corpus, sel, step, state, told_all ? nullptr : bsum, told, (u32)g_tasc_config.enrich_wait);
            TASC_LAUNCH_CHECK();
        }
        TOK_TRY(look(end == budget));
        TASC_REQUIRE(h.bad == 0, "tok_enrich: corpus holds a token outside [0, %d)", vocab_all);
        done = (int)(h.merges - (h.undo || h.late ? 1 : 0));
        if (!h.undo && !h.late) T = h.length;
        if (h.late) tell = false;
        const bool uncertain = h.stuck || h.undo;
        if (full) {
            full -= std::min(full, (u32)(done - begin));
        } else if (uncertain) {
            sieved += (u32)(done - begin);
            if (sieved >= (u32)kFirst) next_full = kFirst;
            full = h.foreign ? (u32)budget : next_full;
            next_full = std::min(2 * next_full, 1u << 16);
            sieved = 0;
            batch = 1;
        } else {
            sieved += (u32)(done - begin);
            batch = std::min(2 * batch, kBatch);
        }
        if (uncertain || h.late) {
            State again = h;
            again.merges = (u32)done;
            again.stuck = again.gave_up = again.undo = again.late = again.retry = again.taken = again.done = 0;
            again.reward = again.want = 0;                           // (the pairs are counted again, or k_pick leaves one)
            TASC_HIP(hipMemcpyAsync(state, &again, sizeof again, hipMemcpyHostToDevice, st));
            TASC_HIP(hipStreamSynchronize(st));
        }
    }
    if (T0 && !whole) TOK_TRY(look(true));
    const int n_done = (int)h.merges;
    T = T0 ? lens[n_done] : 0;
    const Merge* const rows = reinterpret_cast<const Merge*>(report.data() + at_merges);
    const u32* const h_ends = reinterpret_cast<const u32*>(report.data() + at_ends);
    if (T && where == TASC_MEM_HOST) {
        TASC_HIP(hipMemcpyAsync(out_tokens, tok[n_done & 1], T * sizeof(int32_t), hipMemcpyDeviceToHost, st));
        TASC_HIP(hipStreamSynchronize(st));
    }
    counting.keep();
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
