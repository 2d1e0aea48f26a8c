// Corpus n-gram tables on the GPU: counting, pruning, per-context aggregates, export.
//
// Paper, section "Proposed Method: TASC-spec": the drafter is a collection of n-gram models M_n,
// n <= n_max, each derived from the n-gram frequencies in the task corpus and pruned of the
// elements whose frequency is below p_min; the most frequent token is the last resort.
//
// Layout and algorithm (all integer, exact keys):
//   * counting table of one order: open addressing over 8-byte slots {first position + 1 : 32,
//     count : 32}.  A slot names its key by the position of its first occurrence in the corpus,
//     which stays resident, so a slot is claimed and counted with single 64-bit atomics and no
//     multi-word publication is needed.  Probing is linear.
//   * the addition that lifts a count to p_min also lists the slot, so the kept n-grams are known without
//     another pass over the counting table; they are re-inserted into two small tables that carry explicit
//     128-bit keys (32-byte slots, see TascSlot): the full table (context + successor -> count) and the
//     context table (context -> T, most frequent successor).
#include "tasc_internal.h"
#include <algorithm>
#include <string.h>

static thread_local char g_err[512] = "";
void tasc_set_error(const char* fmt, ...) {
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(g_err, sizeof g_err, fmt, ap);
    va_end(ap);
}
extern "C" const char* tasc_last_error(void) { return g_err; }

namespace {

constexpr int kThreads = 256;

// Token histogram.  Corpus tokens follow a steep rank-frequency law, so adding every occurrence straight to the
// global histogram serialises on the few hottest counters.  A workgroup therefore first counts a chunk of
// kUniChunk tokens in an LDS table (open addressing, twice as many slots as tokens, so it cannot fill up) and
// then adds each distinct token's count to a global histogram once: one of kUniCopies, by workgroup id, and so (the
// dispatcher deals ids to the 8 XCDs in turn) one per XCD, whose lines stay in that XCD's L2.
constexpr int kUniChunk = 2048, kUniSlots = 4096, kUniCopies = 8;
__global__ __launch_bounds__(kThreads) void k_unigram(const int32_t* __restrict__ tok, u64 T, int vocab, u32* hist, u32* bad) {
    __shared__ u32 s_key[kUniSlots];
    __shared__ u32 s_cnt[kUniSlots];
    hist += (size_t)(blockIdx.x % kUniCopies) * vocab;
    for (int i = threadIdx.x; i < kUniSlots; i += kThreads) { s_key[i] = 0xFFFFFFFFu; s_cnt[i] = 0; }
    __syncthreads();
    for (u64 c0 = (u64)blockIdx.x * kUniChunk; c0 < T; c0 += (u64)gridDim.x * kUniChunk) {
        for (int j = threadIdx.x; j < kUniChunk; j += kThreads) {
            const u64 i = c0 + j;
            if (i >= T) break;
            const int t = tok[i];
            if (t < 0 || t >= vocab) { atomicOr(bad, 1u); continue; }
            u32 h = ((u32)t * 2654435761u) >> 20;                      // top 12 bits: kUniSlots = 4096
            for (;;) {
                u32 old = s_key[h];                                        // (most tokens of a chunk have been seen)
                if (old == 0xFFFFFFFFu) old = atomicCAS(&s_key[h], 0xFFFFFFFFu, (u32)t);
                if (old == 0xFFFFFFFFu || old == (u32)t) { atomicAdd(&s_cnt[h], 1u); break; }
                h = (h + 1) & (kUniSlots - 1);
            }
        }
        __syncthreads();
        for (int i = threadIdx.x; i < kUniSlots; i += kThreads) {
            const u32 k = s_key[i];
            if (k != 0xFFFFFFFFu) {
                atomicAdd(&hist[k], s_cnt[i]);
                s_key[i] = 0xFFFFFFFFu;
                s_cnt[i] = 0;
            }
        }
        __syncthreads();
    }
}

// hist = the sum of the copies; best[0] = max over tokens of (count << 32) | (0xFFFFFFFF - token): largest count, smallest id
__global__ void k_unigram_argmax(const u32* copies, int vocab, u32* hist, u64* best) {
    int i = blockIdx.x * blockDim.x + threadIdx.x;
    u64 v = 0;
    for (; i < vocab; i += gridDim.x * blockDim.x) {
        u32 n = 0;
#pragma unroll
        for (int q = 0; q < kUniCopies; ++q) n += copies[(size_t)q * vocab + i];
        hist[i] = n;
        u64 c = ((u64)n << 32) | (u64)(0xFFFFFFFFu - (u32)i);
        v = c > v ? c : v;
    }
    for (int o = 32; o > 0; o >>= 1) {
        u64 w = __shfl_xor(v, o);
        v = w > v ? w : v;
    }
    if ((threadIdx.x & 63) == 0) atomicMax(best, v);
}

// rem[i] = tokens left in the document from position i on, saturated at 255
__global__ void k_mark_doc_tails(const int64_t* doc_off, int64_t n_docs, int n_max, uint8_t* rem) {
    int64_t d = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (d >= n_docs) return;
    int64_t b = doc_off[d], e = doc_off[d + 1];
    for (int j = 1; j < n_max && e - j >= b; ++j) rem[e - j] = (uint8_t)j;
}

template <int N>
__device__ inline bool same_window(const int32_t* __restrict__ tok, u64 p, const int32_t* w) {
    bool eq = true;
#pragma unroll
    for (int j = 0; j < N; ++j) eq = eq && (tok[p + j] == w[j]);
    return eq;
}

// Counting in two levels.  A workgroup takes chunks of kChunk consecutive corpus positions (coalesced scan,
// the chunk's tokens staged in LDS), counts the chunk's windows in an LDS hash table whose slots name their
// key by a position inside the chunk, and then adds every distinct window of the chunk to the global table
// once, with its chunk count.  Task corpora concentrate on few n-grams (the paper's typical-set argument), so
// the frequent ones would otherwise serialise hundreds of thousands of atomics on one address.
//
// What bounds it: the additions to the global table, a random slot each (half to 9 tenths of the windows, whatever the
// chunk length: 0.65 / 0.89 of the 2- / 5-grams at 2048 positions, 0.55 / 0.84 at 8192), and the corpus positions they
// are compared with.  So they run with full waves and kInFlight of them per thread on the way at once: the claims are
// listed as they are made (scanning the LDS table for them left two lanes of three idle), and the loads of kInFlight
// entries go out before the first is looked at.  32 M tokens, orders 2 to 5: 2.7 / 3.0 / 3.3 / 3.3 ms -> 2.05 / 2.2 / 2.3 / 2.4 ms
// an order, with the tally of the counting table (0.13 ms) inside and the kept n-grams listed, so that k_keep takes 0.2 ms instead
// of the 0.46 ms of a scan; additions to one counter by every wave of 2 M (materialising the contexts) had cost 0.1 ms.
constexpr int kChunk = 2048;
constexpr int kLdsSlots = 2 * kChunk;
constexpr int kInFlight = 4;
constexpr int kListed = 384;       // kept n-grams a chunk collects in LDS before it appends them to the list

// counters: [0] distinct n-grams, [1] kept n-grams; list (nullable, then nothing is kept) receives the slots whose count
// has reached p_min, counters[1] of them
template <int N>
__global__ __launch_bounds__(kThreads) void k_count(const int32_t* __restrict__ tok, const uint8_t* __restrict__ rem, u64 T,
                                                    int bits, u64* slots, u64 mask, u32 p_min, u64* counters, u64* list) {
    __shared__ int32_t s_tok[kChunk + TASC_MAX_ORDER];
    __shared__ u32 s_slot[kLdsSlots];          // {position in the chunk + 1 : 16, count : 16}
    __shared__ uint16_t s_claim[kChunk];       // the slots in use
    __shared__ u64 s_list[kListed];
    __shared__ u32 s_n, s_nl;
    __shared__ u64 s_at;
    const int tid = threadIdx.x;
    for (int i = tid; i < kLdsSlots; i += kThreads) s_slot[i] = 0;
    if (tid == 0) { s_n = 0; s_nl = 0; }
    u32 distinct = 0;
    for (u64 base = (u64)blockIdx.x * kChunk; base < T; base += (u64)gridDim.x * kChunk) {
        const int n_here = (int)min((u64)(kChunk + N - 1), T - base);
        for (int i = tid; i < n_here; i += kThreads) s_tok[i] = tok[base + i];
        __syncthreads();
        const int n_win = (int)min((u64)kChunk, T - base);
        for (int i = tid; i < n_win; i += kThreads) {
            if (rem[base + i] < N) continue;           // the window would leave its document
            u64 lo = 0, hi = 0;
#pragma unroll
            for (int j = 0; j < N; ++j) tasc_key_put(lo, hi, j, bits, (u32)s_tok[i + j]);
            u32 idx = (u32)(tasc_hash_key(lo, hi, N) >> 20) & (kLdsSlots - 1);
            for (int probe = 0; probe < kLdsSlots; ++probe) {
                u32 sl = s_slot[idx];
                if (sl == 0) {
                    const u32 old = atomicCAS(&s_slot[idx], 0u, ((u32)(i + 1) << 16) | 1u);
                    if (old == 0) {
                        s_claim[atomicAdd(&s_n, 1u)] = (uint16_t)idx;
                        break;
                    }
                    sl = old;
                }
                const int p = (int)(sl >> 16) - 1;
                bool eq = true;
#pragma unroll
                for (int j = 0; j < N; ++j) eq = eq && (s_tok[p + j] == s_tok[i + j]);
                if (eq) {
                    atomicAdd(&s_slot[idx], 1u);
                    break;
                }
                idx = (idx + 1) & (kLdsSlots - 1);
            }
        }
        __syncthreads();
        const int n_claim = (int)s_n;
        for (int e0 = tid; e0 < n_claim; e0 += kThreads * kInFlight) {
            int pos[kInFlight];
            u32 cnt[kInFlight];
            u64 idx[kInFlight], g[kInFlight];
            bool eq[kInFlight];
#pragma unroll
            for (int u = 0; u < kInFlight; ++u) {
                const int e = e0 + u * kThreads;
                pos[u] = -1;
                cnt[u] = 0;
                idx[u] = 0;
                g[u] = 0;
                if (e < n_claim) {
                    const int sidx = s_claim[e];
                    const u32 sl = s_slot[sidx];
                    s_slot[sidx] = 0;                  // ready for the next chunk
                    pos[u] = (int)(sl >> 16) - 1;
                    cnt[u] = sl & 0xFFFFu;
                    u64 lo = 0, hi = 0;
#pragma unroll
                    for (int j = 0; j < N; ++j) tasc_key_put(lo, hi, j, bits, (u32)s_tok[pos[u] + j]);
                    idx[u] = tasc_hash_key(lo, hi, N) & mask;
                    g[u] = __hip_atomic_load(&slots[idx[u]], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                }
            }
#pragma unroll
            for (int u = 0; u < kInFlight; ++u) {
                eq[u] = false;
                if (pos[u] >= 0 && g[u] != 0) {
                    const int32_t* w = tok + ((g[u] >> 32) - 1);
                    bool same = true;
#pragma unroll
                    for (int j = 0; j < N; ++j) same = same & (w[j] == s_tok[pos[u] + j]);
                    eq[u] = same;
                }
            }
#pragma unroll
            for (int u = 0; u < kInFlight; ++u) {
                if (pos[u] < 0) continue;
                bool reached = false;                  // this addition lifted the count to p_min
                for (u64 probe = 0; probe <= mask; ++probe) {
                    if (g[u] == 0) {
                        const u64 old = atomicCAS(&slots[idx[u]], 0ull, ((base + pos[u] + 1) << 32) | cnt[u]);
                        if (old == 0) {
                            ++distinct;
                            reached = cnt[u] >= p_min;
                            break;
                        }
                        g[u] = old;
                        eq[u] = true;
                        for (int j = 0; j < N; ++j) eq[u] = eq[u] && (tok[(g[u] >> 32) - 1 + j] == s_tok[pos[u] + j]);
                    }
                    if (eq[u]) {
                        if (list && p_min > 1) {
                            const u32 before = (u32)atomicAdd(&slots[idx[u]], (u64)cnt[u]);
                            reached = before < p_min && before + cnt[u] >= p_min;
                        } else {
                            atomicAdd(&slots[idx[u]], (u64)cnt[u]);
                        }
                        break;
                    }
                    idx[u] = (idx[u] + 1) & mask;
                    g[u] = __hip_atomic_load(&slots[idx[u]], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    eq[u] = false;
                    if (g[u] != 0) {
                        eq[u] = true;
                        for (int j = 0; j < N; ++j) eq[u] = eq[u] && (tok[(g[u] >> 32) - 1 + j] == s_tok[pos[u] + j]);
                    }
                }
                if (list && reached) {
                    const u32 at = atomicAdd(&s_nl, 1u);
                    if (at < kListed) {
                        s_list[at] = idx[u];
                    } else {                           // full (p_min 1 lists every n-gram): one addition for the lanes that are here
                        const u64 here = __ballot(1);
                        const int lane = tid & 63, lead = __ffsll((unsigned long long)here) - 1;
                        u64 first = 0;
                        if (lane == lead) first = atomicAdd(&counters[1], (u64)__popcll(here));
                        first = __shfl(first, lead);
                        list[first + __popcll(here & ((1ull << lane) - 1))] = idx[u];
                    }
                }
            }
        }
        __syncthreads();
        // the list is appended when it is half full, and with the last chunk
        const u32 nl = min(s_nl, (u32)kListed);
        const bool flush = list && nl > 0 && (nl >= kListed / 2 || base + (u64)gridDim.x * kChunk >= T);
        if (flush) {
            if (tid == 0) s_at = atomicAdd(&counters[1], (u64)nl);
            __syncthreads();
            for (u32 i = tid; i < nl; i += kThreads) list[s_at + i] = s_list[i];
        }
        __syncthreads();
        if (tid == 0) {
            s_n = 0;
            if (flush) s_nl = 0;
        }
    }
    for (int o = 32; o > 0; o >>= 1) distinct += __shfl_xor(distinct, o);
    __syncthreads();
    if ((tid & 63) == 0) s_slot[tid >> 6] = distinct;
    __syncthreads();
    if (tid == 0) {
        u64 n = 0;
        for (int w = 0; w < kThreads / 64; ++w) n += s_slot[w];
        if (n) atomicAdd(&counters[0], n);             // additions to one address cost 3 ns each: one per workgroup
    }
}

// the listed slots' contents (position + 1, final count) in their place
__global__ __launch_bounds__(kThreads) void k_collect(const u64* __restrict__ slots, const u64* __restrict__ counters, u64* list) {
    const u64 n = counters[1];
    for (u64 i = (u64)blockIdx.x * kThreads + threadIdx.x; i < n; i += (u64)gridDim.x * kThreads) list[i] = slots[list[i]];
}

struct CtxRef {   // context table under construction: key named by a corpus position
    u32 pos1;     // position + 1 of the context's first token, 0 = empty
    u32 total;    // T: sum of kept successor counts
    u64 best;     // max of (count << 32) | (0xFFFFFFFF - successor)
};

template <int N>
__global__ __launch_bounds__(kThreads) void k_keep(const int32_t* __restrict__ tok, const u64* __restrict__ kept,
                                                   u64 n_kept, int bits, TascSlot* full, u64 full_mask,
                                                   CtxRef* ctx, u64 ctx_mask) {
    u64 i = (u64)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n_kept) return;
    u64 s = kept[i];
    u32 cnt = (u32)s;
    u64 p = (s >> 32) - 1;
    int32_t w[N];
    u64 lo = 0, hi = 0, clo = 0, chi = 0;
#pragma unroll
    for (int j = 0; j < N; ++j) {
        w[j] = tok[p + j];
        tasc_key_put(lo, hi, j, bits, (u32)w[j]);
        if (j < N - 1) tasc_key_put(clo, chi, j, bits, (u32)w[j]);
    }
    // full table: keys are distinct, so claiming a slot (count 0 -> cnt) is all the synchronisation needed
    u64 idx = tasc_hash_key(lo, hi, N) & full_mask;
    for (u64 probe = 0; probe <= full_mask; ++probe) {
        if (atomicCAS(&full[idx].a, 0u, cnt) == 0u) {
            full[idx].lo = lo;
            full[idx].hi = hi;
            break;
        }
        idx = (idx + 1) & full_mask;
    }
    // context table: many kept n-grams share a context
    idx = tasc_hash_key(clo, chi, N - 1) & ctx_mask;
    for (u64 probe = 0; probe <= ctx_mask; ++probe) {
        u32 q = __hip_atomic_load(&ctx[idx].pos1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        bool mine = false;
        if (q == 0) {
            u32 old = atomicCAS(&ctx[idx].pos1, 0u, (u32)(p + 1));
            mine = old == 0;
            q = old;
        }
        if (mine || same_window<N - 1>(tok, (u64)q - 1, w)) {
            atomicAdd(&ctx[idx].total, cnt);
            atomicMax(&ctx[idx].best, ((u64)cnt << 32) | (u64)(0xFFFFFFFFu - (u32)w[N - 1]));
            break;
        }
        idx = (idx + 1) & ctx_mask;
    }
}

// gives every context slot its explicit key; same index, so the probe sequences stay valid
__global__ __launch_bounds__(kThreads) void k_materialize_ctx(const int32_t* __restrict__ tok, const CtxRef* ref, u64 cap, int n_ctx_tok,
                                  int bits, TascSlot* out, u64* n_contexts) {
    u32 n = 0;
    for (u64 i = (u64)blockIdx.x * kThreads + threadIdx.x; i < cap; i += (u64)gridDim.x * kThreads) {
        CtxRef r = ref[i];
        TascSlot s = {0, 0, 0, 0, 0, 0};
        if (r.pos1 != 0) {
            for (int j = 0; j < n_ctx_tok; ++j) tasc_key_put(s.lo, s.hi, j, bits, (u32)tok[(u64)r.pos1 - 1 + j]);
            s.a = r.total;
            s.b = 0xFFFFFFFFu - (u32)r.best;
            s.c = (u32)(r.best >> 32);
            ++n;
        }
        out[i] = s;
    }
    __shared__ u32 s_w[kThreads / 64];
    for (int o = 32; o > 0; o >>= 1) n += __shfl_xor(n, o);
    if ((threadIdx.x & 63) == 0) s_w[threadIdx.x >> 6] = n;
    __syncthreads();
    if (threadIdx.x == 0) {                            // one addition per workgroup, not per context
        u64 sum = 0;
        for (int w = 0; w < kThreads / 64; ++w) sum += s_w[w];
        if (sum) atomicAdd(n_contexts, sum);
    }
}

u64 pow2_at_least(u64 v) {
    u64 c = 1;
    while (c < v) c <<= 1;
    return c;
}

// a workgroup counts several chunks, so that it clears its LDS table once
unsigned count_grid(u64 T) { return (unsigned)std::min<u64>((T + kChunk - 1) / kChunk, 4096); }

#define TASC_BY_ORDER(n, call)                                                                                                  \
    switch (n) {                                                                                                                \
        case 2: call(2); break; case 3: call(3); break; case 4: call(4); break; case 5: call(5); break; case 6: call(6); break;  \
        case 7: call(7); break; default: call(8); break;                                                                        \
    }

// slots of the counting table of `windows` windows
u64 count_cap(u64 windows) { return pow2_at_least(std::max<u64>(1024, windows + windows / 2)); }

struct Cleanup {   // frees temporaries on every exit path
    std::vector<void*> ptrs;
    std::vector<hipEvent_t> evs;
    ~Cleanup() {
        for (void* p : ptrs) (void)hipFree(p);
        for (hipEvent_t e : evs) (void)hipEventDestroy(e);
    }
};

}  // namespace

extern "C" tasc_status tasc_ngram_build(const int32_t* tokens, const int64_t* doc_offsets, int64_t n_docs,
                                        int32_t vocab, int32_t n_max, int32_t p_min, tasc_mem where, void* stream,
                                        tasc_ngram** out) {
    TASC_REQUIRE(out != nullptr && doc_offsets != nullptr, "ngram_build: null argument");
    TASC_REQUIRE(n_docs >= 0 && vocab >= 1, "ngram_build: n_docs %lld, vocab %d", (long long)n_docs, vocab);
    TASC_REQUIRE(n_max >= 2 && n_max <= TASC_MAX_ORDER, "ngram_build: n_max %d outside [2, %d]", n_max, TASC_MAX_ORDER);
    TASC_REQUIRE(p_min >= 1, "ngram_build: p_min %d < 1", p_min);
    TASC_REQUIRE(where == TASC_MEM_HOST || where == TASC_MEM_DEVICE, "ngram_build: bad memory kind");
    int bits = 1;
    while ((1ll << bits) < vocab) ++bits;
    TASC_REQUIRE(n_max * bits <= 128, "ngram_build: n_max %d x %d bits per token exceeds the 128-bit key", n_max, bits);
    TASC_REQUIRE(doc_offsets[0] == 0, "ngram_build: doc_offsets[0] != 0");
    u64 windows[TASC_MAX_ORDER + 1] = {0};                     // per order, from the document lengths
    for (int64_t d = 0; d < n_docs; ++d) {
        const int64_t len = doc_offsets[d + 1] - doc_offsets[d];
        TASC_REQUIRE(len >= 0, "ngram_build: doc_offsets decrease at %lld", (long long)d);
        for (int n = 2; n <= n_max; ++n)
            if (len >= n) windows[n] += (u64)(len - n + 1);
    }
    const u64 T = (u64)doc_offsets[n_docs];
    TASC_REQUIRE(T < 0xFFFFFFFFull, "ngram_build: corpus of %llu tokens is too large", T);
    TASC_REQUIRE(T == 0 || tokens != nullptr, "ngram_build: null tokens");
    hipStream_t st = (hipStream_t)stream;

    Cleanup tmp;
    tasc_ngram* ng = new tasc_ngram();
    memset(&ng->view, 0, sizeof ng->view);
    memset(ng->slots, 0, sizeof ng->slots);
    memset(&ng->stats, 0, sizeof ng->stats);
    ng->unigram = nullptr;
    memset(ng->tables, 0, sizeof ng->tables);
    ng->p_min = p_min;
    ng->view.n_max = n_max;
    ng->view.bits = bits;
    ng->view.vocab = vocab;
    ng->view.fallback = 0;
    ng->stats.n_tokens = (int64_t)T;
    struct Guard {   // destroys the half-built handle unless released
        tasc_ngram* p;
        ~Guard() { if (p) tasc_ngram_destroy(p); }
    } guard{ng};
    hipEvent_t ev0, ev1, evc[TASC_MAX_ORDER + 1][2];
    auto event = [&](hipEvent_t* e) -> tasc_status {
        TASC_HIP(hipEventCreate(e));
        tmp.evs.push_back(*e);
        return TASC_OK;
    };
#define TASC_TRY(expr) do { tasc_status _rc = (expr); if (_rc != TASC_OK) return _rc; } while (0)
    TASC_TRY(event(&ev0));
    TASC_TRY(event(&ev1));

    // One block for everything that is only needed here: counters ([n][0] distinct, [n][1] kept, [n][2] contexts of order n;
    // [0][3] unigram best, [0][4] bad-token flag), document ends, counting table, kept n-grams of every order (their counts add
    // up to the windows, so there are at most windows / p_min), a host corpus.  The orders go through in groups whose lists
    // take no more than TASC_CFG_BUILD_LIST_KIB (one group but for corpora of a billion tokens), each with one look at its counts.
    size_t used = 0;
    auto carve = [&](size_t bytes) { const size_t at = used; used += (bytes + 255) / 256 * 256; return at; };
    const size_t at_counters = carve((TASC_MAX_ORDER + 1) * 8 * sizeof(u64));
    const size_t at_copies = carve(T > 0 ? (size_t)vocab * sizeof(u32) * kUniCopies : 0);
    const bool any = windows[2] > 0;
    const u64 slots_cap = any ? count_cap(windows[2]) : 0;     // windows[n] falls with n
    const size_t at_rem = carve(any ? T : 0), at_off = carve(any ? (size_t)(n_docs + 1) * sizeof(int64_t) : 0);
    const size_t at_slots = carve(slots_cap * sizeof(u64));
    const size_t list_bytes = (size_t)g_tasc_config.build_list_kib << 10;
    size_t at_list[TASC_MAX_ORDER + 1] = {0}, lists = 0, longest = 0;
    int group_end[TASC_MAX_ORDER + 2] = {0};                   // [n] = one past the last order of the group that n begins
    for (int n = 2, first = 2; n <= n_max; ++n) {
        const size_t bytes = (windows[n] / (u64)p_min * sizeof(u64) + 255) / 256 * 256;
        if (n > first && lists + bytes > list_bytes) {
            first = n;
            lists = 0;
        }
        at_list[n] = lists;
        lists += bytes;
        longest = std::max(longest, lists);
        group_end[first] = n + 1;
    }
    const size_t at_lists = carve(longest);
    for (int n = 2; n <= n_max; ++n) at_list[n] += at_lists;
    const size_t at_tok = carve(where == TASC_MEM_HOST ? T * sizeof(int32_t) : 0);
    char* arena;
    TASC_HIP(hipMalloc((void**)&arena, used)); tmp.ptrs.push_back(arena);
    u64 (*d_counters)[8] = (u64(*)[8])(arena + at_counters);
    u64 h_counters[TASC_MAX_ORDER + 1][8];
    memset(h_counters, 0, sizeof h_counters);
    TASC_HIP(hipMalloc((void**)&ng->unigram, (size_t)vocab * sizeof(u32)));

    const int32_t* d_tok = tokens;
    if (where == TASC_MEM_HOST && T > 0) {
        TASC_HIP(hipMemcpyAsync(arena + at_tok, tokens, T * sizeof(int32_t), hipMemcpyHostToDevice, st));
        d_tok = (const int32_t*)(arena + at_tok);
    }
    TASC_HIP(hipEventRecord(ev0, st));
    u32* const d_copies = (u32*)(arena + at_copies);
    TASC_HIP(hipMemsetAsync(T > 0 ? d_copies : ng->unigram, 0, (size_t)vocab * sizeof(u32) * (T > 0 ? kUniCopies : 1), st));
    TASC_HIP(hipMemsetAsync(d_counters, 0, sizeof h_counters, st));
    if (T > 0) {
        unsigned grid = (unsigned)std::min<u64>((T + kUniChunk - 1) / kUniChunk, 2048);
        k_unigram<<<dim3(grid), dim3(kThreads), 0, st>>>(d_tok, T, vocab, d_copies, (u32*)&d_counters[0][4]);
        TASC_LAUNCH_CHECK();
        k_unigram_argmax<<<dim3(64), dim3(kThreads), 0, st>>>(d_copies, vocab, ng->unigram, &d_counters[0][3]);
        TASC_LAUNCH_CHECK();
    }
    uint8_t* const d_rem = (uint8_t*)(arena + at_rem);
    u64* const d_slots = (u64*)(arena + at_slots);
    if (any) {
        int64_t* const d_off = (int64_t*)(arena + at_off);
        TASC_HIP(hipMemcpyAsync(d_off, doc_offsets, (size_t)(n_docs + 1) * sizeof(int64_t), hipMemcpyHostToDevice, st));
        TASC_TRY(tasc_mark_tails(d_off, n_docs, n_max, T, d_rem, st));
    }
    for (int n0 = 2; n0 <= n_max; n0 = group_end[n0]) {
        // every order of the group in turn through the one counting table (a token outside the vocabulary only spoils its key;
        // it is reported below)
        for (int n = n0; n < group_end[n0]; ++n) {
            ng->stats.windows[n] = (int64_t)windows[n];
            if (windows[n] == 0) continue;
            TASC_TRY(event(&evc[n][0]));
            TASC_TRY(event(&evc[n][1]));
            u64* const list = (u64*)(arena + at_list[n]);
            const u64 cap = count_cap(windows[n]);
            TASC_HIP(hipMemsetAsync(d_slots, 0, cap * sizeof(u64), st));
            TASC_HIP(hipEventRecord(evc[n][0], st));
#define CALL(N) k_count<N><<<dim3(count_grid(T)), dim3(kThreads), 0, st>>>(d_tok, d_rem, T, bits, d_slots, cap - 1, (u32)p_min, d_counters[n], list)
            TASC_BY_ORDER(n, CALL)
#undef CALL
            TASC_LAUNCH_CHECK();
            TASC_HIP(hipEventRecord(evc[n][1], st));
            k_collect<<<dim3(1024), dim3(kThreads), 0, st>>>(d_slots, d_counters[n], list);
            TASC_LAUNCH_CHECK();
        }
        TASC_HIP(hipMemcpyAsync(h_counters, d_counters, sizeof h_counters, hipMemcpyDeviceToHost, st));
        TASC_HIP(hipStreamSynchronize(st));
        TASC_REQUIRE(h_counters[0][4] == 0, "ngram_build: corpus holds a token outside [0, %d)", vocab);
        // the finished tables of the group in one block; their context tables are built in the counting table's memory
        u64 fcap[TASC_MAX_ORDER + 1] = {0}, total = 0, most = 0;
        for (int n = n0; n < group_end[n0]; ++n) {
            ng->stats.distinct[n] = (int64_t)h_counters[n][0];
            ng->stats.kept[n] = (int64_t)h_counters[n][1];
            if (h_counters[n][1] == 0) continue;
            fcap[n] = pow2_at_least(std::max<u64>(64, 2 * h_counters[n][1]));
            total += 2 * fcap[n];
            most = std::max(most, fcap[n]);
        }
        if (total == 0) continue;
        TASC_HIP(hipMalloc((void**)&ng->tables[n0], total * sizeof(TascSlot)));
        CtxRef* ref = (CtxRef*)d_slots;
        if (most * sizeof(CtxRef) > slots_cap * sizeof(u64)) {
            TASC_HIP(hipMalloc((void**)&ref, most * sizeof(CtxRef)));
            tmp.ptrs.push_back(ref);
        }
        TascSlot* at = ng->tables[n0];
        for (int n = n0; n < group_end[n0]; ++n) {
            if (fcap[n] == 0) continue;
            TascSlot *full = at, *ctx = at + fcap[n];
            at += 2 * fcap[n];
            TASC_HIP(hipMemsetAsync(full, 0, fcap[n] * sizeof(TascSlot), st));
            TASC_HIP(hipMemsetAsync(ref, 0, fcap[n] * sizeof(CtxRef), st));
            const u64 kept = h_counters[n][1];
            const u64* list = (const u64*)(arena + at_list[n]);
#define CALL(N) k_keep<N><<<dim3((unsigned)((kept + kThreads - 1) / kThreads)), dim3(kThreads), 0, st>>>(d_tok, list, kept, bits, full, fcap[n] - 1, ref, fcap[n] - 1)
            TASC_BY_ORDER(n, CALL)
#undef CALL
            TASC_LAUNCH_CHECK();
            k_materialize_ctx<<<dim3((unsigned)std::min<u64>((fcap[n] + kThreads - 1) / kThreads, 2048)), dim3(kThreads), 0, st>>>(
                d_tok, ref, fcap[n], n - 1, bits, ctx, &d_counters[n][2]);
            TASC_LAUNCH_CHECK();
            ng->slots[n][0] = ctx;
            ng->slots[n][1] = full;
            ng->view.ord[n].ctx = ctx;
            ng->view.ord[n].full = full;
            ng->view.ord[n].ctx_mask = ng->view.ord[n].full_mask = fcap[n] - 1;
        }
    }
    if (T > 0) ng->view.fallback = (int32_t)(0xFFFFFFFFu - (u32)h_counters[0][3]);
    TASC_HIP(hipMemcpyAsync(h_counters, d_counters, sizeof h_counters, hipMemcpyDeviceToHost, st));
    TASC_HIP(hipEventRecord(ev1, st));
    TASC_HIP(hipStreamSynchronize(st));
    float ms = 0.f;
    for (int n = 2; n <= n_max; ++n) {
        ng->stats.contexts[n] = (int64_t)h_counters[n][2];
        if (windows[n] == 0) continue;
        TASC_HIP(hipEventElapsedTime(&ms, evc[n][0], evc[n][1]));
        ng->stats.count_ms += ms;
    }
    TASC_HIP(hipEventElapsedTime(&ms, ev0, ev1));
    ng->stats.build_ms = ms;
    guard.p = nullptr;
    *out = ng;
    return TASC_OK;
}

tasc_status tasc_mark_tails(const int64_t* d_off, int64_t n_docs, int32_t n_max, u64 T, uint8_t* d_rem, hipStream_t st) {
    TASC_HIP(hipMemsetAsync(d_rem, 0xFF, T, st));
    if (n_docs > 0) k_mark_doc_tails<<<dim3((unsigned)((n_docs + kThreads - 1) / kThreads)), dim3(kThreads), 0, st>>>(d_off, n_docs, n_max, d_rem);
    TASC_LAUNCH_CHECK();
    return TASC_OK;
}

u64 tasc_count_cap(u64 windows) { return count_cap(windows); }

tasc_status tasc_count_order(const int32_t* d_tok, const uint8_t* d_rem, u64 T, int32_t n, int32_t bits, u64* d_slots, u64 cap, u64* d_counters,
                             hipStream_t st) {
    TASC_HIP(hipMemsetAsync(d_slots, 0, cap * sizeof(u64), st));
#define CALL(N) k_count<N><<<dim3(count_grid(T)), dim3(kThreads), 0, st>>>(d_tok, d_rem, T, bits, d_slots, cap - 1, 1u, d_counters, (u64*)nullptr)
    TASC_BY_ORDER(n, CALL)
#undef CALL
    TASC_LAUNCH_CHECK();
    return TASC_OK;
}

extern "C" void tasc_ngram_destroy(tasc_ngram* ng) {
    if (!ng) return;
    for (TascSlot* t : ng->tables)
        if (t) (void)hipFree(t);
    if (ng->unigram) (void)hipFree(ng->unigram);
    delete ng;
}

namespace {
// downloads the occupied slots of one table, sorted by their token strings
tasc_status fetch_sorted(const tasc_ngram* ng, int order, int which, int ntok, std::vector<TascSlot>& rows) {
    rows.clear();
    const TascSlot* d = ng->slots[order][which];
    if (!d) return TASC_OK;
    u64 cap = (which == 0 ? ng->view.ord[order].ctx_mask : ng->view.ord[order].full_mask) + 1;
    std::vector<TascSlot> all(cap);
    TASC_HIP(hipMemcpy(all.data(), d, cap * sizeof(TascSlot), hipMemcpyDeviceToHost));
    for (const TascSlot& s : all)
        if (s.a != 0) rows.push_back(s);
    const int bits = ng->view.bits;
    std::sort(rows.begin(), rows.end(), [=](const TascSlot& x, const TascSlot& y) {
        for (int j = 0; j < ntok; ++j) {
            u32 a = tasc_key_get(x.lo, x.hi, j, bits), b = tasc_key_get(y.lo, y.hi, j, bits);
            if (a != b) return a < b;
        }
        return false;
    });
    return TASC_OK;
}
}  // namespace

extern "C" tasc_status tasc_ngram_export(const tasc_ngram* ng, int32_t order, int32_t* ctx_next, uint32_t* counts,
                                         int64_t* n_inout) {
    TASC_REQUIRE(ng && n_inout, "ngram_export: null argument");
    TASC_REQUIRE(order >= 2 && order <= ng->view.n_max, "ngram_export: order %d outside [2, %d]", order, ng->view.n_max);
    const int64_t kept = ng->stats.kept[order];
    const int64_t cap = *n_inout;
    *n_inout = kept;
    if (!ctx_next && !counts) return TASC_OK;
    TASC_REQUIRE(ctx_next && counts, "ngram_export: one output array is null");
    if (cap < kept) {
        tasc_set_error("ngram_export: room for %lld rows, %lld needed", (long long)cap, (long long)kept);
        return TASC_ENOMEM;
    }
    std::vector<TascSlot> rows;
    tasc_status rc = fetch_sorted(ng, order, 1, order, rows);
    if (rc != TASC_OK) return rc;
    if ((int64_t)rows.size() != kept) {
        tasc_set_error("ngram_export: table holds %zu rows, expected %lld", rows.size(), (long long)kept);
        return TASC_ESTATE;
    }
    for (size_t i = 0; i < rows.size(); ++i) {
        for (int j = 0; j < order; ++j)
            ctx_next[i * order + j] = (int32_t)tasc_key_get(rows[i].lo, rows[i].hi, j, ng->view.bits);
        counts[i] = rows[i].a;
    }
    return TASC_OK;
}

extern "C" tasc_status tasc_ngram_export_contexts(const tasc_ngram* ng, int32_t order, int32_t* ctx, uint32_t* total,
                                                  int32_t* top, uint32_t* top_count, int64_t* n_inout) {
    TASC_REQUIRE(ng && n_inout, "ngram_export_contexts: null argument");
    TASC_REQUIRE(order >= 2 && order <= ng->view.n_max, "ngram_export_contexts: order %d outside [2, %d]", order,
                 ng->view.n_max);
    const int64_t n = ng->stats.contexts[order];
    const int64_t cap = *n_inout;
    *n_inout = n;
    if (!ctx && !total && !top && !top_count) return TASC_OK;
    TASC_REQUIRE(ctx && total && top && top_count, "ngram_export_contexts: one output array is null");
    if (cap < n) {
        tasc_set_error("ngram_export_contexts: room for %lld rows, %lld needed", (long long)cap, (long long)n);
        return TASC_ENOMEM;
    }
    std::vector<TascSlot> rows;
    tasc_status rc = fetch_sorted(ng, order, 0, order - 1, rows);
    if (rc != TASC_OK) return rc;
    if ((int64_t)rows.size() != n) {
        tasc_set_error("ngram_export_contexts: table holds %zu rows, expected %lld", rows.size(), (long long)n);
        return TASC_ESTATE;
    }
    for (size_t i = 0; i < rows.size(); ++i) {
        for (int j = 0; j < order - 1; ++j)
            ctx[i * (order - 1) + j] = (int32_t)tasc_key_get(rows[i].lo, rows[i].hi, j, ng->view.bits);
        total[i] = rows[i].a;
        top[i] = (int32_t)rows[i].b;
        top_count[i] = rows[i].c;
    }
    return TASC_OK;
}

extern "C" tasc_status tasc_ngram_unigram(const tasc_ngram* ng, int32_t* fallback, uint32_t* counts) {
    TASC_REQUIRE(ng, "ngram_unigram: null handle");
    if (counts) TASC_HIP(hipMemcpy(counts, ng->unigram, (size_t)ng->view.vocab * sizeof(u32), hipMemcpyDeviceToHost));
    if (fallback) *fallback = ng->view.fallback;
    return TASC_OK;
}

extern "C" tasc_status tasc_ngram_get_stats(const tasc_ngram* ng, tasc_ngram_stats* out) {
    TASC_REQUIRE(ng && out, "ngram_get_stats: null argument");
    *out = ng->stats;
    return TASC_OK;
}
