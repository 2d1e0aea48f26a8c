// Corpus n-gram tables on the GPU: counting, pruning, per-context aggregates, export.
//
// Paper, section "Proposed Method: TASC-spec": the drafter is a collection of n-gram models M_n,
// n <= n_max, each derived from the n-gram frequencies in the task corpus and pruned of the
// elements whose frequency is below p_min; the most frequent token is the last resort.
//
// All integer, exact keys.  The counts of an order come from count.hip as a list of the n-grams that reach p_min, with packed
// 128-bit keys; the list is inserted into two small tables of 32-byte slots (see TascSlot): the full table (context + successor ->
// count) and the context table (context -> T, most frequent successor).
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

// Token histogram.  Additions to counters in memory are what it would wait for (20 G/s, and hot tokens serialise), so a workgroup
// counts a slice of the corpus in LDS, for one range of the vocabulary, and writes its counters out: the ranges' workgroups of a
// slice read it from one L2.  32 M tokens, vocabulary 151,936 (five ranges): 103 us, 767 with additions to memory
// (k_unigram).
constexpr int kUniThreads = 1024, kUniRange = 36864, kUniRanges = 32, kUniSlice = 32768;   // 144 KB of counters
constexpr int kUniCopies = 8;
__global__ __launch_bounds__(kUniThreads) void k_unigram_range(const int32_t* __restrict__ tok, u64 T, int vocab, int ranges, int range, u64 slice,
                                                               u32* __restrict__ copies, u32* bad) {
    extern __shared__ u32 s_cnt[];
    // (ids are dealt to the 8 XCDs in turn: the ranges of a slice side by side on one of them)
    const u32 j = blockIdx.x / 8, r = j % ranges, sl = j / ranges * 8 + blockIdx.x % 8;
    const u32 first = r * range, n = min((u32)range, (u32)vocab - first);
    for (u32 i = threadIdx.x; i < n; i += kUniThreads) s_cnt[i] = 0;
    __syncthreads();
    const u64 b = min(T, sl * slice), e = min(T, b + slice);
    bool out = false;
    for (u64 i0 = b + threadIdx.x; i0 < e; i0 += kUniThreads * 8) {
        u32 t[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) t[u] = i0 + u * kUniThreads < e ? (u32)tok[i0 + u * kUniThreads] : first;
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            out = out || t[u] >= (u32)vocab;
            if (t[u] - first < n && i0 + u * kUniThreads < e) atomicAdd(&s_cnt[t[u] - first], 1u);
        }
    }
    if (out) atomicOr(bad, 1u);
    __syncthreads();
    for (u32 i = threadIdx.x; i < n; i += kUniThreads) copies[(size_t)sl * vocab + first + i] = s_cnt[i];
}

// Larger vocabularies, which would be read too often that way: a workgroup first counts a chunk of kUniChunk tokens in an LDS table
// (open addressing, twice as many slots as tokens, so it cannot fill up) and then adds each distinct token's count to a
// histogram in memory once: one of kUniCopies, by workgroup id, and so one per XCD, whose lines stay in that XCD's L2.
constexpr int kUniChunk = 2048, kUniSlots = 4096;
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
__global__ __launch_bounds__(kThreads) void k_unigram_argmax(const u32* copies, int n_copies, int vocab, u32* hist, u64* best) {
    u64 v = 0;
    for (u32 i = blockIdx.x * blockDim.x + threadIdx.x; i < (u32)vocab; i += gridDim.x * blockDim.x) {
        u32 n = 0;
#pragma unroll 8
        for (int q = 0; q < n_copies; ++q) n += copies[(size_t)q * vocab + i];
        hist[i] = n;
        u64 c = ((u64)n << 32) | (u64)(0xFFFFFFFFu - i);
        v = c > v ? c : v;
    }
    for (int o = 32; o > 0; o >>= 1) {
        u64 w = __shfl_xor(v, o);
        v = w > v ? w : v;
    }
    // (additions and maxima to one address take 9 ns each, whoever makes them: a wave's each were 21 of 32 us at 151,936 tokens)
    __shared__ u64 s_v[kThreads / 64];
    if ((threadIdx.x & 63) == 0) s_v[threadIdx.x >> 6] = v;
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < kThreads / 64; ++w) v = s_v[w] > v ? s_v[w] : v;
        atomicMax(best, v);
    }
}

__global__ void k_mark_doc_ends(const int64_t* doc_off, int64_t n_docs, uint8_t* last) {
    const int64_t d = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (d < n_docs && doc_off[d] < doc_off[d + 1]) last[doc_off[d + 1] - 1] = 1;
}

struct CtxRef {   // context table under construction: key named by a kept n-gram
    u32 ref1;     // its place in the list + 1, 0 = empty
    u32 total;    // T: sum of kept successor counts
    u64 best;     // max of (count << 32) | (0xFFFFFFFF - successor)
};
// key of an n-gram's first m tokens
__device__ inline void key_head(u64& lo, u64& hi, int m, int bits) {
    const int b = m * bits;
    if (b < 64) lo &= (1ull << b) - 1;
    hi = b > 64 ? hi & ((1ull << (b - 64)) - 1) : 0;
}

// The finished tables of several orders in three launches, whose chains of dependent round trips (a probe each) run beside each other: one order has
// 130 to 280 workgroups of them, half the chip's room, and their longest lanes decide.  The keys and their contexts, 32 M tokens, orders 2 to 5, with
// clearing and k_materialize_ctx: 405 us order by order, 212 so (k_keep 166: about the rate of its atomics).
struct Finish {
    TascKept kept;
    u64 n_kept;
    TascSlot *full, *ctx;
    CtxRef* ref;
    u64 cap;                   // slots of each table
    u64* n_contexts;
    int32_t n;
    u32 first;                 // k_keep: the order's first workgroup
};
struct FinishAll {
    Finish order[TASC_MAX_ORDER - 1];
    int32_t orders, bits;
};

__global__ __launch_bounds__(kThreads) void k_clear_tables(FinishAll all) {
    const Finish& f = all.order[blockIdx.y];
    static_assert(sizeof(TascSlot) == 32 && sizeof(CtxRef) == 16, "16 bytes a store");
    uint4 *const full = reinterpret_cast<uint4*>(f.full), *const ref = reinterpret_cast<uint4*>(f.ref);
    for (u64 i = (u64)blockIdx.x * kThreads + threadIdx.x; i < f.cap; i += (u64)gridDim.x * kThreads) {
        full[i] = make_uint4(0, 0, 0, 0);
        full[f.cap + i] = make_uint4(0, 0, 0, 0);
        ref[i] = make_uint4(0, 0, 0, 0);
    }
}

// Kept n-grams -> full table, and their contexts -> context table.  Frequent contexts have thousands of kept successors, whose
// additions to one slot would wait for each other (32 M tokens, orders 2 to 5: 220 us an order); a workgroup merges those
// of its kThreadsKeep n-grams in LDS first: 34 to 70 us an order alone.
constexpr int kThreadsKeep = 1024;
__global__ __launch_bounds__(kThreadsKeep) void k_keep(FinishAll all) {
    int o = 0;
    while (o + 1 < all.orders && blockIdx.x >= all.order[o + 1].first) ++o;
    const Finish& f = all.order[o];
    const TascKept kept = f.kept;
    const u64 n_kept = f.n_kept, full_mask = f.cap - 1, ctx_mask = f.cap - 1;
    const int n = f.n, bits = all.bits;
    TascSlot* const full = f.full;
    CtxRef* const ctx = f.ref;
    constexpr int SLOTS = 2 * kThreadsKeep;
    __shared__ u64 s_lo[kThreadsKeep], s_hi[kThreadsKeep], s_best[SLOTS];
    __shared__ u32 s_ref[SLOTS], s_total[SLOTS];
    const int tid = threadIdx.x;
    const u64 i = (u64)(blockIdx.x - f.first) * kThreadsKeep + tid;
    for (int q = tid; q < SLOTS; q += kThreadsKeep) { s_ref[q] = 0; s_total[q] = 0; s_best[q] = 0; }
    const bool on = i < n_kept;
    u64 lo = on ? kept.lo[i] : 0, hi = on ? kept.hi[i] : 0;
    const u32 cnt = on ? kept.count[i] : 0;
    if (on) {
        // full table: keys are distinct, so claiming a slot (count 0 -> cnt) is all the synchronisation needed
        u64 idx = tasc_slot_of(tasc_hash_key(lo, hi), full_mask);
        for (u64 probe = 0; probe <= full_mask; ++probe) {
            if (atomicCAS(&full[idx].a, 0u, cnt) == 0u) {
                full[idx].lo = lo;
                full[idx].hi = hi;
                break;
            }
            idx = (idx + 1) & full_mask;
        }
    }
    const u32 succ = tasc_key_get(lo, hi, n - 1, bits);
    key_head(lo, hi, n - 1, bits);
    s_lo[tid] = lo;
    s_hi[tid] = hi;
    __syncthreads();
    const u64 hash = tasc_hash_key(lo, hi);
    int own = -1;
    if (on) {
        u32 at = (u32)(hash >> 40) & (SLOTS - 1);
        for (int probe = 0; probe < SLOTS; ++probe) {
            u32 r = s_ref[at];
            if (r == 0) {
                r = atomicCAS(&s_ref[at], 0u, (u32)tid + 1);
                if (r == 0) {
                    own = (int)at;
                    r = tid + 1;
                }
            }
            if (s_lo[r - 1] == lo && s_hi[r - 1] == hi) {
                atomicAdd(&s_total[at], cnt);
                atomicMax(&s_best[at], ((u64)cnt << 32) | (u64)(0xFFFFFFFFu - succ));
                break;
            }
            at = (at + 1) & (SLOTS - 1);
        }
    }
    __syncthreads();
    if (own < 0) return;
    u64 idx = tasc_slot_of(hash, ctx_mask);
    for (u64 probe = 0; probe <= ctx_mask; ++probe) {
        u32 q = __hip_atomic_load(&ctx[idx].ref1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (q == 0) q = atomicCAS(&ctx[idx].ref1, 0u, (u32)(i + 1));
        u64 qlo = lo, qhi = hi;
        if (q != 0) {
            qlo = kept.lo[q - 1];
            qhi = kept.hi[q - 1];
            key_head(qlo, qhi, n - 1, bits);
        }
        if (qlo == lo && qhi == hi) {
            atomicAdd(&ctx[idx].total, s_total[own]);
            atomicMax(&ctx[idx].best, s_best[own]);
            break;
        }
        idx = (idx + 1) & ctx_mask;
    }
}

// gives every context slot its explicit key; same index, so the probe sequences stay valid.  Few and large workgroups: each adds once to the order's
// number of contexts, and 2048 of 256 threads an order waited for that longer than for the tables (62 us, 32 so, four orders of 0.5 M to 1 M slots).
constexpr int kThreadsCtx = 1024, kGroupsCtx = 256;
__global__ __launch_bounds__(kThreadsCtx) void k_materialize_ctx(FinishAll all) {
    const Finish& f = all.order[blockIdx.y];
    const TascKept kept = f.kept;
    const CtxRef* const ref = f.ref;
    const u64 cap = f.cap;
    const int n_ctx_tok = f.n - 1, bits = all.bits;
    TascSlot* const out = f.ctx;
    u64* const n_contexts = f.n_contexts;
    u32 n = 0;
    for (u64 i = (u64)blockIdx.x * kThreadsCtx + threadIdx.x; i < cap; i += (u64)gridDim.x * kThreadsCtx) {
        CtxRef r = ref[i];
        TascSlot s = {0, 0, 0, 0, 0, 0};
        if (r.ref1 != 0) {
            s.lo = kept.lo[r.ref1 - 1];
            s.hi = kept.hi[r.ref1 - 1];
            key_head(s.lo, s.hi, n_ctx_tok, bits);
            s.a = r.total;
            s.b = 0xFFFFFFFFu - (u32)r.best;
            s.c = (u32)(r.best >> 32);
            ++n;
        }
        out[i] = s;
    }
    __shared__ u32 s_w[kThreadsCtx / 64];
    for (int o = 32; o > 0; o >>= 1) n += __shfl_xor(n, o);
    if ((threadIdx.x & 63) == 0) s_w[threadIdx.x >> 6] = n;
    __syncthreads();
    if (threadIdx.x == 0) {                            // one addition per workgroup, not per context
        u64 sum = 0;
        for (int w = 0; w < kThreadsCtx / 64; ++w) sum += s_w[w];
        if (sum) atomicAdd(n_contexts, sum);
    }
}

u64 pow2_at_least(u64 v) {
    u64 c = 1;
    while (c < v) c <<= 1;
    return c;
}

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
    u64 windows[TASC_MAX_ORDER + 1] = {0};                     // per order, from the document lengths: first what short documents lack
    for (int64_t d = 0; d < n_docs; ++d) {
        const int64_t len = doc_offsets[d + 1] - doc_offsets[d];
        if (len >= n_max - 1) continue;
        TASC_REQUIRE(len >= 0, "ngram_build: doc_offsets decrease at %lld", (long long)d);
        for (int n = 2; n <= n_max; ++n) windows[n] += (u64)std::max<int64_t>(0, n - 1 - len);
    }
    const u64 T = (u64)doc_offsets[n_docs];
    TASC_REQUIRE(T < 0xFFFFFFFFull, "ngram_build: corpus of %llu tokens is too large", T);
    TASC_REQUIRE(T == 0 || tokens != nullptr, "ngram_build: null tokens");
    for (int n = 2; n <= n_max; ++n) windows[n] += T - (u64)(n - 1) * (u64)n_docs;
    hipStream_t st = (hipStream_t)stream;

    Cleanup tmp;
    TascScratch scratch;
    tasc_ngram* ng = new tasc_ngram();
    tasc_handles_add(1);
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
    // [0][3] unigram best, [0][4] bad-token flag), document ends, an order's records, kept n-grams of every order (their counts add
    // up to the windows, so there are at most windows / p_min), a host corpus.  The orders go through in groups whose lists
    // take no more than TASC_CFG_BUILD_LIST_KIB (one group but for corpora of hundreds of millions of tokens), each with one look at
    // its counts.
    size_t used = 0;
    auto carve = [&](size_t bytes) { const size_t at = used; used += (bytes + 255) / 256 * 256; return at; };
    const size_t at_counters = carve((TASC_MAX_ORDER + 1) * 8 * sizeof(u64));
    const int uni_ranges = (int)(((int64_t)vocab + kUniRange - 1) / kUniRange), uni_range = (int)(((int64_t)vocab + uni_ranges - 1) / uni_ranges);
    // slices of kUniSlice tokens or more, eight at a time and no more workgroups than a round
    const u32 uni_slices = uni_ranges > kUniRanges ? kUniCopies : 8 * (u32)std::clamp<u64>((T + 8 * kUniSlice - 1) / (8 * kUniSlice), 1, std::max(1, 32 / uni_ranges));
    const size_t at_copies = carve(T > 0 ? (size_t)vocab * sizeof(u32) * uni_slices : 0);
    const bool any = windows[2] > 0;
    const size_t at_last = carve(any ? T : 0), at_off = carve(any ? (size_t)(n_docs + 1) * sizeof(int64_t) : 0);
    // (with p_min 1 every n-gram is kept, the unique ones too)
    const bool prune = p_min > 1;
    size_t rec_bytes = 0, offs_bytes = 0, deal_bytes = 0;
    for (int n = 2; n <= n_max; ++n) {
        if (windows[n] == 0) continue;
        const TascCountPlan p = tasc_count_plan(T, windows[n], n * bits > 64, prune && n > 2);
        rec_bytes = std::max(rec_bytes, p.rec_bytes);
        offs_bytes = std::max(offs_bytes, p.offs_bytes);
        deal_bytes = std::max(deal_bytes, p.deal_bytes);
    }
    const size_t at_rec = carve(rec_bytes), at_roff = carve(offs_bytes), at_deal = carve(deal_bytes), twice_bytes = any && prune ? ((size_t)1 << tasc_twice_bits(T)) / 8 : 0, at_twice = carve(2 * twice_bytes);
    const size_t list_bytes = (size_t)g_tasc_config.build_list_kib << 10;
    size_t at_list[TASC_MAX_ORDER + 1] = {0}, lists = 0, longest = 0;
    int group_end[TASC_MAX_ORDER + 2] = {0};                   // [n] = one past the last order of the group that n begins
    for (int n = 2, first = 2; n <= n_max; ++n) {
        const size_t bytes = (windows[n] / (u64)p_min * (2 * sizeof(u64) + sizeof(u32)) + 255) / 256 * 256;
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
    TASC_TRY(scratch.get(used));
    char* const arena = scratch.p;
    u64 (*d_counters)[8] = (u64(*)[8])(arena + at_counters);
    u64 h_counters[TASC_MAX_ORDER + 1][8];
    memset(h_counters, 0, sizeof h_counters);
    TASC_TRY(tasc_device_malloc((void**)&ng->unigram, (size_t)vocab * sizeof(u32)));

    const int32_t* d_tok = tokens;
    if (where == TASC_MEM_HOST && T > 0) {
        TASC_HIP(hipMemcpyAsync(arena + at_tok, tokens, T * sizeof(int32_t), hipMemcpyHostToDevice, st));
        d_tok = (const int32_t*)(arena + at_tok);
    }
    TASC_HIP(hipEventRecord(ev0, st));
    u32* const d_copies = (u32*)(arena + at_copies);
    TASC_HIP(hipMemsetAsync(d_counters, 0, sizeof h_counters, st));
    if (T == 0) {
        TASC_HIP(hipMemsetAsync(ng->unigram, 0, (size_t)vocab * sizeof(u32), st));
    } else {
        if (uni_ranges <= kUniRanges) {
            TASC_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(k_unigram_range), hipFuncAttributeMaxDynamicSharedMemorySize, kUniRange * 4));
            k_unigram_range<<<dim3(uni_slices * uni_ranges), dim3(kUniThreads), uni_range * 4, st>>>(
                d_tok, T, vocab, uni_ranges, uni_range, (T + uni_slices - 1) / uni_slices, d_copies, (u32*)&d_counters[0][4]);
        } else {
            TASC_HIP(hipMemsetAsync(d_copies, 0, (size_t)vocab * sizeof(u32) * kUniCopies, st));
            const unsigned grid = (unsigned)std::min<u64>((T + kUniChunk - 1) / kUniChunk, 2048);
            k_unigram<<<dim3(grid), dim3(kThreads), 0, st>>>(d_tok, T, vocab, d_copies, (u32*)&d_counters[0][4]);
        }
        TASC_LAUNCH_CHECK();
        k_unigram_argmax<<<dim3((unsigned)std::min<int64_t>(((int64_t)vocab + kThreads - 1) / kThreads, 1024)), dim3(kThreads), 0, st>>>(
            d_copies, (int)uni_slices, vocab, ng->unigram, &d_counters[0][3]);
        TASC_LAUNCH_CHECK();
    }
    uint8_t* const d_last = (uint8_t*)(arena + at_last);
    const TascCountBufs bufs{(u64*)(arena + at_rec), (uint16_t*)(arena + at_roff), (u64*)(arena + at_deal)};
    auto kept_of = [&](int n) {
        u64* const lo = (u64*)(arena + at_list[n]);
        const size_t most = windows[n] / (u64)p_min;
        return TascKept{lo, lo + most, (u32*)(lo + 2 * most)};
    };
    if (any) {
        int64_t* const d_off = (int64_t*)(arena + at_off);
        TASC_HIP(hipMemcpyAsync(d_off, doc_offsets, (size_t)(n_docs + 1) * sizeof(int64_t), hipMemcpyHostToDevice, st));
        TASC_TRY(tasc_mark_ends(d_off, n_docs, T, d_last, st));
    }
    for (int n0 = 2; n0 <= n_max; n0 = group_end[n0]) {
        // every order of the group in turn through the one set of records (a token outside the vocabulary only spoils its key;
        // it is reported below)
        for (int n = n0; n < group_end[n0]; ++n) {
            ng->stats.windows[n] = (int64_t)windows[n];
            if (windows[n] == 0) continue;
            TASC_TRY(event(&evc[n][0]));
            TASC_TRY(event(&evc[n][1]));
            const TascCountPlan p = tasc_count_plan(T, windows[n], n * bits > 64, prune && n > 2);
            // the map of the order below is read while this order's is filled, if there is one above it
            u32* const below = prune && n > 2 ? (u32*)(arena + at_twice + (n & 1) * twice_bytes) : nullptr;
            u32* const mine = prune && n < n_max ? (u32*)(arena + at_twice + (1 - (n & 1)) * twice_bytes) : nullptr;
            TASC_HIP(hipEventRecord(evc[n][0], st));
            if (mine) TASC_HIP(hipMemsetAsync(mine, 0, twice_bytes, st));
            TASC_TRY(tasc_count_partition(p, d_tok, d_last, mine != nullptr, T, nullptr, n, 1, bits, bufs, below, &d_counters[n][0], st));
            TASC_TRY(tasc_count_tables(p, n, bits, (u32)p_min, bufs, d_counters[n], kept_of(n), mine, T, st));
            TASC_HIP(hipEventRecord(evc[n][1], st));
        }
        TASC_HIP(hipMemcpyAsync(h_counters, d_counters, sizeof h_counters, hipMemcpyDeviceToHost, st));
        TASC_HIP(hipStreamSynchronize(st));
        TASC_REQUIRE(h_counters[0][4] == 0, "ngram_build: corpus holds a token outside [0, %d)", vocab);
        // the finished tables of the group in one block; their context tables are built in the records' memory
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
        TASC_TRY(tasc_device_malloc((void**)&ng->tables[n0], total * sizeof(TascSlot)));
        CtxRef* ref = (CtxRef*)bufs.rec;
        u64 room = rec_bytes / sizeof(CtxRef);
        if (most > room) {
            TASC_TRY(tasc_device_malloc((void**)&ref, most * sizeof(CtxRef)));
            tmp.ptrs.push_back(ref);
            room = most;
        }
        TascSlot* at = ng->tables[n0];
        FinishAll all{};
        all.bits = bits;
        u64 used_ref = 0, largest = 0;
        u32 groups = 0;
        auto finish = [&]() -> tasc_status {                   // the orders collected so far
            if (all.orders == 0) return TASC_OK;
            const dim3 grid((unsigned)std::min<u64>((largest + kThreads - 1) / kThreads, 2048), (unsigned)all.orders);
            k_clear_tables<<<grid, dim3(kThreads), 0, st>>>(all);
            TASC_LAUNCH_CHECK();
            k_keep<<<dim3(groups), dim3(kThreadsKeep), 0, st>>>(all);
            TASC_LAUNCH_CHECK();
            k_materialize_ctx<<<dim3((unsigned)std::min<u64>((largest + kThreadsCtx - 1) / kThreadsCtx, kGroupsCtx), (unsigned)all.orders), dim3(kThreadsCtx), 0, st>>>(all);
            TASC_LAUNCH_CHECK();
            all.orders = 0;
            used_ref = largest = 0;
            groups = 0;
            return TASC_OK;
        };
        for (int n = n0; n < group_end[n0]; ++n) {
            if (fcap[n] == 0) continue;
            TascSlot *full = at, *ctx = at + fcap[n];
            at += 2 * fcap[n];
            const u64 kept = h_counters[n][1];
            if (used_ref + fcap[n] > room) TASC_TRY(finish()); // (the records' memory holds the contexts of all orders as a rule)
            all.order[all.orders++] = Finish{kept_of(n), kept, full, ctx, ref + used_ref, fcap[n], &d_counters[n][2], n, groups};
            used_ref += fcap[n];
            largest = std::max(largest, fcap[n]);
            groups += (u32)((kept + kThreadsKeep - 1) / kThreadsKeep);
            ng->slots[n][0] = ctx;
            ng->slots[n][1] = full;
            ng->view.ord[n].ctx = ctx;
            ng->view.ord[n].full = full;
            ng->view.ord[n].ctx_mask = ng->view.ord[n].full_mask = fcap[n] - 1;
        }
        TASC_TRY(finish());
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
    scratch.keep();
    guard.p = nullptr;
    *out = ng;
    return TASC_OK;
}

tasc_status tasc_mark_ends(const int64_t* d_off, int64_t n_docs, u64 T, uint8_t* d_last, hipStream_t st) {
    TASC_HIP(hipMemsetAsync(d_last, 0, T, st));
    if (n_docs > 0) k_mark_doc_ends<<<dim3((unsigned)((n_docs + kThreads - 1) / kThreads)), dim3(kThreads), 0, st>>>(d_off, n_docs, d_last);
    TASC_LAUNCH_CHECK();
    return TASC_OK;
}

extern "C" void tasc_ngram_destroy(tasc_ngram* ng) {
    if (!ng) return;
    for (TascSlot* t : ng->tables)
        if (t) (void)hipFree(t);
    if (ng->unigram) (void)hipFree(ng->unigram);
    delete ng;
    tasc_handles_add(-1);
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
