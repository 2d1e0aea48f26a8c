// Draft proposal: k tokens per sequence from the mixture of the corpus drafter and the context
// drafter (paper, section "Proposed Method: TASC-spec":
//     p_mixed(x|c) = lambda p_corp(x|c) + (1 - lambda) p_prompt(x|c),
// each source queried in descending order of n, first match wins, most frequent token if none).
//
// The sequence's committed tokens sit in LDS; the context drafter is not a stored table: for the running suffix, the places of
// its last token get the length of their match with it, the longest match gives the context's order, and the tokens that
// follow the matching positions are its successor multiset.  Exact integer scores.
#include "tasc_internal.h"

namespace {

struct DraftArgs {
    TascNgramView ng;
    const int32_t* tokens;    // [B, max_len]
    const int32_t* n_tok;     // [B]
    const int32_t* n_prompt;  // [B]
    int32_t max_len, k, q16, p_min_ctx, ctx_gen;
    int32_t* drafts;          // [B, k]
};

__device__ inline bool probe(const TascSlot* __restrict__ tab, u64 mask, u64 lo, u64 hi, TascSlot& out) {
    u64 idx = tasc_slot_of(tasc_hash_key(lo, hi), mask);
    for (u64 p = 0; p <= mask; ++p) {
        TascSlot s = tab[idx];
        if (s.a == 0) return false;
        if (s.lo == lo && s.hi == hi) {
            out = s;
            return true;
        }
        idx = (idx + 1) & mask;
    }
    return false;
}

// One workgroup per sequence.  All its waves bring the tokens to LDS and sort the positions into buckets by their token (or leave
// them in order where that costs more than it saves: kUnsorted); then one
// WAVE makes the k sequential proposals: every exchange between lanes is a ballot, a lane read or an LDS access of the
// same wave, so they cross no workgroup barrier.  What bounds it is that chain of dependent steps and not memory (64 sequences of 64
// to 2,300 tokens, k = 8: 35 us, 55 with one wave and a pass over the sequence per proposal, and no longer at any length from 60 tokens on; its tokens and slots
// are 0.7 MB):
//   * the running suffix comes from LDS into registers, all tokens of it at once, and keys are shifted together from it
//     without a loop over LDS; what a lane asks for in every proposal (its order, that order's tables) is looked up once;
//   * corpus source: lanes 0 .. n_max-2 request the first slot of one order each, and the answers are only looked at after the
//     context phase, so the round trip runs under it;
//   * context source: the bucket of the last token, a lane per position; only the positions of the last token
//     are compared with the rest of the suffix.  The successors of the longest
//     matches are counted with a ballot per distinct one while the list fits the wave's lanes, else in a hash table in LDS
//     (token -> multiplicity; entries carry a generation number, so the table is never cleared); the distinct ones are the
//     candidates;
//   * the candidates' corpus counts are requested at EVERY order before the corpus context is known (a second round
//     trip that would otherwise wait for the first), and the ones of the matching order are used;
//   * the argmax over (score, smallest token) is a reduction over neighbouring lanes (DPP, no LDS round trips).
constexpr int kHashSlots = 2 * TASC_DRAFT_MAX_LEN;        // more than any sequence has successors
static_assert(TASC_DRAFT_MAX_LEN <= 4096 && TASC_DRAFT_MAX_LEN % 4 == 0 && TASC_MAX_ORDER <= 16, "list entries, token reads");

// wave reductions: after the six steps lane 63 has the result, which a lane read hands to all
template <int CTRL, int ROWS>
__device__ __forceinline__ u32 dpp_max_step(u32 v) {
    const u32 w = (u32)__builtin_amdgcn_update_dpp((int)v, (int)v, CTRL, ROWS, 0xf, false);
    return w > v ? w : v;
}
__device__ __forceinline__ u32 wave_max_u32(u32 v) {
    v = dpp_max_step<0x111, 0xf>(v);          // row_shr:1, 2, 4, 8: within 16 lanes
    v = dpp_max_step<0x112, 0xf>(v);
    v = dpp_max_step<0x114, 0xf>(v);
    v = dpp_max_step<0x118, 0xf>(v);
    v = dpp_max_step<0x142, 0xa>(v);          // row_bcast:15, 31: across them
    v = dpp_max_step<0x143, 0xc>(v);
    return (u32)__builtin_amdgcn_readlane((int)v, 63);
}
__device__ __forceinline__ u64 wave_max_u64(u64 v) {
    const u32 hi = wave_max_u32((u32)(v >> 32));
    return ((u64)hi << 32) | wave_max_u32((u32)(v >> 32) == hi ? (u32)v : 0u);
}
template <int CTRL, int ROWS>
__device__ __forceinline__ int dpp_add_step(int v) { return v + __builtin_amdgcn_update_dpp(0, v, CTRL, ROWS, 0xf, false); }
__device__ __forceinline__ int wave_add(int v) {
    v = dpp_add_step<0x111, 0xf>(v);
    v = dpp_add_step<0x112, 0xf>(v);
    v = dpp_add_step<0x114, 0xf>(v);
    v = dpp_add_step<0x118, 0xf>(v);
    v = dpp_add_step<0x142, 0xa>(v);
    v = dpp_add_step<0x143, 0xc>(v);
    return __builtin_amdgcn_readlane(v, 63);
}
__device__ __forceinline__ TascSlot slot_load(const TascSlot* p) {
    const uint4 a = reinterpret_cast<const uint4*>(p)[0], b = reinterpret_cast<const uint4*>(p)[1];
    TascSlot s;
    s.lo = (u64)a.x | ((u64)a.y << 32); s.hi = (u64)a.z | ((u64)a.w << 32);
    s.a = b.x; s.b = b.y; s.c = b.z; s.d = b.w;
    return s;
}
// finishes a probe whose first slot `s` (index idx) has been loaded already
__device__ __forceinline__ bool probe_finish(const TascSlot* __restrict__ tab, u64 mask, u64 lo, u64 hi, u64 idx, TascSlot& s) {
    for (u64 p = 0; p <= mask; ++p) {
        if (s.a == 0) return false;
        if (s.lo == lo && s.hi == hi) return true;
        idx = (idx + 1) & mask;
        s = slot_load(tab + idx);
    }
    return false;
}

// The key of the m tokens t[m - 1], .., t[0], the oldest as element 0 (the layout of tasc_key_put): shifted together from the
// newest one down, so every shift is by `bits`.
__device__ __forceinline__ void key_of(const u32* t, int m, int bits, u64& lo, u64& hi) {
    lo = hi = 0;
#pragma unroll
    for (int i = 0; i < TASC_MAX_ORDER; ++i) {
        const u64 h = (hi << bits) | (lo >> (64 - bits)), l = (lo << bits) | t[i];
        if (i < m) { hi = h; lo = l; }
    }
}

constexpr int kDraftWaves = 8, kDraftThreads = 64 * kDraftWaves;
constexpr int kBuckets = 1024;                            // of positions by their token
// Sorting takes 0.5 to 1.5 us.  It is left out where nothing is looked for in the context (lambda 1: a proposal 6.6 | 6.0 us, eight
// 13.3 | 12.0, one sequence) and where the proposals, times 64 positions that a sequence has room for, are no more than this: each
// then reads all positions (one proposal, room for 480: 30 tokens with orders to 5 6.9 | 6.0, 256 sequences of 300 8.3 | 7.6; over 256
// sequences of 3900 a pass over all of them took 15.2, the sort and one bucket 9.4).
constexpr int kUnsorted = 8;
__device__ __forceinline__ u32 bucket_of(u32 tok) { return (tok * 0x9E3779B1u) >> 22; }
static_assert(kBuckets == 1 << 10 && kBuckets == 2 * kDraftThreads, "bucket_of, two buckets per thread");

// SORTED: positions in buckets by their token; else all of them in order, in one
template <bool SORTED>
__global__ __launch_bounds__(kDraftThreads) void k_draft(DraftArgs a) {
    __shared__ __attribute__((aligned(16))) int32_t s_tok[TASC_DRAFT_MAX_LEN];
    __shared__ uint16_t s_index[TASC_DRAFT_MAX_LEN];      // positions that a token follows, by bucket of their token
    __shared__ __attribute__((aligned(16))) u32 s_bucket[kBuckets + 1];                // the buckets' first places
    __shared__ uint16_t s_pos[TASC_DRAFT_MAX_LEN];        // positions of the last token before the end; of lists beyond 64: {match length - 1 : 4, position : 12}
    __shared__ __attribute__((aligned(16))) u64 s_tab[kHashSlots];   // {generation : 16, multiplicity : 16, token : 32}
    __shared__ uint16_t s_dl[TASC_DRAFT_MAX_LEN];         // slots of the distinct successors of the current generation
    __shared__ int32_t s_d[TASC_MAX_K];                   // the proposals so far
    __shared__ u32 s_wave[kDraftWaves];
    __shared__ int s_nd;
    __shared__ TascSlot s_hit[TASC_MAX_ORDER + 1];

    const int b = blockIdx.x, tid = threadIdx.x, lane = tid & 63;
    const u64 lt_mask = (1ull << lane) - 1;
    const int N = a.n_tok[b];
    const int Nctx = a.ctx_gen ? N : min(N, a.n_prompt[b]);   // tokens the context statistics cover
    const int32_t* seq = a.tokens + (size_t)b * a.max_len;
    const u64 q = (u64)a.q16, qb = (u64)(65536 - a.q16);
    u32 tab_mask = 127;                                    // slots of the hash table: at least twice the successors there can be
    while (tab_mask + 1 < 2 * (u32)Nctx) tab_mask = 2 * tab_mask + 1;

    // ---- all waves: tokens to LDS; positions sorted by bucket
    {
        constexpr int PER = TASC_DRAFT_MAX_LEN / kDraftThreads;
        int32_t t[PER];
        u32 rank[PER];
#pragma unroll
        for (int u = 0; u < PER; ++u) t[u] = seq[min(u * kDraftThreads + tid, N - 1)];
        for (u32 i = 2 * tid; i <= tab_mask; i += 2 * kDraftThreads) *reinterpret_cast<ulonglong2*>(&s_tab[i]) = make_ulonglong2(0, 0);   // generation 0 = never used
        if (SORTED) *reinterpret_cast<uint2*>(&s_bucket[2 * tid]) = make_uint2(0, 0);
#pragma unroll
        for (int u = 0; u < PER; ++u)
            if (u * kDraftThreads + tid < N) s_tok[u * kDraftThreads + tid] = t[u];
        __syncthreads();
        if constexpr (SORTED) {
#pragma unroll
            for (int u = 0; u < PER; ++u)
                if (u * kDraftThreads + tid < Nctx - 1) rank[u] = atomicAdd(&s_bucket[bucket_of((u32)t[u])], 1u);
            __syncthreads();
            const uint2 n = *reinterpret_cast<const uint2*>(&s_bucket[2 * tid]);
            u32 at = n.x + n.y;
            for (int o = 1; o < 64; o <<= 1) {
                const u32 v = __shfl_up(at, o);
                if (lane >= o) at += v;
            }
            if (lane == 63) s_wave[tid >> 6] = at;
            __syncthreads();
            for (int w = 0; w < (tid >> 6); ++w) at += s_wave[w];
            *reinterpret_cast<uint2*>(&s_bucket[2 * tid]) = make_uint2(at - n.x - n.y, at - n.y);
            if (tid == kDraftThreads - 1) s_bucket[kBuckets] = at;
            __syncthreads();
#pragma unroll
            for (int u = 0; u < PER; ++u)
                if (u * kDraftThreads + tid < Nctx - 1) s_index[s_bucket[bucket_of((u32)t[u])] + rank[u]] = (uint16_t)(u * kDraftThreads + tid);
            __syncthreads();
        }
    }
    if (tid >= 64) return;

    // ---- the first wave: the proposals, one after the other
    const int n_max = a.ng.n_max, bits = a.ng.bits, n_ord = n_max - 1;
    u32 gen = 0;
    // what the lane asks for in every proposal: contexts of my_n - 1 tokens, and counts of f_ord-grams
    const int my_n = max(n_max - lane, 2), f_ord = n_max - lane % n_ord;
    const TascSlot* const my_ctx = a.ng.ord[my_n].ctx;
    const u64 my_ctx_mask = a.ng.ord[my_n].ctx_mask;
    const TascSlot* const f_full = a.ng.ord[f_ord].full;
    const u64 f_full_mask = a.ng.ord[f_ord].full_mask;

    for (int j = 0; j < a.k; ++j) {
        const int wlen = N + j;
        const int nsuf = min(n_max - 1, wlen);             // at least 1
        u32 run[TASC_MAX_ORDER + 1];                       // a candidate, then the suffix
        u32* const suf = run + 1;                          // suf[i] = i-th token from the end of the running context
        run[0] = suf[TASC_MAX_ORDER - 1] = 0;
#pragma unroll
        for (int i = 0; i < TASC_MAX_ORDER - 1; ++i) suf[i] = (u32)(i < j ? s_d[j - 1 - i] : s_tok[max(N - 1 - (i - j), 0)]);

        // ---- corpus source: the first slot of every order is requested now and examined after the context phase
        const bool c_probe = q > 0 && lane < n_max - 1 && my_n - 1 <= nsuf && my_ctx != nullptr;
        u64 c_lo = 0, c_hi = 0, c_idx = 0;
        TascSlot c_slot = {0, 0, 0, 0, 0, 0};
        if (c_probe) {
            key_of(suf, my_n - 1, bits, c_lo, c_hi);
            c_idx = tasc_slot_of(tasc_hash_key(c_lo, c_hi), my_ctx_mask);
            c_slot = slot_load(my_ctx + c_idx);
        }

        // ---- context source
        int n_ctx = 0, T_ctx = 0, n_dist = 0;
        bool in_regs = false;                              // the candidates are (cand_x, cand_c) of the lanes below n_dist, else in the table
        int cand_x = 0, cand_c = 0;
        if (qb > 0) {
            int n_list = 0, my_ml = 0, e_at = 0;
            // the places of the last token: those of its bucket that are it ...
            const u32 bk = bucket_of(suf[0]);
            const int from = SORTED ? (int)s_bucket[bk] : 0, to = SORTED ? (int)s_bucket[bk + 1] : max(Nctx - 1, 0);
            auto place = [&](int i) { return SORTED ? (int)s_index[i] : i; };
            const bool direct = to - from <= 64;           // a lane each, no list
            if (direct) {
                e_at = from + lane < to ? place(from + lane) : 0;
            } else {
                for (int p0 = from; p0 < to; p0 += 64) {
                    const int at = place(min(p0 + lane, to - 1));
                    const bool hit = p0 + lane < to && (u32)s_tok[at] == suf[0];
                    const u64 m = __ballot(hit);
                    if (hit) s_pos[n_list + __popcll(m & lt_mask)] = (uint16_t)at;
                    n_list += __popcll(m);
                }
            }
            __builtin_amdgcn_s_waitcnt(0);
            __builtin_amdgcn_wave_barrier();
            // ... and how much of the suffix before it matches there
            int e_ml = 0, e_x = 0;                         // the lane's (last) list entry: match length and successor
            auto match = [&](int at) __attribute__((always_inline)) {
                int before[TASC_MAX_ORDER - 2];
#pragma unroll
                for (int i = 1; i < TASC_MAX_ORDER - 1; ++i) before[i - 1] = s_tok[max(at - i, 0)];
                e_x = s_tok[at + 1];
                int ml = 1;
                bool on = true;
#pragma unroll
                for (int i = 1; i < TASC_MAX_ORDER - 1; ++i) {
                    on = on && i < nsuf && at - i >= 0 && (u32)before[i - 1] == suf[i];
                    ml += on ? 1 : 0;
                }
                return ml;
            };
            if (direct) {
                const bool hit = from + lane < to && (u32)s_tok[e_at] == suf[0];
                const int ml = match(e_at);
                e_ml = hit ? ml : 0;
                my_ml = e_ml;
                n_list = __popcll(__ballot(hit));
            } else {
                for (int e0 = 0; e0 < n_list; e0 += 64) {
                    const int at = s_pos[min(e0 + lane, n_list - 1)], ml = match(at);
                    e_ml = e0 + lane < n_list ? ml : 0;
                    my_ml = max(my_ml, e_ml);
                    if (n_list > 64 && e_ml) s_pos[e0 + lane] = (uint16_t)(((ml - 1) << 12) | at);
                }
            }
            int lmax = 0;
            if (n_list > 0) {
                lmax = 1;
                for (int v = nsuf; v > 1; --v)
                    if (__ballot(my_ml >= v)) { lmax = v; break; }
            }
            __builtin_amdgcn_s_waitcnt(0);
            __builtin_amdgcn_wave_barrier();
            in_regs = direct || n_list <= 64;
            // back off from the longest matching context until one has a kept successor
            for (int n = lmax + 1; n >= 2 && !n_ctx; --n) {
                int t = 0;
                if (in_regs) {
                    n_dist = 0;
                    u64 todo = __ballot(e_ml >= n - 1);
                    while (todo) {                         // one round per distinct successor
                        const int key = __builtin_amdgcn_readlane(e_x, __ffsll((unsigned long long)todo) - 1);
                        const u64 same = __ballot(e_x == key) & todo;
                        const int cnt = __popcll(same);
                        if (lane == n_dist) { cand_x = key; cand_c = cnt; }
                        ++n_dist;
                        if (cnt >= a.p_min_ctx) t += cnt;
                        todo &= ~same;
                    }
                } else {
                    ++gen;
                    if (lane == 0) s_nd = 0;
                    __builtin_amdgcn_s_waitcnt(0);
                    __builtin_amdgcn_wave_barrier();
                    for (int e0 = 0; e0 < n_list; e0 += 64) {
                        const int e = e0 + lane;
                        const int w = e < n_list ? s_pos[e] : 0;
                        const bool in = e < n_list && (w >> 12) + 1 >= n - 1;
                        const u32 key = in ? (u32)s_tok[(w & 0xFFF) + 1] : 0u;
                        const u64 act = __ballot(in);
                        if (!act) continue;
                        // a run of one token (every lane the same successor) is added in one go by the first lane
                        const int first = __ffsll((unsigned long long)act) - 1;
                        const u32 k0 = (u32)__builtin_amdgcn_readlane((int)key, first);
                        const bool uniform = __ballot(in && key == k0) == act;
                        const u64 add = uniform ? (u64)__popcll(act) : 1ull;
                        if (uniform ? lane == first : in) {
                            u32 slot = (u32)tasc_mix64(key) & tab_mask;
                            for (;;) {
                                const u64 w64 = s_tab[slot];
                                if ((u32)(w64 >> 48) != gen) {
                                    // empty for this generation: claim it
                                    const u64 neu = ((u64)gen << 48) | (add << 32) | key;
                                    if (atomicCAS(reinterpret_cast<unsigned long long*>(&s_tab[slot]), w64, neu) == w64) {
                                        s_dl[atomicAdd(&s_nd, 1)] = (uint16_t)slot;
                                        break;
                                    }
                                    continue;              // somebody else took it: look at it again
                                }
                                if ((u32)w64 == key) {
                                    atomicAdd(reinterpret_cast<unsigned long long*>(&s_tab[slot]), add << 32);
                                    break;
                                }
                                slot = (slot + 1) & tab_mask;
                            }
                        }
                    }
                    __builtin_amdgcn_s_waitcnt(0);
                    __builtin_amdgcn_wave_barrier();
                    n_dist = s_nd;
                    for (int e = lane; e < n_dist; e += 64) {
                        const int c = (int)((s_tab[s_dl[e]] >> 32) & 0xFFFFu);
                        if (c >= a.p_min_ctx) t += c;
                    }
                    t = wave_add(t);
                }
                if (t > 0) { n_ctx = n; T_ctx = t; }
            }
        }
        // candidate e, from wherever the candidates are
        auto candidate = [&](int e, int& x, int& c) {
            if (in_regs) {
                x = __shfl(cand_x, e & 63);
                c = __shfl(cand_c, e & 63);
            } else {
                const u64 w = s_tab[s_dl[min(e, n_dist - 1)]];
                x = (int)(u32)w;
                c = (int)((w >> 32) & 0xFFFFu);
            }
        };

        // ---- the candidates' corpus counts, requested at every order a corpus context could match (pair = candidate x order)
        const bool spec = q > 0 && n_ctx && n_dist * n_ord <= 64;
        u64 f_lo = 0, f_hi = 0, f_idx = 0;
        TascSlot f_slot = {0, 0, 0, 0, 0, 0};
        int f_n = 0, f_x = 0, f_c = 0;
        if (spec) {
            candidate(lane / n_ord, f_x, f_c);
            if (lane < n_dist * n_ord) {
                if (f_c >= a.p_min_ctx && f_ord - 1 <= nsuf && f_full != nullptr) {
                    f_n = f_ord;
                    run[0] = (u32)f_x;
                    key_of(run, f_n, bits, f_lo, f_hi);
                    f_idx = tasc_slot_of(tasc_hash_key(f_lo, f_hi), f_full_mask);
                    f_slot = slot_load(f_full + f_idx);
                }
            }
        }

        // ---- the corpus context: the highest order whose probe hits
        bool found = false;
        if (c_probe && probe_finish(my_ctx, my_ctx_mask, c_lo, c_hi, c_idx, c_slot)) {
            s_hit[my_n] = c_slot;
            found = true;
        }
        const u64 found_mask = __ballot(found);
        const int n_corp = found_mask ? n_max - (__ffsll((unsigned long long)found_mask) - 1) : 0;   // lowest lane = highest order
        __builtin_amdgcn_s_waitcnt(0);
        __builtin_amdgcn_wave_barrier();

        // ---- proposal
        int x;
        if (!n_corp && !n_ctx) {
            x = a.ng.fallback;
        } else if (!n_ctx) {
            x = (int)s_hit[n_corp].b;
        } else {
            const u64 T_corp = n_corp ? s_hit[n_corp].a : 0;
            u64 my_score = 0;
            int my_x = 0x7FFFFFFF;
            if (spec) {
                // one lane per (candidate, order): the lanes of the matching order (or, without a corpus match, of the
                // highest order: one per candidate) score
                const bool scorer = lane < n_dist * n_ord && f_c >= a.p_min_ctx && (n_corp ? f_ord == n_corp : f_ord == n_max);
                if (scorer) {
                    u64 sc;
                    if (n_corp) {
                        const u64 c_corp = (f_n == n_corp && probe_finish(f_full, f_full_mask, f_lo, f_hi, f_idx, f_slot)) ? f_slot.a : 0;
                        sc = q * c_corp * (u64)T_ctx + qb * (u64)f_c * T_corp;
                    } else {
                        sc = (u64)f_c;
                    }
                    my_score = sc;
                    my_x = f_x;
                }
            } else {
                u64 lo0 = 0, hi0 = 0;
                if (n_corp) key_of(suf, n_corp - 1, bits, lo0, hi0);
                for (int e0 = 0; e0 < n_dist; e0 += 64) {
                    int xe, c;
                    candidate(e0 + lane, xe, c);
                    if (e0 + lane >= n_dist || c < a.p_min_ctx) continue;
                    u64 sc;
                    if (n_corp) {
                        u64 lo = lo0, hi = hi0;
                        tasc_key_put(lo, hi, n_corp - 1, bits, (u32)xe);
                        TascSlot hit;
                        const u64 c_corp = probe(a.ng.ord[n_corp].full, a.ng.ord[n_corp].full_mask, lo, hi, hit) ? hit.a : 0;
                        sc = q * c_corp * (u64)T_ctx + qb * (u64)c * T_corp;
                    } else {
                        sc = (u64)c;
                    }
                    if (sc > my_score || (sc == my_score && xe < my_x)) { my_score = sc; my_x = xe; }
                }
            }
            if (n_corp && lane == 63) {
                // the corpus' own best successor: scores at least this even if the context never saw it (merged into
                // whatever the lane holds already)
                const u64 sc = q * (u64)s_hit[n_corp].c * (u64)T_ctx;
                const int xe = (int)s_hit[n_corp].b;
                if (sc > my_score || (sc == my_score && xe < my_x)) { my_score = sc; my_x = xe; }
            }
            const u64 best = wave_max_u64(my_x != 0x7FFFFFFF ? my_score : 0);
            const int cand = (my_x != 0x7FFFFFFF && my_score == best) ? my_x : 0x7FFFFFFF;
            x = (int)(0x7FFFFFFFu - wave_max_u32(0x7FFFFFFFu - (u32)cand));          // the smallest
        }
        if (lane == 0) {
            s_d[j] = x;
            a.drafts[(size_t)b * a.k + j] = x;
        }
        __builtin_amdgcn_s_waitcnt(0);
        __builtin_amdgcn_wave_barrier();
    }
}

}  // namespace

extern "C" tasc_status tasc_draft(const tasc_ngram* ng, tasc_session* s, const tasc_spec_params* p, int32_t* drafts,
                                  void* stream) {
    TASC_REQUIRE(ng && s && p && drafts, "draft: null argument");
    TASC_REQUIRE(p->k >= 1 && p->k <= TASC_MAX_K, "draft: k %d outside [1, %d]", p->k, TASC_MAX_K);
    TASC_REQUIRE(p->lambda_q16 >= 0 && p->lambda_q16 <= 65536, "draft: lambda_q16 %d outside [0, 65536]", p->lambda_q16);
    TASC_REQUIRE(p->p_min_ctx >= 1, "draft: p_min_ctx %d < 1", p->p_min_ctx);
    TASC_REQUIRE(ng->view.vocab == s->model->desc.vocab, "draft: table vocabulary %d, model vocabulary %d", ng->view.vocab,
                 s->model->desc.vocab);
    if (!s->prefilled) {
        tasc_set_error("draft: session has no prompt yet");
        return TASC_ESTATE;
    }
    TASC_REQUIRE(s->max_len <= TASC_DRAFT_MAX_LEN, "draft: max_len %d exceeds %d", s->max_len, TASC_DRAFT_MAX_LEN);
    DraftArgs a;
    a.ng = ng->view;
    a.tokens = s->d.tokens;
    a.n_tok = s->d.n_tok;
    a.n_prompt = s->d.n_prompt;
    a.max_len = s->max_len;
    a.k = p->k;
    a.q16 = p->lambda_q16;
    a.p_min_ctx = p->p_min_ctx;
    a.ctx_gen = p->ctx_includes_generated;
    a.drafts = drafts;
    {
        TascProfScope ps(TASC_KC_DRAFT, (hipStream_t)stream);
        const bool sorted = p->lambda_q16 < 65536 && p->k * ((s->max_len + 63) / 64) > kUnsorted;
        (sorted ? k_draft<true> : k_draft<false>)<<<dim3(s->batch), dim3(kDraftThreads), 0, (hipStream_t)stream>>>(a);
    }
    TASC_LAUNCH_CHECK();
    return TASC_OK;
}
