// Exact n-gram counts of a corpus: the counting stage of the table build and of the tokenizer enrichment.
//
// A counting table of tens of millions of random slots in memory is bound by the rate of its atomics (9 to 12 G windows/s on
// this card, whatever is done to keep more of them in flight), so no count is ever kept in memory.  Two kernels per order:
//   * k_partition: a workgroup takes a chunk of consecutive corpus positions, merges equal windows of the chunk in an LDS table and
//     writes what is left, ordered by partition, as records into the chunk's own region, with the partitions' offsets beside
//     it: no exchange between workgroups, nothing to reserve, and the regions are as large as the corpus whatever its n-grams are;
//   * k_tables: one partition, all chunks: a workgroup gathers the partition's records into a hash table in its LDS and
//     reads the finished counts off it; of more windows than partitions can take, in several rounds (tasc_count_plan).
// Partitions are ranges of the key's 64-bit hash.  With the upper half `hi` of the 128-bit key given, the hash is a bijection of the
// lower half, so (hash, hi) is the key itself: records and LDS slots hold 8 bytes for keys of up to 64 bits and 16 beyond, the
// comparison is exact, and nothing looks at the corpus again.
// Both kernels live on dependent LDS round trips: a hash probe is an exchange, a comparison and an addition, and a wave that takes one
// window or record per lane at a time waits for its unluckiest lane at each.  So a lane that is done with one takes its next at once.
// And of the orders above the second, a window whose first or last n - 1 tokens occur once in the corpus occurs once itself: a map of
// the (n-1)-grams that occur more often (a few per cent of the distinct ones) takes a third to half of the windows out.
// Whether that is so takes a look at the map for every position; what the order below saw of its windows, chunk by chunk, spares two looks in three.
// 32 M tokens, orders 2 to 5 together, us: 9135 with a table in memory; k_partition 1300 (1840 with loads that wait for each other where a chunk
// begins and all looks at the map), k_turn 90, k_tables 1020 (2540 and 1840 without the map).  All wait for LDS and L2 with one or two workgroups
// a compute unit: a chunk of order 4 is 53 k cycles, 6 of them for its loads, 14 at the map, 11 to merge, 11 for keys and ranks, 11 to put in order.
// Measured and left out: workgroups that go on to a next chunk with its loads ahead (registers: 369 / 409 / 386 for orders 3 to 5 and k_turn, 366 /
// 402 / 378 so), chunks of 4096 two to a unit (an eighth less here, more in k_tables than that), the map's loads before the merging (no overlap).
#include "tasc_internal.h"
#include <algorithm>

namespace {

// A record is {low 56 bits of the hash : 56, count - 1 : 8}, followed by the key's upper half where keys have more than 64 bits;
// larger counts of a chunk take several.  The upper 8 bits of the hash follow from the partition: at least TASC_COUNT_MIN_PARTS =
// 256 ranges of the hash's upper 32 bits, so a range is no longer than 2^24.
__device__ inline u32 part_of(u64 hash, u32 parts) { return __umulhi((u32)(hash >> 32), parts); }
__device__ inline u64 hash_of(u64 rec, u32 part, u32 parts) {
    const u32 first = (u32)((((u64)part << 32) + parts - 1) / parts);         // smallest upper half of the partition
    const u32 low24 = (u32)(rec >> 40);
    const u32 top = (first >> 24) + (low24 < (first & 0xFFFFFFu) ? 1u : 0u);
    return ((u64)top << 56) | (rec >> 8);
}

// exclusive scan over the workgroup; s_wave holds a word per wave and may be used again after the next barrier
template <int TH>
__device__ __forceinline__ u32 block_scan(u32 v, u32* s_wave, u32& total) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    u32 at = v;
    for (int o = 1; o < 64; o <<= 1) {
        const u32 w = __shfl_up(at, o);
        if (lane >= o) at += w;
    }
    if (lane == 63) s_wave[wave] = at;
    __syncthreads();
    u32 before = 0;
    total = 0;
#pragma unroll
    for (int w = 0; w < TH / 64; ++w) {
        const u32 n = s_wave[w];
        before += w < wave ? n : 0;
        total += n;
    }
    return before + at - v;
}

// A hash of n tokens that costs two instructions a token; good enough for a chunk's table, and for the map of n-grams that occur twice
__device__ __forceinline__ u32 light_step(u32 h, u32 tok, int j) { return h ^ (j == 0 ? tok : (tok << (13 * j % 32)) | (tok >> (32 - 13 * j % 32))); }   // (never by 0 or 32)
__device__ __forceinline__ u32 light_end(u32 h) { return h * 0x9E3779B1u; }

// marks: a byte a position.  With `twice`, what the order below found out of its windows in its own chunks spares most looks at the map:
// each is a line of the L2 for one bit, and they arrive at a line every 2.5 cycles a compute unit, 21 k cycles a chunk of 8192 where all look.
constexpr u32 kMarkEnd = 1;        // the document's last token
constexpr u32 kMarkOnce = 2;       // the window that begins here occurs once, or is none
constexpr u32 kMarkOften = 4;      // it occurs more than once in the chunk alone

// LDS (dynamic): tokens [C + 8], slots [2 C] of {position in the chunk + 1 : 16, count : 16}, partition counters [parts], wave sums, the
// windows' slots [C], marks, a bit a position [3][C / 8 + 8].  A few rotations of the tokens make a hash that is good enough for the chunk's table; the key and its hash are
// computed once per window that is left.
//
// twice (nullable): a bit per range of the (N - 1)-grams' light hash, set for those that occur at least twice.  A window that begins or ends with
// one that occurs once occurs once itself: it is counted and leaves no record.
template <int N, int C, int TH>
__device__ __forceinline__ void partition_chunk(const int32_t* __restrict__ tok, uint8_t* marks, bool keep_marks, u64 T, int bits, u32 parts,
                                                const u32* __restrict__ twice, int twice_bits, u64* distinct, u64* __restrict__ rec,
                                                uint16_t* __restrict__ offs) {
    constexpr int W = C / TH;
    extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
    u32* s_slot = reinterpret_cast<u32*>(lds);
    u32* s_tok = s_slot + 2 * C;
    u32* s_hist = s_tok + C + 8;
    u32* s_wave = s_hist + ((parts + 1) & ~1u);           // (8-byte words behind it)
    uint16_t* s_claim = reinterpret_cast<uint16_t*>(s_wave + TH / 64);
    uint8_t* s_end = reinterpret_cast<uint8_t*>(s_claim + C);      // bit i of each: the mark of position i
    uint8_t* s_once = s_end + C / 8 + 8;
    uint8_t* s_often = s_once + C / 8 + 8;
    const int tid = threadIdx.x, lane = tid & 63;
    const u64 base = (u64)blockIdx.x * C;
    const int n_here = (int)min((u64)(C + N - 1), T - base), n_win = (int)min((u64)C, T - base);
    // The chunk is asked for at once: its tokens, eight positions' document ends a thread, and the N - 1 positions behind it.
    u32 t_in[W];
#pragma unroll
    for (int w = 0; w < W; ++w) t_in[w] = (u32)tok[base + min(w * TH + tid, n_here - 1)];
    const u32 t_tail = (u32)tok[base + min(C + min(tid, N - 2), n_here - 1)];
    u64 e_in[C / 8 > TH ? C / 8 / TH : 1];
    const bool marks_mine = C / 8 >= TH || tid < C / 8;
#pragma unroll
    for (int q = 0; q < (int)(sizeof e_in / 8); ++q) {
        const u64 at = base + 8 * (q * TH + tid);
        e_in[q] = 0;
        if (!marks_mine) continue;
        if (at + 8 <= T) e_in[q] = *reinterpret_cast<const u64*>(marks + at);
        else
            for (int e = 0; e < 8; ++e) e_in[q] |= at + e < T ? (u64)marks[at + e] << (8 * e) : 0;
    }
    const bool e_tail = tid < 8 && base + C + tid < T && (marks[base + C + tid] & kMarkEnd);
    for (int i = tid; i < 2 * C / 4; i += TH) reinterpret_cast<uint4*>(s_slot)[i] = make_uint4(0, 0, 0, 0);
    for (u32 i = tid; i < parts; i += TH) s_hist[i] = 0;
#pragma unroll
    for (int w = 0; w < W; ++w) s_tok[w * TH + tid] = t_in[w];
    if (tid < N - 1) s_tok[C + tid] = t_tail;
    // (a bit of eight bytes into one)
    auto plane = [](u64 v, u32 mark) __attribute__((always_inline)) { return (uint8_t)(((v / mark & 0x0101010101010101ull) * 0x0102040810204080ull) >> 56); };
    const bool pruned = N > 2 && twice;
#pragma unroll
    for (int q = 0; q < (int)(sizeof e_in / 8); ++q)
        if (marks_mine) {
            s_end[q * TH + tid] = plane(e_in[q], kMarkEnd);
            if (pruned) s_once[q * TH + tid] = plane(e_in[q], kMarkOnce);
            if (pruned) s_often[q * TH + tid] = plane(e_in[q], kMarkOften);
        }
    const u64 tail = __ballot(e_tail);
    if (tid == 0) s_end[C / 8] = (uint8_t)tail;
    __syncthreads();
    // a window stays inside its document if none of its tokens but the last ends one
    u32 inside = 0;                                        // bit w: window w TH + tid
#pragma unroll
    for (int w = 0; w < W; ++w) {
        const int i = w * TH + tid;
        const u32* const e = reinterpret_cast<const u32*>(s_end) + (i >> 5);
        const u32 ends = __funnelshift_r(e[0], e[1], i & 31);
        inside |= (i < n_win && (ends & ((1u << (N - 1)) - 1)) == 0) ? 1u << w : 0;      // (the corpus' last token ends a document)
    }
    if (pruned) {
        auto word_of = [&](int i, u32& bit) __attribute__((always_inline)) {
            u32 h = 0;
#pragma unroll
            for (int j = 0; j < N - 1; ++j) h = light_step(h, s_tok[i + j], j);
            h = light_end(h) >> (32 - twice_bits);
            bit = h & 31;
            return twice[h >> 5];
        };
        u32 word[W], bit[W], word_c = 0, bit_c = 0;        // of the lane's positions, and of the one past the chunk
        u64 often[W], once[W];
#pragma unroll
        for (int w = 0; w < W; ++w) {
            often[w] = reinterpret_cast<const u64*>(s_often)[(w * TH + tid) / 64];
            once[w] = reinterpret_cast<const u64*>(s_once)[(w * TH + tid) / 64];
            word[w] = bit[w] = 0;
            if ((((often[w] | once[w]) >> lane) & 1) == 0) word[w] = word_of(w * TH + tid, bit[w]);
        }
        if (tid == 0) word_c = word_of(C, bit_c);
#pragma unroll
        for (int w = 0; w < W; ++w) {
            often[w] |= __ballot((word[w] >> bit[w]) & 1);
            if (lane == 0) reinterpret_cast<u64*>(s_often)[(w * TH + tid) / 64] = often[w];
        }
        if (tid == 0) reinterpret_cast<u64*>(s_often)[C / 64] = (word_c >> bit_c) & 1;
        __syncthreads();
        u32 gone = 0;
#pragma unroll
        for (int w = 0; w < W; ++w) {
            const u64 here = often[w], next = reinterpret_cast<const u64*>(s_often)[(w * TH + tid) / 64 + 1];
            const u64 both = here & ((here >> 1) | (next << 63));
            if (((inside >> w) & 1) && !((both >> lane) & 1)) gone |= 1u << w;
        }
        inside &= ~gone;
        u32 n = (u32)__popc(gone);
        for (int o = 32; o > 0; o >>= 1) n += __shfl_xor(n, o);
        if (lane == 0) s_wave[tid >> 6] = n;
        __syncthreads();
        if (tid == 0) {
            u32 all = 0;
            for (int w = 0; w < TH / 64; ++w) all += s_wave[w];
            if (all) atomicAdd(distinct, (u64)all);
        }
    }

    // ---- equal windows merged: a lane probes once per turn and takes its next window as soon as it is done with one
    u32 mine = 0;                                          // bit w: the window claimed its slot, s_claim[w TH + tid]
    const u32 alive = inside;
    {
        u32 t[N], idx = 0;
        int i = 0;
        bool busy = false;
        for (;;) {
            if (!busy && inside != 0) {
                i = (__ffs((int)inside) - 1) * TH + tid;
                inside &= inside - 1;
#pragma unroll
                for (int j = 0; j < N; ++j) t[j] = s_tok[i + j];
                u32 h = 0;
#pragma unroll
                for (int j = 0; j < N; ++j) h = light_step(h, t[j], j);
                idx = light_end(h) >> (31 - __builtin_ctz(C));
                busy = true;
            }
            if (__ballot(busy) == 0) break;
            if (busy) {
                // (the exchange at once: a look first would be one more round trip)
                const u32 sl = atomicCAS(&s_slot[idx], 0u, ((u32)(i + 1) << 16) | 1u);
                if (sl == 0) {
                    s_claim[i] = (uint16_t)idx;
                    mine |= 1u << (i / TH);
                    busy = false;
                } else {
                    const int p = (int)(sl >> 16) - 1;
                    bool eq = true;
#pragma unroll
                    for (int j = 0; j < N; ++j) eq = eq & (s_tok[p + j] == t[j]);
                    if (eq) {
                        atomicAdd(&s_slot[idx], 1u);
                        s_claim[i] = (uint16_t)idx;
                    }
                    busy = !eq;
                    idx = (idx + 1) & (2 * C - 1);         // (twice as many slots as windows: one is free)
                }
            }
        }
    }
    __syncthreads();

    // ---- the windows that are left, and how many records of a partition come before each
    const bool wide = N * bits > 64;
    u64 hash[W], hi[W];
    u32 cnt[W], rank[W];
#pragma unroll
    for (int w = 0; w < W; ++w) cnt[w] = s_slot[s_claim[w * TH + tid] & (2 * C - 1)] & 0xFFFFu;      // (of a window that is not alive: anything)
    if (keep_marks) {
#pragma unroll
        for (int w = 0; w < W; ++w) {
            const u64 live = __ballot((alive >> w) & 1), many = __ballot(((alive >> w) & 1) && cnt[w] > 1);
            if (lane == 0) {
                reinterpret_cast<u64*>(s_once)[(w * TH + tid) / 64] = ~live;
                reinterpret_cast<u64*>(s_often)[(w * TH + tid) / 64] = many;
            }
        }
    }
#pragma unroll
    for (int w = 0; w < W; ++w) {
        const u32* at = s_tok + w * TH + tid;
        u64 lo = 0;
        hi[w] = 0;
#pragma unroll
        for (int j = 0; j < N; ++j) tasc_key_put(lo, hi[w], j, bits, at[j]);
        hash[w] = tasc_hash_key(lo, hi[w]);
        if (!((mine >> w) & 1)) cnt[w] = 0;
        if (cnt[w]) rank[w] = atomicAdd(&s_hist[part_of(hash[w], parts)], (cnt[w] + 255) / 256);
    }
    __syncthreads();
    if (keep_marks && marks_mine) {
        // eight bits into eight bytes
        auto spread = [](u64 b) __attribute__((always_inline)) {
            return (((b * 0x0101010101010101ull & 0x8040201008040201ull) + 0x7F7F7F7F7F7F7F7Full) >> 7) & 0x0101010101010101ull;
        };
#pragma unroll
        for (int q = 0; q < (int)(sizeof e_in / 8); ++q) {
            const int g = q * TH + tid;
            const u64 at = base + 8 * g, v = spread(s_end[g]) * kMarkEnd | spread(s_once[g]) * kMarkOnce | spread(s_often[g]) * kMarkOften;
            if (at + 8 <= T) *reinterpret_cast<u64*>(marks + at) = v;
            else
                for (int e = 0; e < 8; ++e)
                    if (at + e < T) marks[at + e] = (uint8_t)(v >> (8 * e));
        }
    }
    // exclusive scan of the partitions' record counts, a run of consecutive partitions per thread
    const u32 per = ((parts + TH - 1) / TH) | 1, p0 = min(tid * per, parts), p1 = min(p0 + per, parts);     // (odd: no bank conflicts)
    u32 sum = 0, total;
    for (u32 p = p0; p < p1; ++p) sum += s_hist[p];
    u32 at = block_scan<TH>(sum, s_wave, total);
    for (u32 p = p0; p < p1; ++p) {
        const u32 n = s_hist[p];
        s_hist[p] = at;
        at += n;
    }
    __syncthreads();
    for (u32 p = tid; p <= parts; p += TH) offs[p] = (uint16_t)(p < parts ? s_hist[p] : total);
    // ---- records in order: put together in the slots' memory, stored as whole lines
    const u32 step = wide ? C / 2 : C;                     // records that fit there
    u64* s_rec = reinterpret_cast<u64*>(s_slot);
    for (u32 first = 0; first < total; first += step) {
#pragma unroll
        for (int w = 0; w < W; ++w) {
            if (!cnt[w]) continue;
            u32 to = s_hist[part_of(hash[w], parts)] + rank[w] - first;
            for (u32 n = cnt[w]; n > 0; ++to) {
                const u32 c = min(n, 256u);
                n -= c;
                if (to >= step) continue;
                const u64 r = (hash[w] << 8) | (c - 1);
                if (wide) reinterpret_cast<ulonglong2*>(s_rec)[to] = make_ulonglong2(r, hi[w]);
                else s_rec[to] = r;
            }
        }
        __syncthreads();
        const u32 here = min(total - first, step), units = wide ? here : (here + 1) / 2;     // of 16 bytes
        ulonglong2* dst = reinterpret_cast<ulonglong2*>(rec) + (wide ? base + first : (base + first) / 2);
        for (u32 u = tid; u < units; u += TH) dst[u] = reinterpret_cast<const ulonglong2*>(s_rec)[u];
        __syncthreads();
    }
}

struct PartitionArgs {
    const int32_t* tok;
    const u64* d_T;            // nullable: the corpus' length, where the host does not know it (T is then no less)
    uint8_t* marks;            // kMark... of a position
    bool keep_marks;           // leave those for the order above
    u64 T;
    int32_t bits, n0;          // n0 + blockIdx.y = order of the launch's block
    u32 parts, row;            // row = parts + 1, rounded up: a chunk's offsets
    const u32* twice;          // nullable: [2^twice_bits / 32], see partition_chunk
    int32_t twice_bits;
    u64* distinct;             // += n-grams that left no record
    size_t order_recs;         // 8-byte words of an order's records
    u64* rec;                  // [orders][chunks C] of 8 bytes, or 16 for keys of more than 64 bits
    uint16_t* offs;            // [orders][chunks][row]
};
template <int C, int TH>
__global__ __launch_bounds__(TH) void k_partition(PartitionArgs a) {
    if (a.d_T) a.T = *a.d_T;
    if ((u64)blockIdx.x * C >= a.T) return;
    const int n = a.n0 + blockIdx.y;
    u64* const rec = a.rec + blockIdx.y * a.order_recs;
    uint16_t* const offs = a.offs + ((size_t)blockIdx.y * gridDim.x + blockIdx.x) * a.row;
    switch (n) {
        case 2: partition_chunk<2, C, TH>(a.tok, a.marks, a.keep_marks, a.T, a.bits, a.parts, a.twice, a.twice_bits, a.distinct, rec, offs); break;
        case 3: partition_chunk<3, C, TH>(a.tok, a.marks, a.keep_marks, a.T, a.bits, a.parts, a.twice, a.twice_bits, a.distinct, rec, offs); break;
        case 4: partition_chunk<4, C, TH>(a.tok, a.marks, a.keep_marks, a.T, a.bits, a.parts, a.twice, a.twice_bits, a.distinct, rec, offs); break;
        case 5: partition_chunk<5, C, TH>(a.tok, a.marks, a.keep_marks, a.T, a.bits, a.parts, a.twice, a.twice_bits, a.distinct, rec, offs); break;
        case 6: partition_chunk<6, C, TH>(a.tok, a.marks, a.keep_marks, a.T, a.bits, a.parts, a.twice, a.twice_bits, a.distinct, rec, offs); break;
        case 7: partition_chunk<7, C, TH>(a.tok, a.marks, a.keep_marks, a.T, a.bits, a.parts, a.twice, a.twice_bits, a.distinct, rec, offs); break;
        default: partition_chunk<8, C, TH>(a.tok, a.marks, a.keep_marks, a.T, a.bits, a.parts, a.twice, a.twice_bits, a.distinct, rec, offs); break;
    }
}

// [chunks][row] -> [row][chunks], both padded to whole tiles of 64: with the offsets as they are written, every lane of k_tables would
// read lines of its own for two offsets
__global__ __launch_bounds__(256) void k_turn(const uint16_t* __restrict__ in, u32 row, u32 col, u32 chunks, uint16_t* __restrict__ out) {
    __shared__ uint16_t s[64][66];
    const u32 p0 = blockIdx.x * 64, c0 = blockIdx.y * 64;
    for (int q = threadIdx.x; q < 64 * 32; q += 256) {
        const u32 c = c0 + q / 32;
        const u32 v = c < chunks ? *reinterpret_cast<const u32*>(in + (size_t)c * row + p0 + 2 * (q % 32)) : 0;
        s[q / 32][2 * (q % 32)] = (uint16_t)v;
        s[q / 32][2 * (q % 32) + 1] = (uint16_t)(v >> 16);
    }
    __syncthreads();
    for (int q = threadIdx.x; q < 64 * 32; q += 256) {
        const int p = q / 32, c = 2 * (q % 32);
        *reinterpret_cast<u32*>(out + (size_t)(p0 + p) * col + c0 + c) = (u32)s[c][p] | ((u32)s[c + 1][p] << 16);
    }
}

constexpr int kTabThreads = 768;
constexpr int kSlotsNarrow = 5376, kSlotsWide = 3072;      // 60 KB of tables: two workgroups per compute unit
constexpr int kPrimeNarrow = 5351, kPrimeWide = 3067;      // (primes: any step visits all of them)
constexpr int kStageNarrow = 1536, kStageWide = 768;       // records on their way into the table: 12 KB
constexpr int kRuns = 4;                                   // chunks of a thread at a time
constexpr u64 kLow57 = (1ull << 57) - 1;
constexpr int kMaxProbe = 128;                             // a longer probe sequence means a table that is as good as full
constexpr u32 kMostRounds = 256;
// A range that overflows is cut in two, by the hash down to kFinest ranges of a partition (one value of the hash's upper half each), then
// by the rest of the key: (hash, hi) is the key, so a range of the finest kind holds one n-gram, and no corpus can fail.  Behind
// a dense spot the ranges grow again, up to kCoarse times as many as at the start.
constexpr u32 kFinest = 1u << 24, kCoarse = 8;
typedef unsigned __int128 u128;
template <bool WIDE>
constexpr u128 kPlaces = (u128)1 << (WIDE ? 120 : 56);
template <bool WIDE>
__device__ __forceinline__ u128 place_of(u64 rec, u64 hi) {                // of a key among those of one value of the hash's upper half
    const u64 low = rec >> 8, h = ((low << 24) | (low >> 32)) & ((1ull << 56) - 1);      // (the bits that still differ first)
    return WIDE ? ((u128)(hi * 0x9E3779B97F4A7C15ull) << 56) | h : h;
}

struct TablesArgs {
    const u64* rec;
    const uint16_t* offs;
    size_t order_recs, order_offs;     // from one order to the next
    u32 chunk_step, part_step;         // offs[chunk * chunk_step + partition * part_step]
    u32 chunks, chunk, parts;
    const u64* d_T;            // nullable, as above (chunks is then an upper bound)
    int32_t n, bits;
    u32 p_min, rounds;         // rounds: ranges that a partition is cut into from the start
    u64* counters;             // [0] distinct n-grams, [1] kept n-grams
    TascKept kept;
    u32* twice;                // nullable: see k_partition
    int32_t twice_bits;
    TascGram* best;            // [orders][parts] the partition's n-gram with the largest count, smallest tuple among equals
    u64* deal;                 // room for deal_recs records per workgroup
    u32 deal_recs;
};

template <bool WIDE>
constexpr int table_bytes() { return WIDE ? kSlotsWide * 20 : kSlotsNarrow * 12; }
template <bool WIDE>
constexpr int tables_lds() { return table_bytes<WIDE>() + (WIDE ? kStageWide * 16 : kStageNarrow * 8); }

// BEST: no list, but the most frequent n-gram of the workgroup's partition.
// A partition is counted in `rounds` ranges, one table after the other, and each gathers all of the partition's records and drops those
// of the others.  DEAL, for many rounds: the records are gathered twice, to count those of every round and to lay them out round by
// round in memory of the workgroup's own, as many rounds at a time as fit there (one that does not fit alone gathers for itself).  Where all
// of them together are more than that, a few n-grams may be most of the corpus: the whole partition is tried in one table first, until that is full.
template <bool WIDE, bool BEST, bool DEAL>
__device__ __forceinline__ void partition_table(const TablesArgs& a, u32 part, TascGram* best_out) {
    constexpr int SLOTS = WIDE ? kSlotsWide : kSlotsNarrow, PRIME = WIDE ? kPrimeWide : kPrimeNarrow, PER = SLOTS / kTabThreads;
    constexpr int STAGE = WIDE ? kStageWide : kStageNarrow, RW = WIDE ? 2 : 1, MINE = STAGE / kTabThreads;
    static_assert(SLOTS % kTabThreads == 0 && STAGE % kTabThreads == 0 && table_bytes<WIDE>() % 16 == 0, "slots and records per thread; clearing");
    extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
    u64* s_key = reinterpret_cast<u64*>(lds);                                  // {low 56 bits of the hash, 1, upper 7 bits of hi}; 0 = free
    u64* s_hi = s_key + SLOTS;                                                 // WIDE only: {1 : 7, low 57 bits of hi}; 0 = nobody's yet
    u32* s_cnt = reinterpret_cast<u32*>(s_key + RW * SLOTS);
    u64* s_rec = reinterpret_cast<u64*>(lds + table_bytes<WIDE>());            // first where they are, then the records
    __shared__ u32 s_full, s_nn, s_wave[2][kTabThreads / 64];
    __shared__ u64 s_at;
    __shared__ u128 s_place, s_places;                     // the part of a finest range that is being counted
    __shared__ u32 s_len[DEAL ? kMostRounds : 1], s_end[DEAL ? kMostRounds : 1], s_next;      // DEAL: rounds' records; the end of what is laid out of them; end of the laid out rounds
    const int tid = threadIdx.x, lane = tid & 63;
    auto hi_of = [&](u64 key, int i) { return WIDE ? ((key & 0x7F) << 57) | (s_hi[i] & kLow57) : 0ull; };
    TascGram best{0, 0, 0, 0};
    u32 distinct = 0;                                      // (a thread's are fewer than the corpus' positions)
    const u32 runs = a.chunks > 2 * kTabThreads ? kRuns : a.chunks > kTabThreads ? 2 : 1;
    const uint16_t* const offs = a.offs + (size_t)part * a.part_step;
    u64* const deal = DEAL ? a.deal + (size_t)blockIdx.x * a.deal_recs * RW : nullptr;

    u32 fine = 1, num = 0;                                 // the range that is being counted: num of rounds x fine
    bool within = false;                                   // only s_place .. of it
    bool dealt = false;                                    // its round's records lie in `deal`
    bool whole = false;                                    // DEAL: the whole partition is tried in one
    // which of den ranges: from the lower half of the product that chose the partition
    auto range_of = [&](u64 r, u32 den) { return (u32)(((u64)((u32)(hash_of(r, part, a.parts) >> 32) * a.parts) * den) >> 32); };

    // every thread inserts the records of s_rec that it put there; a lane probes once per turn
    auto insert = [&](u32 here) __attribute__((always_inline)) {
        u32 e = tid, idx = 0, step = 0, c = 0;
        int probes = 0;
        u64 key = 0, hv = 0;
        bool busy = false;
        for (;;) {
            if (!busy && e < here) {
                const u64 r = s_rec[RW * e];
                const u64 hi = WIDE ? s_rec[RW * e + RW - 1] : 0;
                e += kTabThreads;
                busy = true;
                if ((DEAL && (dealt || whole) ? 1 : a.rounds) * fine > 1) {
                    busy = range_of(r, a.rounds * fine) == num;
                    if (within) busy = busy && place_of<WIDE>(r, hi) - s_place < s_places;
                }
                key = (r & ~0xFFull) | 0x80 | (hi >> 57);
                hv = (hi & kLow57) | ~kLow57;
                c = (u32)(r & 0xFF) + 1;
                idx = __umulhi((u32)(r >> 8), (u32)PRIME);
                step = ((u32)(r >> 20) & 1023) + 1;
                probes = 0;
            }
            if (__ballot(busy || e < here) == 0) break;
            if (!busy) continue;
            // Nobody waits for anybody: a slot whose hash is there without its hi takes the hi of whoever comes first, and the
            // one that claimed it goes on where that was another's.
            const u64 k = atomicCAS(&s_key[idx], 0ull, key);
            bool mine = k == 0 || k == key;
            if (WIDE && mine) {
                const u64 v = atomicCAS(&s_hi[idx], 0ull, hv);
                mine = v == 0 || v == hv;
            }
            if (mine) atomicAdd(&s_cnt[idx], c);
            busy = !mine;
            idx += step;
            idx -= idx >= (u32)PRIME ? PRIME : 0;
            if (busy && ++probes == kMaxProbe) {
                s_full = 1;
                busy = false;
            }
        }
    };
    // the records src[e] of `from`, e < here, through s_rec into the table
    auto load_insert = [&](const u64* from, u32 here, auto src) __attribute__((always_inline)) {
        u64 r[MINE][RW];
#pragma unroll
        for (int k = 0; k < MINE; ++k) {
            const u32 e = k * kTabThreads + tid;
            if (e < here) {
                if constexpr (WIDE) {
                    const ulonglong2 v = reinterpret_cast<const ulonglong2*>(from)[src(e)];
                    r[k][0] = v.x;
                    r[k][1] = v.y;
                } else {
                    r[k][0] = from[src(e)];
                }
            }
        }
#pragma unroll
        for (int k = 0; k < MINE; ++k) {
            const u32 e = k * kTabThreads + tid;
            if (e < here) {
                if constexpr (WIDE) reinterpret_cast<ulonglong2*>(s_rec)[e] = make_ulonglong2(r[k][0], r[k][1]);
                else s_rec[e] = r[k][0];
            }
        }
        insert(here);
    };
    // all records of the partition, STAGE at a time: use(how many), with where they are in s_rec; returns how many in all
    auto gather = [&](auto use) __attribute__((always_inline)) {
        u32 all = 0;
        for (u32 c0 = 0; c0 < a.chunks; c0 += runs * kTabThreads) {
            // the thread's runs and their place among the records of these chunks
            u32 at[kRuns], len[kRuns], sum = 0, total;
#pragma unroll
            for (int u = 0; u < kRuns; ++u) {
                const u32 c = c0 + tid * runs + u;
                at[u] = len[u] = 0;
                if (u < (int)runs && c < a.chunks) {
                    at[u] = offs[(size_t)c * a.chunk_step];
                    len[u] = offs[(size_t)c * a.chunk_step + a.part_step] - at[u];
                }
                sum += len[u];
            }
            const u32 before = block_scan<kTabThreads>(sum, s_wave[(c0 / (runs * kTabThreads)) & 1], total);
            for (u32 first = 0; first < total; first += STAGE) {
                u32 to = before;
#pragma unroll
                for (int u = 0; u < kRuns; ++u) {
                    // (only the part of a run that belongs here: an n-gram that fills its chunks has 32 records in each)
                    u32 from = 0, end = len[u];
                    if (total > (u32)STAGE) {
                        from = min(max(to, first) - to, end);
                        end = min(max(first + STAGE, to) - to, end);
                    }
                    for (u32 j = from; j < end; ++j) reinterpret_cast<u32*>(s_rec + RW * (to + j - first))[0] = (c0 + tid * runs + u) * a.chunk + at[u] + j;
                    to += len[u];
                }
                __syncthreads();
                use(min(total - first, (u32)STAGE));
                __syncthreads();
                if (DEAL && whole && s_full) return all;
            }
            all += total;
        }
        return all;
    };
    auto gathered = [&](u32 e) { return reinterpret_cast<const u32*>(s_rec + RW * e)[0]; };

    if (DEAL) {
        for (u32 i = tid; i < a.rounds; i += kTabThreads) s_len[i] = 0;
        whole = gather([&](u32 here) __attribute__((always_inline)) {
#pragma unroll
            for (int k = 0; k < MINE; ++k) {
                const u32 e = k * kTabThreads + tid;
                if (e < here) atomicAdd(&s_len[range_of(a.rec[(size_t)RW * gathered(e)], a.rounds)], 1u);
            }
        }) > a.deal_recs;                                  // (more records than it should have: few n-grams, maybe, often)
    }
    for (u32 round = 0, end; round < a.rounds; round = end) {
        end = a.rounds;
        dealt = false;
        if (DEAL && !whole) {
            if (tid == 0) {
                u32 r = round;
                for (u32 sum = 0; r < a.rounds && s_len[r] <= a.deal_recs - sum; ++r) {
                    s_end[r] = sum;
                    sum += s_len[r];
                }
                s_next = r;
            }
            __syncthreads();
            dealt = s_next > round;
            end = dealt ? s_next : round + 1;
            if (dealt) {
                gather([&](u32 here) __attribute__((always_inline)) {
#pragma unroll
                    for (int k = 0; k < MINE; ++k) {
                        const u32 e = k * kTabThreads + tid;
                        if (e >= here) continue;
                        const u32 src = gathered(e);
                        u64 r, hi = 0;
                        if constexpr (WIDE) {
                            const ulonglong2 v = reinterpret_cast<const ulonglong2*>(a.rec)[src];
                            r = v.x;
                            hi = v.y;
                        } else {
                            r = a.rec[src];
                        }
                        const u32 to = range_of(r, a.rounds);
                        if (to < round || to >= end) continue;
                        const u32 at = atomicAdd(&s_end[to], 1u);
                        if constexpr (WIDE) reinterpret_cast<ulonglong2*>(deal)[at] = make_ulonglong2(r, hi);
                        else deal[at] = r;
                    }
                });
            }
        }
        fine = 1;
        num = round;
        while (num < (DEAL && whole ? 1 : end * fine)) {
            for (int i = tid; i < table_bytes<WIDE>() / 16; i += kTabThreads) reinterpret_cast<ulonglong2*>(lds)[i] = make_ulonglong2(0, 0);
            if (tid == 0) s_full = s_nn = 0;
            if (DEAL && dealt) {
                const u32 n = s_len[num / fine];
                const u64* const from = deal + (size_t)RW * (s_end[num / fine] - n);
                __syncthreads();
                for (u32 first = 0; first < n; first += STAGE)           // (a thread's records are its own: no barriers)
                    load_insert(from + (size_t)RW * first, min(n - first, (u32)STAGE), [](u32 e) { return e; });
            } else {
                gather([&](u32 here) __attribute__((always_inline)) { load_insert(a.rec, here, gathered); });
            }
            __syncthreads();
            if (s_full) {                                      // more n-grams than slots: the range in two halves
                __syncthreads();
                if (DEAL && whole) {                       // they are not few: round by round after all
                    whole = false;
                    end = 0;
                    break;
                }
                if (a.rounds * fine < kFinest) {
                    fine *= 2;
                    num *= 2;
                } else {
                    if (tid == 0) {
                        if (!within) s_place = 0;
                        s_places = within ? s_places / 2 : kPlaces<WIDE> / 2;
                    }
                    within = true;
                }
                continue;
            }
            u32 keep = 0, most = 0;
            auto set_bit = [&](int i) {
                const u64 hi = hi_of(s_key[i], i), lo = tasc_hash_lo(hash_of(s_key[i], part, a.parts), hi);
                u32 h = 0;
                for (int j = 0; j < a.n; ++j) {
                    const u32 t = tasc_key_get(lo, hi, j, a.bits), r = 13 * j % 32;
                    h ^= r == 0 ? t : (t << r) | (t >> (32 - r));
                }
                h = light_end(h) >> (32 - a.twice_bits);
                atomicOr(&a.twice[h >> 5], 1u << (h & 31));
            };
#pragma unroll
            for (int s = 0; s < PER; ++s) {
                const int i = s * kTabThreads + tid;
                if (s_key[i] == 0) continue;
                ++distinct;
                if (s_cnt[i] >= a.p_min) ++keep;
                most = max(most, s_cnt[i]);
                if (!BEST && a.twice && s_cnt[i] > 1) {
                    const u32 q = atomicAdd(&s_nn, 1u);
                    if (q < (u32)STAGE) reinterpret_cast<u32*>(s_rec)[q] = i;
                    else set_bit(i);
                }
            }
            if (!BEST && a.twice) {                            // (few slots have a bit to set: one a lane, once they are known)
                __syncthreads();
                for (u32 q = tid; q < min(s_nn, (u32)STAGE); q += kTabThreads) set_bit((int)reinterpret_cast<const u32*>(s_rec)[q]);
            }
            if (BEST) {
                // only what has the largest count is taken apart
                for (int o = 32; o > 0; o >>= 1) most = max(most, (u32)__shfl_xor((int)most, o));
                if (lane == 0) s_wave[0][tid >> 6] = most;
                __syncthreads();
                for (int w = 0; w < kTabThreads / 64; ++w) most = max(most, s_wave[0][w]);
                for (int i = tid; i < SLOTS && most >= best.count; i += kTabThreads) {
                    const u64 key = s_key[i];
                    if (key == 0 || s_cnt[i] != most) continue;
                    const u64 hi = hi_of(key, i);
                    const TascGram g{tasc_hash_lo(hash_of(key, part, a.parts), hi), hi, most, (u32)a.n};
                    if (tasc_gram_before(g, best, a.bits)) best = g;
                }
            }
            if (!BEST) {
                // the kept n-grams behind those of other workgroups: one addition per workgroup and range
                u32 all;
                const u32 before = block_scan<kTabThreads>(keep, s_wave[0], all);
                if (tid == 0) s_at = all ? atomicAdd(&a.counters[1], (u64)all) : 0;
                __syncthreads();
                u64 to = s_at + before;
                if (keep) {
#pragma unroll
                    for (int s = 0; s < PER; ++s) {
                        const int i = s * kTabThreads + tid;
                        const u64 key = s_key[i];
                        const u32 c = s_cnt[i];
                        if (key == 0 || c < a.p_min) continue;
                        const u64 hi = hi_of(key, i);
                        a.kept.lo[to] = tasc_hash_lo(hash_of(key, part, a.parts), hi);
                        a.kept.hi[to] = hi;
                        a.kept.count[to] = c;
                        ++to;
                    }
                }
            }
            __syncthreads();
            if (within) {                                      // on to the next part, of the largest size that begins there
                if (tid == 0) {
                    s_place += s_places;
                    s_places = s_place & (~s_place + 1);
                }
                __syncthreads();
                within = s_place != kPlaces<WIDE>;
                __syncthreads();
                if (within) continue;
            }
            ++num;
            while (fine > kCoarse && num % 2 == 0) {
                fine /= 2;
                num /= 2;
            }
        }
    }
    if (BEST) {
        TascGram* s_best = reinterpret_cast<TascGram*>(lds);
        static_assert(kTabThreads <= 1024 && kTabThreads * sizeof(TascGram) <= table_bytes<false>(), "a candidate per thread in the tables' LDS");
        s_best[tid] = best;
        __syncthreads();
        for (int w = 512; w > 0; w >>= 1) {
            if (tid < w && tid + w < kTabThreads && tasc_gram_before(s_best[tid + w], s_best[tid], a.bits)) s_best[tid] = s_best[tid + w];
            __syncthreads();
        }
        if (tid == 0) *best_out = s_best[0];
    } else {
        u32 n = distinct;
        for (int o = 32; o > 0; o >>= 1) n += __shfl_xor(n, o);
        if (lane == 0) s_wave[0][tid >> 6] = n;
        __syncthreads();
        if (tid == 0) {
            u64 all = 0;
            for (int w = 0; w < kTabThreads / 64; ++w) all += s_wave[0][w];
            if (all) atomicAdd(&a.counters[0], all);
        }
    }
}

// The partition number i, i % 8 the XCD of its workgroup (the dispatcher deals ids to the 8 XCDs in turn): each XCD takes one contiguous
// range of the partitions, so that the records of neighbouring partitions, which share cache lines, are read into one L2.
__device__ inline u32 my_part(u32 i, u32 parts) {
    const u32 xcd = i % 8;
    return xcd * (parts / 8) + min(xcd, parts % 8) + i / 8;
}
// A partition per workgroup, or, with records dealt, one after the other in the workgroup's memory
constexpr u32 kDealWgs = 512;                              // two per compute unit; a multiple of 8
template <bool WIDE, bool DEAL>
__global__ __launch_bounds__(kTabThreads) __attribute__((amdgpu_waves_per_eu(6, 6))) void k_tables(TablesArgs a) {
    if (!DEAL) partition_table<WIDE, false, false>(a, my_part(blockIdx.x, a.parts), nullptr);
    else
        for (u32 i = blockIdx.x; i < a.parts; i += gridDim.x) {
            partition_table<WIDE, false, true>(a, my_part(i, a.parts), nullptr);
            __syncthreads();
        }
}

// every order n + blockIdx.y (one order only with records dealt)
template <bool DEAL>
__global__ __launch_bounds__(kTabThreads) __attribute__((amdgpu_waves_per_eu(6, 6))) void k_tables_best(TablesArgs a) {
    const u32 y = blockIdx.y;
    a.n += (int32_t)y;
    a.rec += y * a.order_recs;
    a.offs += y * a.order_offs;
    a.best += (size_t)y * a.parts;
    if (a.d_T) a.chunks = (u32)((*a.d_T + a.chunk - 1) / a.chunk);
    for (u32 i = blockIdx.x; i < a.parts; i += gridDim.x) {
        if (a.n * a.bits > 64) partition_table<true, true, DEAL>(a, my_part(i, a.parts), a.best + i);
        else partition_table<false, true, DEAL>(a, my_part(i, a.parts), a.best + i);
        if (!DEAL) return;
        __syncthreads();
    }
}

constexpr int kChunkLarge = 8192, kThreadsLarge = 1024, kChunkSmall = 2048, kThreadsSmall = 512;
size_t partition_lds(u32 chunk, u32 parts) { return (size_t)(2 * chunk + chunk + 8 + parts + 1 + 16) * 4 + 2 * (size_t)chunk + 3 * (chunk / 8 + 8); }
u32 up64(u32 v) { return (v + 63) / 64 * 64; }

}  // namespace

// Chunks of 8192 positions merge more windows (of 32 M tokens 0.55 / 0.84 of the 2- / 5-grams are left, 0.65 / 0.89 with 2048)
// and leave longer runs of a partition, but they need 2 M tokens to fill the chip.  A partition is as many windows as there
// are LDS slots: about half of a corpus' windows are distinct (0.21 to 0.51 of the 2- to 5-grams of 24 M tokens), and where
// nearly all are, it is cut in two; twice as many where most of the unique ones leave no record.  Offsets are turned round where there are many chunks.
// The partitions' counters fit LDS up to TASC_COUNT_MAX_PARTS of them; what a larger corpus has more is counted in rounds.  Where every
// round gathers a partition's records for itself, the time grows with the square of the corpus; records that are laid out by round cost
// two gatherings, a write and a read whatever the rounds are.  Builds of orders 2 to 5, every round for itself | laid out from kDealFrom rounds on, ms:
// 320 M tokens of a phrase corpus 70.6 | 57.8, 640 M 258 | 136, 1.28 G 999 | 281, 4.2 G 10440 | 978; random ones 640 M 250 | 87.
// With two rounds it is no gain unless nearly all windows are distinct (160 M 24.3 | 27.8, random 30.9 | 18.0).
// (A few n-grams that are the whole corpus leave most partitions empty: 1 G tokens of four values 93, of one alone 286, 600 before whole
// partitions were tried; a table of atomics in memory 234 and 100.)
constexpr u64 kDealFrom = 3;
TascCountPlan tasc_count_plan(u64 T, u64 windows, bool wide, bool pruned) {
    TascCountPlan p;
    p.chunk = T >= (u64)256 * kChunkLarge ? kChunkLarge : kChunkSmall;
    p.chunks = (u32)((T + p.chunk - 1) / p.chunk);
    const u64 slots = wide ? kSlotsWide : kSlotsNarrow, per = pruned ? 2 * slots : slots;
    p.parts = (u32)std::clamp<u64>((windows + per - 1) / per, TASC_COUNT_MIN_PARTS, TASC_COUNT_MAX_PARTS);
    p.rounds = (u32)std::max<u64>(1, windows / p.parts / per);
    p.rec_bytes = (size_t)p.chunks * p.chunk * (wide ? 16 : 8);
    p.deal_recs = 0;
    if (windows >= (u64)kDealFrom * per * p.parts) {
        p.rounds = (u32)std::min<u64>(kMostRounds, (windows + per * p.parts - 1) / (per * p.parts));
        p.deal_recs = (u32)(2 * windows / p.parts);
    }
    p.deal_bytes = (size_t)kDealWgs * p.deal_recs * (wide ? 16 : 8);
    p.offs_bytes = (size_t)up64(p.chunks) * up64(p.parts + 1) * sizeof(uint16_t) * (p.chunk == kChunkLarge ? 2 : 1);
    return p;
}

// a bit for every two tokens or so: of 24 M tokens' windows, the distinct n-grams that occur more than once are 2 to 3 %, and the map of 32 M
// tokens lies in an XCD's L2 (8 instead of 2 MB: k_partition 498 / 563 / 583 us for orders 3 to 5, 469 / 523 / 533 so)
int tasc_twice_bits(u64 T) {
    int b = 16;
    while (b < 32 && (1ull << b) < T / 2) ++b;
    return b;
}

tasc_status tasc_count_partition(const TascCountPlan& p, const int32_t* d_tok, uint8_t* d_marks, bool keep_marks, u64 T, const u64* d_T, int32_t n0,
                                 int32_t n_orders, int32_t bits, const TascCountBufs& b, const u32* d_twice, u64* d_counters, hipStream_t st) {
    const u32 row = up64(p.parts + 1);
    PartitionArgs a{d_tok, d_T, d_marks, keep_marks, T, bits, n0, p.parts, row, d_twice, tasc_twice_bits(T), d_counters, p.rec_bytes / sizeof(u64), b.rec, b.offs};
    const size_t lds = partition_lds(p.chunk, p.parts);
    auto launch = [&](auto kernel, int threads) -> tasc_status {
        TASC_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize,
                                     (int)partition_lds(p.chunk, TASC_COUNT_MAX_PARTS)));
        kernel<<<dim3(p.chunks, (unsigned)n_orders), dim3(threads), lds, st>>>(a);
        TASC_LAUNCH_CHECK();
        return TASC_OK;
    };
    if (p.chunk != kChunkLarge) return launch(&k_partition<kChunkSmall, kThreadsSmall>, kThreadsSmall);
    const tasc_status rc = launch(&k_partition<kChunkLarge, kThreadsLarge>, kThreadsLarge);
    if (rc != TASC_OK) return rc;
    const u32 col = up64(p.chunks);
    const size_t one = (size_t)col * row;
    for (int y = 0; y < n_orders; ++y) {
        k_turn<<<dim3(row / 64, col / 64), dim3(256), 0, st>>>(b.offs + (size_t)y * p.chunks * row, row, col, p.chunks, b.offs + n_orders * one + y * one);
        TASC_LAUNCH_CHECK();
    }
    return TASC_OK;
}

static TablesArgs tables_args(const TascCountPlan& p, const u64* d_T, int32_t n, int32_t n_orders, int32_t bits, u32 p_min, const TascCountBufs& b,
                              u64* d_counters, const TascKept& kept, TascGram* d_best) {
    const u32 row = up64(p.parts + 1), col = up64(p.chunks);
    const bool turned = p.chunk == kChunkLarge;
    return TablesArgs{b.rec, turned ? b.offs + (size_t)n_orders * col * row : b.offs, p.rec_bytes / sizeof(u64),
                      turned ? (size_t)col * row : (size_t)p.chunks * row, turned ? 1 : row, turned ? col : 1,
                      p.chunks, p.chunk, p.parts, d_T, n, bits, p_min, p.rounds, d_counters, kept, nullptr, 0, d_best, b.deal, p.deal_recs};
}

tasc_status tasc_count_tables(const TascCountPlan& p, int32_t n, int32_t bits, u32 p_min, const TascCountBufs& b, u64* d_counters,
                              const TascKept& kept, u32* d_twice, u64 T, hipStream_t st) {
    TablesArgs a = tables_args(p, nullptr, n, 1, bits, p_min, b, d_counters, kept, nullptr);
    a.twice = d_twice;
    a.twice_bits = tasc_twice_bits(T);
    auto launch = [&](auto kernel, int lds) -> tasc_status {
        TASC_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, lds));
        kernel<<<dim3(p.deal_recs ? std::min(p.parts, kDealWgs) : p.parts), dim3(kTabThreads), lds, st>>>(a);
        TASC_LAUNCH_CHECK();
        return TASC_OK;
    };
    if (n * bits > 64) return p.deal_recs ? launch(&k_tables<true, true>, tables_lds<true>()) : launch(&k_tables<true, false>, tables_lds<true>());
    return p.deal_recs ? launch(&k_tables<false, true>, tables_lds<false>()) : launch(&k_tables<false, false>, tables_lds<false>());
}

tasc_status tasc_count_best(const TascCountPlan& p, const u64* d_T, int32_t n0, int32_t n_orders, int32_t bits, const TascCountBufs& b,
                            TascGram* d_best, hipStream_t st) {
    const TablesArgs a = tables_args(p, d_T, n0, n_orders, bits, 1, b, nullptr, TascKept{}, d_best);
    constexpr int lds = std::max(tables_lds<false>(), tables_lds<true>());
    auto launch = [&](auto kernel, const TablesArgs& one, dim3 grid) -> tasc_status {
        TASC_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, lds));
        kernel<<<grid, dim3(kTabThreads), lds, st>>>(one);
        TASC_LAUNCH_CHECK();
        return TASC_OK;
    };
    if (!p.deal_recs) return launch(&k_tables_best<false>, a, dim3(p.parts, (unsigned)n_orders));
    for (int y = 0; y < n_orders; ++y) {                   // (in turn: they deal into the same memory)
        TablesArgs one = a;
        one.n += y;
        one.rec += y * a.order_recs;
        one.offs += y * a.order_offs;
        one.best += (size_t)y * p.parts;
        const tasc_status rc = launch(&k_tables_best<true>, one, dim3(std::min(p.parts, kDealWgs)));
        if (rc != TASC_OK) return rc;
    }
    return TASC_OK;
}
