// The tiled bf16 GEMM of forwards of more than 16 rows: out[M, N] = epilogue(A[M, K] W[N, K]^T), both operands k-contiguous.
//
// A workgroup computes BN (output features) x BM (rows) tiles with v_mfma_f32_32x32x16_bf16, the WEIGHT rows as the A operand,
// so a lane ends up with runs of 4 consecutive features of one row.  k advances in stages of SK; ST stages sit in LDS at once,
// filled by loads that go from memory to LDS without passing through registers.  The stages of a workgroup's tiles form ONE
// stream: while the last stages of a tile are multiplied, and while its epilogue runs, the first stages of its next tile are
// already on their way, so a tile pays neither a launch nor a cold first fetch, and the stores of its epilogue drain under
// the next tile's products.
//
// A row's result depends only on its own data and the fixed k order (16 at a time, ascending), not on the tile shape, the
// number of rows or the number of workgroups.
//
// What bounds it: with random operands the matrix cores alone, at the clock the card then holds, take 430 us for
// 16384 x 2048 x 11008 (1.7 PFLOP/s), with the fragment reads 480 us, with the loads from L2 575 us; the stores of two rounds of
// tiles and misses of L2 bring it to 610-640 us.  8 waves of 128 x 64 rather than 4 of 128 x 128: the second wave of a SIMD
// covers the first one's waits (635 against 650-690 us).  Padded rows in LDS are not needed: the swizzle below leaves 2 % of the
// LDS cycles in conflicts.  In the forwards, before -> now: gate/up of a 16384-row prompt chunk (N 22016, k 2048) 1327 -> 1248 us,
// q/k/v 240 -> 206; LM head with logits 1280 x 49152 x 2048 499 -> 296, 576 x 151936 x 1536 510 -> 357 (whole rows of 128 bytes per
// store instead of 4-byte stores to 32 rows).
#pragma once
#include "kernels_small.h"

typedef __attribute__((ext_vector_type(16))) float f32x16;

#define TG_BK 64                                              // k granularity of slices: K is a multiple of it
#define TG_MAX_SLICES 8                                       // most k-slices of a narrow GEMM

// TEPI_PARTIAL: k is cut into `slices` ranges; a slice's sums go to outf[slice][M][N] and k_splitk_reduce (or a kernel that
// fuses it) adds the slices in order.  Used where N is too narrow for the tile count to fill the chip; the number of slices
// depends on N and K only.
// TEPI_ROPE: the fused q/k/v projection of a layer whose output is not sliced: the epilogue rotates the q and k heads (RoPE
// at the row's position), writes q to outb and the new k / v rows straight into the row's cache page.
enum { TEPI_STORE = 0, TEPI_RESID = 1, TEPI_SWIGLU = 2, TEPI_LMHEAD = 3, TEPI_PARTIAL = 4, TEPI_ROPE = 5 };

struct RopeEpi {          // TEPI_ROPE only: what k_rope_kv takes
    const float* cosT;        // [max_pos][hd / 2]
    const float* sinT;
    const int32_t* n_rows;    // [B] active rows of the sequence
    const int32_t* pos0;      // [B] position of the sequence's first row
    const int32_t* block_tab; // [B][max_blocks]
    BF16* kv_layer;           // the layer's pages
    KvGeom gm;
    int32_t max_pos;
};

struct LmEpi {            // TEPI_LMHEAD only
    BiasCsr bias;
    const int32_t* bias_ptr;  // [M][n_strips + 1] cursor table
    const int64_t* row_first; // [M] first entry of the row's bias list
    const float* row_base;    // [M] the row's bias of unseen successors
    float* part_val;          // [M][n_strips]
    int32_t* part_idx;
    float* logits;            // nullable [M][V]
    int32_t n_strips;
};

// rows of the accumulator a lane holds: element i of a 32x32 tile is output feature 8 (i / 4) + 4 (lane / 32) + i % 4
__device__ inline int tile_row(int i, int lane) { return 8 * (i >> 2) + 4 * (lane >> 5) + (i & 3); }

typedef float f32x4_u __attribute__((ext_vector_type(4), aligned(4)));    // four floats at any 4-byte address
typedef float f32x2_u __attribute__((ext_vector_type(2), aligned(4)));
typedef uint32_t u32x2_u __attribute__((ext_vector_type(2), aligned(4)));
typedef uint32_t u32x4_u __attribute__((ext_vector_type(4), aligned(4)));

constexpr int gemm_lds_bytes(int BN, int BM, int WN, int WM, int SK, int ST) { return ST * (BN + BM) * SK * 2 + WN * WM * 4096; }

// The order of a k-block of X products: its R fragment reads go out between the products of the first half (after the first one,
// whose wait for the block's own fragments so covers no newer read; they have the second half to arrive), its L loads between
// the products of the second half.
template <int R, int X, int L, int x = 0>
__device__ __forceinline__ void interleave() {
    constexpr int H = (X + 1) / 2;
    constexpr int r = x < H ? (x + 1) * R / H - x * R / H : 0;
    constexpr int l = x >= H ? (x + 1 - H) * L / (X - H) - (x - H) * L / (X - H) : 0;
    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);                            // MFMA
    if constexpr (r > 0) __builtin_amdgcn_sched_group_barrier(0x100, r, 0);       // LDS reads
    if constexpr (l > 0) __builtin_amdgcn_sched_group_barrier(0x010, l, 0);       // loads to LDS
    if constexpr (x + 1 < X) interleave<R, X, L, x + 1>();
    else __builtin_amdgcn_sched_barrier(0);
}

// BN x BM = output features x rows of the workgroup tile; WN x WM waves, each computing a (BN / WN) x (BM / WM) block as
// TI x TJ MFMA tiles of 32 x 32; SK = k per stage, ST = stages in LDS.
template <int EPI, int BN, int BM, int WN, int WM, int SK, int ST>
__global__ __launch_bounds__(64 * WN * WM) __attribute__((amdgpu_waves_per_eu(1, 2)))
void k_gemm(const BF16* __restrict__ A, const BF16* __restrict__ W, int M, int N, int K, int slices, float* __restrict__ outf,
            BF16* __restrict__ outb, LmEpi lm, RopeEpi rp) {
    constexpr int NW = WN * WM;
    constexpr int SN = BN / WN, SM = BM / WM, TI = SN / 32, TJ = SM / 32, NS = SK / 16;
    constexpr int RB = SK * 2, CPR = SK / 8, RPI = 64 / CPR;      // bytes and 16-byte chunks of a tile row of one stage; rows per load instruction
    constexpr int NI = (BN + BM) / RPI, LPW = NI / NW;            // load instructions per stage, and per wave
    constexpr int STAGE = (BN + BM) * RB;
    static_assert(SN % 32 == 0 && SM % 32 == 0 && NI % NW == 0 && BN % RPI == 0 && (NS == 2 || NS == 4), "tile shape");
    static_assert(LPW * (ST - 1) < 63, "the outstanding loads of a wave fit its counter");
    extern __shared__ __attribute__((aligned(128))) unsigned char lds[];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wn = wave / WM, wm = wave % WM;

    // Work items = (k-slice, tile) pairs, the slice slowest.  The dispatcher deals workgroup ids to the 8 XCDs in turn; each XCD
    // takes one contiguous range of the items, its workgroups side by side.  The tiles of a slice are ordered in bands of GW
    // column tiles, n fastest inside a band, so that the 32 tiles running on an XCD at one time are about GW wide and 32 / GW
    // high and read GW weight and 32 / GW activation panels into its L2.  (With m fastest, 16384 x 2048 x 11008 ran 1 x 32 tiles at
    // a time on every XCD: 2.75 times the panels, and the fabric behind the L2 was what the launch waited for.)
    const int n_mt = (M + BM - 1) / BM, n_nt = (N + BN - 1) / BN, total = n_mt * n_nt, all = total * slices;
    const int xcd = blockIdx.x % 8, step = (gridDim.x - xcd + 7) / 8;
    const int x0 = xcd * (all / 8) + min(xcd, all % 8), x1 = x0 + all / 8 + (xcd < all % 8 ? 1 : 0);
    const int nk_all = K / TG_BK, per = (nk_all + slices - 1) / slices;
    constexpr int GW = 4;
    auto tile_of = [&](int it, int& n0, int& m0) {
        const int v = it % total, band = v / (GW * n_mt), r = v - band * (GW * n_mt), gw = min(GW, n_nt - band * GW);
        n0 = (band * GW + r % gw) * BN;
        m0 = (r / gw) * BM;
    };
    auto item_stages = [&](int it) {                              // stages of an item (0: a slice past the end of k)
        const int kb = (it / total) * per;
        return max(0, min(nk_all, kb + per) - kb) * (TG_BK / SK);
    };

    // ---- loads: a wave instruction brings 64 chunks of 16 bytes, RPI tile rows, to 1 KB of LDS in lane order; chunk c of row
    // r is parked at place c ^ swz(r) of its row, which spreads the rows a fragment read touches over all banks.  Rows past the
    // matrix are read from its last row; what they produce is never stored.
    auto swz = [](int r) __attribute__((always_inline)) { return SK == 64 ? (r >> 1) & 7 : (r >> 2) & 3; };
    const char* lbase[LPW];
    uint32_t loff[LPW];
    int l_it = x0 + blockIdx.x / 8, l_left = 0, issued = 0;       // item being loaded, its stages still to load, stages issued in all
    uint32_t l_k = 0;
    auto load_item = [&]() __attribute__((always_inline)) {       // addresses of the next item with stages
        while (l_it < x1 && (l_left = item_stages(l_it)) == 0) l_it += step;
        if (l_it >= x1) return;
        int n0, m0, lane_ = lane;
        asm volatile("" : "+v"(lane_));                           // (what follows from it is computed here, not kept in registers)
        tile_of(l_it, n0, m0);
        l_k = (uint32_t)(l_it / total) * per * (TG_BK * 2);
#pragma unroll
        for (int p = 0; p < LPW; ++p) {
            const int i = wave * LPW + p;
            const bool is_w = i < BN / RPI;
            const int row0 = is_w ? i * RPI : (i - BN / RPI) * RPI, r = row0 + lane_ / CPR;
            const int last = is_w ? N - 1 - n0 : M - 1 - m0;
            lbase[p] = reinterpret_cast<const char*>(is_w ? W + (size_t)n0 * K : A + (size_t)m0 * K);
            loff[p] = (uint32_t)min(r, last) * (uint32_t)(K * 2) + ((lane_ % CPR) ^ swz(r)) * 16;
        }
    };
    // requests the next stage of the stream (past the last item: the last stage again, which nobody reads, so that the count of
    // loads in flight is the same at every wait)
    auto issue = [&]() __attribute__((always_inline)) {
        unsigned char* dst = lds + (issued % ST) * STAGE + wave * (LPW * 1024);
#pragma unroll
        for (int p = 0; p < LPW; ++p)
            __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(lbase[p] + l_k + loff[p]),
                                             (__attribute__((address_space(3))) void*)(dst + p * 1024), 16, 0, 0);
    };
    auto advance = [&]() __attribute__((always_inline)) {
        ++issued;
        if (--l_left > 0) l_k += RB;
        else if (l_it < x1) {
            l_it += step;
            load_item();
        }
    };
    load_item();
    if (l_it >= x1) return;                                       // no work at all
#pragma unroll 1
    for (int s = 0; s < ST; ++s) {
        issue();
        advance();
    }

    // ---- fragments: lane l reads the 8 k of half l / 32 of row l % 32 of its 32-row tile; double-buffered, one k-block of 16 ahead
    const int frow = lane & 31, fx = swz(frow);
    const unsigned char* fw_base = lds + (wn * SN + frow) * RB;
    const unsigned char* fa_base = lds + (BN + wm * SM + frow) * RB;
    bf16x8 fw[2][TI], fa[2][TJ];
    auto read_frags = [&](int set, int buf, int ks) __attribute__((always_inline)) {
        const int off = buf * STAGE + ((2 * ks + (lane >> 5)) ^ fx) * 16;
#pragma unroll
        for (int i = 0; i < TI; ++i) fw[set][i] = *reinterpret_cast<const bf16x8*>(fw_base + off + i * 32 * RB);
#pragma unroll
        for (int j = 0; j < TJ; ++j) fa[set][j] = *reinterpret_cast<const bf16x8*>(fa_base + off + j * 32 * RB);
    };
    f32x16 acc[TI][TJ];
    auto multiply = [&](int set) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < TI; ++i)
#pragma unroll
            for (int j = 0; j < TJ; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fw[set][i], fa[set][j], acc[i][j], 0, 0, 0);
    };
    int stage = 0, landed = 0;          // stage being multiplied; every stage below `landed` is known to be in LDS
    asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"(LPW * (ST - 1)) : "memory");
    read_frags(0, 0, 0);

    unsigned char* const stg = lds + ST * STAGE + wave * 4096;    // the wave's 4 KB for turning its block around in the epilogue
    for (int it = x0 + blockIdx.x / 8; it < x1; it += step) {
        int n0, m0;
        tile_of(it, n0, m0);
        const int nwave = n0 + SN * wn, mwave = m0 + SM * wm;     // first feature and row of the wave's block
#pragma unroll
        for (int i = 0; i < TI; ++i)
#pragma unroll
            for (int j = 0; j < TJ; ++j)
#pragma unroll
                for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;
        // LM head: what the rows' bias lists hold for the wave's strip (cursors, list start, base) goes straight to the wave's LDS,
        // 4 bytes a lane, and is first looked at in the epilogue
        constexpr int LM_R = (TJ + 1) / 2, LM_AT = 1536;          // rounds of 64 rows; byte offset (5 fields x LM_R x 256 bytes)
        static_assert(EPI != TEPI_LMHEAD || LM_AT + 5 * LM_R * 256 <= 4096, "bias cursors fit the wave's LDS");
        if constexpr (EPI == TEPI_LMHEAD) {
            if (lm.bias.rowptr) {
#pragma unroll
                for (int r = 0; r < LM_R; ++r) {
                    const int m = min(mwave + 64 * r + lane, M - 1), strip = min(nwave / TASC_LM_STRIP, lm.n_strips - 1);
                    const int32_t* cur = lm.bias_ptr + (size_t)m * (lm.n_strips + 1) + strip;
                    const int32_t* first = reinterpret_cast<const int32_t*>(lm.row_first + m);
                    const int32_t* src[5] = {cur, cur + 1, first, first + 1, reinterpret_cast<const int32_t*>(lm.row_base + m)};
#pragma unroll
                    for (int f = 0; f < 5; ++f)
                        __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)src[f],
                                                         (__attribute__((address_space(3))) void*)(stg + LM_AT + (f * LM_R + r) * 256), 4, 0, 0);
                }
            }
        }
        // One stage: the products of k-block ks run while the fragments of ks + 1 are read.  In front of the last k-block
        // every wave has read its last fragment of the stage and seen its own loads of the next stage land: after the barrier
        // the stage's buffer is refilled (ST stages ahead) and the next stage's first fragments are read under the last products.
#pragma unroll 1
        for (int kt = item_stages(it); kt > 0; --kt) {
            const int buf = stage % ST;
#pragma unroll
            for (int ks = 0; ks + 1 < NS; ++ks) {
                read_frags((ks + 1) & 1, buf, ks + 1);
                multiply(ks & 1);
                interleave<TI + TJ, TI * TJ, 0>();
            }
            // (loads return in order; the ones of the ST - 2 stages after the next may still be on their way)
            if (stage + 1 >= landed) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(LPW * (ST - 2)) : "memory");
            asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
            ++stage;
            read_frags(0, stage % ST, 0);
            issue();
            multiply((NS - 1) & 1);
            interleave<TI + TJ, TI * TJ, LPW>();
            advance();
        }
        // The loads in flight belong to the next item; after this wait none is older than the epilogue's stores, which so
        // never stand between a wait and the stage it is for until that stage is ST - 1 stages away.
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        landed = issued;

        // ---- epilogue: acc[i][j][e] = out[m][n], n = nwave + 32 i + tile_row(e, lane), m = mwave + 32 j + lane % 32.
        // A lane holds 4-feature pieces of 32 different rows, so a direct store would write 16 or 32 bytes of 32 rows per
        // instruction; the wave turns each piece around in its own 4 KB of LDS (chunks of 16 bytes, swizzled by row) and
        // stores whole 128-byte row segments.
        int el = lane;
        asm volatile("" : "+v"(el));
        const int lr = el & 31, lh = el >> 5, sr = el >> 3, sc = el & 7;
        if constexpr (EPI == TEPI_SWIGLU) {
            // rows 0..15 of a 32-feature tile are gate features, rows 16..31 the up rows of the same features
            constexpr int OB = SN, CH = OB / 16;                  // bytes and chunks of a row's SN / 2 bf16 outputs
            static_assert(CH == 4 || CH == 8, "output row of the wave");
            const int Nh = N / 2, f0 = nwave / 2;
#pragma unroll
            for (int j = 0; j < TJ; ++j) {
                if (j > 0) __builtin_amdgcn_wave_barrier();
#pragma unroll
                for (int i = 0; i < TI; ++i)
#pragma unroll
                    for (int q = 0; q < 2; ++q) {
                        float o[4];
#pragma unroll
                        for (int u = 0; u < 4; ++u) {
                            const float g = acc[i][j][4 * q + u], up = acc[i][j][8 + 4 * q + u];
                            o[u] = g / (1.0f + __expf(-g)) * up;
                        }
                        *reinterpret_cast<u32x2*>(stg + lr * OB + (((2 * i + q) ^ (lr & (CH - 1))) * 16) + 8 * lh) = pack_bf16x4(o[0], o[1], o[2], o[3]);
                    }
                __builtin_amdgcn_wave_barrier();
                u32x4 o[CH / 2];
#pragma unroll
                for (int p = 0; p < CH / 2; ++p) {
                    const int r = p * (64 / CH) + el / CH, ch = el % CH;
                    o[p] = *reinterpret_cast<const u32x4*>(stg + r * OB + ((ch ^ (r & (CH - 1))) * 16));
                }
#pragma unroll
                for (int p = 0; p < CH / 2; ++p) {
                    const int m = mwave + 32 * j + p * (64 / CH) + el / CH, f = f0 + (el % CH) * 8;
                    if (m < M && f < Nh) *reinterpret_cast<u32x4*>(outb + (size_t)m * Nh + f) = o[p];
                }
            }
        } else if constexpr (EPI == TEPI_LMHEAD) {
            static_assert(SN == TASC_LM_STRIP || 2 * SN == TASC_LM_STRIP, "a strip is the features of one wave or of two");
            float w_best[TJ];
            int32_t w_idx[TJ];
            const int strip = nwave / TASC_LM_STRIP;
            float lm_base[TJ];
            int64_t lm_first[TJ];
            int32_t lm_p0[TJ], lm_p1[TJ];                         // the strip's part of the row's list, relative to lm_first
#pragma unroll
            for (int j = 0; j < TJ; ++j) {
                const int32_t* f = reinterpret_cast<const int32_t*>(stg + LM_AT) + 32 * j + lr;
                lm_base[j] = 0.f;
                lm_first[j] = 0;
                lm_p0[j] = lm_p1[j] = 0;
                if (lm.bias.rowptr) {
                    lm_p0[j] = f[0];
                    lm_p1[j] = nwave < N && mwave + 32 * j + lr < M ? f[64 * LM_R] : lm_p0[j];
                    lm_first[j] = (int64_t)(uint32_t)f[128 * LM_R] | ((int64_t)f[192 * LM_R] << 32);
                    lm_base[j] = __int_as_float(f[256 * LM_R]);
                }
            }
            // the lane number once more, so that what follows from it is computed where it is used and not kept in registers
            auto lane_again = [&]() __attribute__((always_inline)) {
                int l_ = el;
                asm volatile("" : "+v"(l_));
                return l_;
            };
            // The seen successors of a row get their own bias instead of `base`: the wave scatters the differences into a patch in
            // its LDS and every lane adds the elements of its registers.  With a corpus of 32 to 160 M tokens the rows of frequent
            // tokens hold most of a strip's features (119 of 128 and more in a fifth of the (row, strip) pairs at 160 M), the others
            // few or none, so rows are taken in groups of eight and a group goes one of two ways.  Latency bounds both: a
            // list's lines come from memory, once per step.  LM head without logits (us; four entries a row fetched ahead and longer
            // lists read again for each tile of 32 features | this): 1280 x 151936 x 2048 at 160 M tokens 1340 | 880, 576 x 151936 x
            // 1536 at 80 M 540 | 425, 224 x 151936 x 896 at 32 M 181 | 141; where hardly any list is long, at 0.5 M, 780 | 750,
            // 310 | 310, 114 | 108.  All lists the first way, in rounds of 32 entries: 960, 452, 147; the second way from five
            // entries on instead of 17: 46 instead of 31 for 40 x 49152 x 896 at 0.5 M.
#pragma unroll
            for (int j = 0; j < TJ; ++j) {
                constexpr int GR = 8;
                float* const patch = reinterpret_cast<float*>(stg);
                const int len = lm_p1[j] - lm_p0[j];
                const int64_t start = lm_first[j] + lm_p0[j];
                constexpr int FEW = 16;
                const uint32_t long_rows = (uint32_t)__ballot(len > FEW);
                // At most FEW in every row of the group: fetched by the row's lanes, four by each in a round, and patched in
                // [32 rows][32 features]; tiles without any are left alone.
                const int few = ((long_rows >> (lr & ~(GR - 1))) & 0xFF) != 0 ? 0 : len;
#pragma unroll 1
                for (int p = 0; __ballot(p < few) != 0; p += 8) {
                    const int l_ = lane_again(), r_ = l_ & 31, h_ = l_ >> 5;
                    const int64_t at = start + (p + 4 * h_ < few ? p + 4 * h_ : 0);      // (4 entries from any one on, or from the end of an empty list, are there: padded)
                    const u32x4_u e_c = *reinterpret_cast<const u32x4_u*>(lm.bias.col + at);
                    const f32x4_u e_v = *reinterpret_cast<const f32x4_u*>(lm.bias.val + at);
                    uint32_t e_n[4];
#pragma unroll
                    for (int q = 0; q < 4; ++q) e_n[q] = p + 4 * h_ + q < few ? e_c[q] - (uint32_t)nwave : ~0u;
#pragma unroll
                    for (int i = 0; i < TI; ++i) {
                        if (__ballot((e_n[0] >> 5) == i || (e_n[1] >> 5) == i || (e_n[2] >> 5) == i || (e_n[3] >> 5) == i) == 0) continue;
                        __builtin_amdgcn_wave_barrier();
#pragma unroll
                        for (int q = 0; q < 4; ++q) *reinterpret_cast<float4*>(stg + q * 1024 + l_ * 16) = make_float4(0.f, 0.f, 0.f, 0.f);
                        __builtin_amdgcn_wave_barrier();
#pragma unroll
                        for (int q = 0; q < 4; ++q)
                            if ((e_n[q] >> 5) == i) patch[r_ * 32 + (((e_n[q] & 31) + 4 * (r_ & 7)) & 31)] = e_v[q] - lm_base[j];
                        __builtin_amdgcn_wave_barrier();
#pragma unroll
                        for (int q = 0; q < 4; ++q) {
                            const float4 t = *reinterpret_cast<const float4*>(patch + r_ * 32 + ((8 * q + 4 * h_ + 4 * (r_ & 7)) & 31));
                            acc[i][j][4 * q] += t.x; acc[i][j][4 * q + 1] += t.y; acc[i][j][4 * q + 2] += t.z; acc[i][j][4 * q + 3] += t.w;
                        }
                        __builtin_amdgcn_wave_barrier();
                    }
                }
                // More: the whole wave on one row after the other, two entries a lane, patched in [8 rows][SN features]; the next
                // group's entries are requested before this group's patch is added.
                uint32_t todo = 0;
#pragma unroll
                for (int g = 0; g < 32 / GR; ++g) todo |= ((long_rows >> (GR * g)) & 0xFF) != 0 ? 1u << g : 0;
                if (todo != 0) {
                    static_assert(TASC_LM_STRIP <= 128, "a row's part of a strip in one load per lane");
                    static_assert(GR * SN * 4 <= 4096, "the patch fits the wave's LDS");
                    const int l_ = lane_again();
                    u32x2_u c[GR];
                    f32x2_u v[GR];
                    auto fetch = [&](int g) __attribute__((always_inline)) {
#pragma unroll
                        for (int r = 0; r < GR; ++r) {            // (2 entries from any one on, or from the end of an empty list, are there: padded)
                            const int64_t at = (int64_t)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)start, g * GR + r) |
                                               ((int64_t)__builtin_amdgcn_readlane((int)(start >> 32), g * GR + r) << 32);
                            const uint32_t off = 2 * l_ < __builtin_amdgcn_readlane(len, g * GR + r) ? 8 * l_ : 0;
                            c[r] = *reinterpret_cast<const u32x2_u*>(reinterpret_cast<const char*>(lm.bias.col + at) + off);
                            v[r] = *reinterpret_cast<const f32x2_u*>(reinterpret_cast<const char*>(lm.bias.val + at) + off);
                        }
                    };
                    fetch(__builtin_ctz(todo));
#pragma unroll 1
                    while (todo != 0) {
                        const int g = __builtin_ctz(todo);
                        todo &= todo - 1;
                        __builtin_amdgcn_wave_barrier();
#pragma unroll
                        for (int q = 0; q < GR * SN * 4 / 1024; ++q) *reinterpret_cast<float4*>(stg + q * 1024 + l_ * 16) = make_float4(0.f, 0.f, 0.f, 0.f);
                        __builtin_amdgcn_wave_barrier();
#pragma unroll
                        for (int r = 0; r < GR; ++r) {
                            const int n = __builtin_amdgcn_readlane(len, g * GR + r);
                            const float base = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(lm_base[j]), g * GR + r));
#pragma unroll
                            for (int u = 0; u < 2; ++u) {
                                const uint32_t f = c[r][u] - (uint32_t)nwave;
                                if (2 * l_ + u < n && f < (uint32_t)SN) patch[r * SN + (f ^ ((r & 3) << 3))] = v[r][u] - base;
                            }
                        }
                        __builtin_amdgcn_wave_barrier();
                        if (todo != 0) fetch(__builtin_ctz(todo));
                        if ((l_ & 31) / GR == g) {
                            const int a_ = lane_again(), r_ = a_ & (GR - 1);
                            const float* row = patch + r_ * SN;
#pragma unroll
                            for (int q = 0; q < 4; ++q) {
                                const float* at = row + ((8 * q + 4 * (a_ >> 5)) ^ ((r_ & 3) << 3));
#pragma unroll
                                for (int i = 0; i < TI; ++i) {
                                    const float4 t = *reinterpret_cast<const float4*>(at + 32 * i);
                                    acc[i][j][4 * q] += t.x; acc[i][j][4 * q + 1] += t.y; acc[i][j][4 * q + 2] += t.z; acc[i][j][4 * q + 3] += t.w;
                                }
                                __builtin_amdgcn_sched_barrier(0);            // (few registers of the patch at a time)
                            }
                        }
                        __builtin_amdgcn_wave_barrier();
                    }
                }
                float best = -INFINITY;
                int32_t best_i = 0x7FFFFFFF;
#pragma unroll
                for (int i = 0; i < TI; ++i)
#pragma unroll
                    for (int e = 0; e < 16; ++e) {
                        const int n = nwave + 32 * i + tile_row(e, el);       // ascending: the first of equal values stays
                        acc[i][j][e] += lm_base[j];
                        if (n < N && acc[i][j][e] > best) { best = acc[i][j][e]; best_i = n; }
                    }
                // the two lane halves hold different features of the same row
                const float ov = __shfl_xor(best, 32);
                const int32_t oi = __shfl_xor(best_i, 32);
                if (ov > best || (ov == best && oi < best_i)) { best = ov; best_i = oi; }
                w_best[j] = best;
                w_idx[j] = best_i;
                if (lm.logits) {
#pragma unroll
                    for (int i = 0; i < TI; ++i) {
                        __builtin_amdgcn_wave_barrier();
#pragma unroll
                        for (int q = 0; q < 4; ++q)
                            *reinterpret_cast<float4*>(stg + lr * 128 + (((2 * q + lh) ^ (lr & 7)) * 16)) =
                                make_float4(acc[i][j][4 * q], acc[i][j][4 * q + 1], acc[i][j][4 * q + 2], acc[i][j][4 * q + 3]);
                        __builtin_amdgcn_wave_barrier();
                        f32x4 o[4];
#pragma unroll
                        for (int p = 0; p < 4; ++p) {
                            const int r = 8 * p + sr;
                            o[p] = *reinterpret_cast<const f32x4*>(stg + r * 128 + ((sc ^ (r & 7)) * 16));
                        }
#pragma unroll
                        for (int p = 0; p < 4; ++p) {
                            const int mm = mwave + 32 * j + 8 * p + sr, n = nwave + 32 * i + 4 * sc;
                            if (mm < M) {
                                float* dst = lm.logits + (size_t)mm * N + n;
                                if (n + 4 <= N) *reinterpret_cast<f32x4_u*>(dst) = o[p];
                                else
                                    for (int u = 0; u < 4; ++u)
                                        if (n + u < N) dst[u] = o[p][u];
                            }
                        }
                    }
                    __builtin_amdgcn_wave_barrier();
                }
            }
            if constexpr (SN < TASC_LM_STRIP) {
                // the odd wave column hands its half of the strip to the even one (its 4 KB are not written again before the
                // next tile's epilogue, many barriers on)
                if ((wn & 1) && el < 32) {
#pragma unroll
                    for (int j = 0; j < TJ; ++j) {
                        reinterpret_cast<float*>(stg)[32 * j + lr] = w_best[j];
                        reinterpret_cast<int32_t*>(stg)[128 + 32 * j + lr] = w_idx[j];
                    }
                }
                asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
                if (!(wn & 1)) {
                    const unsigned char* other = stg + WM * 4096;
#pragma unroll
                    for (int j = 0; j < TJ; ++j) {
                        const float ov = reinterpret_cast<const float*>(other)[32 * j + lr];
                        if (ov > w_best[j]) { w_best[j] = ov; w_idx[j] = reinterpret_cast<const int32_t*>(other)[128 + 32 * j + lr]; }
                    }
                }
            }
            if (el < 32 && strip < lm.n_strips && (SN == TASC_LM_STRIP || !(wn & 1))) {
#pragma unroll
                for (int j = 0; j < TJ; ++j) {
                    const int m = mwave + 32 * j + lr;
                    if (m < M) {
                        lm.part_val[(size_t)m * lm.n_strips + strip] = w_best[j];
                        lm.part_idx[(size_t)m * lm.n_strips + strip] = w_idx[j];
                    }
                }
            }
        } else if constexpr (EPI == TEPI_ROPE) {
            // head_dim divides the wave's span, so the rotation partner of a register is a register of the same lane
            // (half a head = 16, 32 or 64 features further on).  Same arithmetic as k_rope_kv.
            const KvGeom& gm = rp.gm;
#pragma unroll
            for (int j = 0; j < TJ; ++j) {
                const int m = mwave + 32 * j + lr, mc = min(m, M - 1);
                const int b = gm.seq(mc), ir = gm.index(mc, b), pos = rp.pos0[b] + ir;
                const bool active = m < M && ir < rp.n_rows[b];
                const int tpos = pos < rp.max_pos ? pos : rp.max_pos - 1, slot = pos % TASC_KV_BLOCK;
                BF16* const page = rp.kv_layer + (active ? (size_t)rp.block_tab[(size_t)b * gm.max_blocks + pos / TASC_KV_BLOCK] * gm.page_elems : 0);
#pragma unroll
                for (int i = 0; i < TI; ++i) {
                    const int n = nwave + 32 * i, head = n / gm.hd, e0 = n % gm.hd;      // wave-uniform
                    const int half = gm.hd / 2;
                    if (n >= N) continue;
                    if (head >= gm.H + gm.Hkv || e0 >= half) continue;                   // values; or done with its partner
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        if (half == 16 && q >= 2) continue;                              // head_dim 32: the partner is 8 registers on
                        const int e = e0 + 8 * q + 4 * lh;
                        const float4 cs = *reinterpret_cast<const float4*>(rp.cosT + (size_t)tpos * half + e);
                        const float4 sn = *reinterpret_cast<const float4*>(rp.sinT + (size_t)tpos * half + e);
                        const float c_[4] = {cs.x, cs.y, cs.z, cs.w}, s_[4] = {sn.x, sn.y, sn.z, sn.w};
                        auto turn = [&](f32x16& x, int xe, f32x16& y, int ye, int u) __attribute__((always_inline)) {
                            const float a_ = x[xe], b_ = y[ye];
                            x[xe] = a_ * c_[u] - b_ * s_[u];
                            y[ye] = b_ * c_[u] + a_ * s_[u];
                        };
#pragma unroll
                        for (int u = 0; u < 4; ++u) {
                            const int x = 4 * q + u;
                            if (half == 64) { if (i + 2 < TI) turn(acc[i][j], x, acc[i + 2 < TI ? i + 2 : i][j], x, u); }
                            else if (half == 32) { if (i + 1 < TI) turn(acc[i][j], x, acc[i + 1 < TI ? i + 1 : i][j], x, u); }
                            else if (q < 2) turn(acc[i][j], x, acc[i][j], (x + 8) & 15, u);
                        }
                    }
                }
#pragma unroll
                for (int i = 0; i < TI; ++i) {
                    const int n = nwave + 32 * i, head = n / gm.hd, e0 = n % gm.hd;
                    if (n >= N) continue;
                    if (head < gm.H + gm.Hkv) {
                        // bf16 [32 rows][32 features] = 64 bytes a row through LDS, 16 bytes of a row per lane
                        __builtin_amdgcn_wave_barrier();
#pragma unroll
                        for (int q = 0; q < 4; ++q)
                            *reinterpret_cast<u32x2*>(stg + lr * 64 + ((q ^ (lr & 3)) * 16) + 8 * lh) =
                                pack_bf16x4(acc[i][j][4 * q], acc[i][j][4 * q + 1], acc[i][j][4 * q + 2], acc[i][j][4 * q + 3]);
                        // where the row goes: q rows by row index, k rows by page and slot
                        BF16* dst = nullptr;
                        if (head < gm.H) { if (m < M) dst = outb + (size_t)m * gm.H * gm.hd + n; }
                        else if (active) dst = page + (size_t)((head - gm.H) * TASC_KV_BLOCK + slot) * gm.hd + e0;
                        __builtin_amdgcn_wave_barrier();
#pragma unroll
                        for (int p = 0; p < 2; ++p) {
                            const int r = 16 * p + (el >> 2), ch = el & 3;
                            const u32x4 o = *reinterpret_cast<const u32x4*>(stg + r * 64 + ((ch ^ (r & 3)) * 16));
                            const uint64_t d64 = (uint64_t)dst;
                            const uint64_t dr = (uint64_t)(uint32_t)__shfl((int)(uint32_t)d64, r) | ((uint64_t)(uint32_t)__shfl((int)(uint32_t)(d64 >> 32), r) << 32);
                            if (dr) *reinterpret_cast<u32x4*>(reinterpret_cast<BF16*>(dr) + 8 * ch) = o;
                        }
                    } else if (active) {
                        // values transposed: consecutive lanes are consecutive rows, so a sequence's rows fill consecutive slots
                        uint16_t* vt = reinterpret_cast<uint16_t*>(page) + (size_t)gm.Hkv * TASC_KV_BLOCK * gm.hd +
                                       (size_t)((head - gm.H - gm.Hkv) * gm.hd + e0 + 4 * lh) * TASC_KV_BLOCK + slot;
#pragma unroll
                        for (int q = 0; q < 4; ++q)
#pragma unroll
                            for (int u = 0; u < 4; ++u) vt[(8 * q + u) * TASC_KV_BLOCK] = f2bf(acc[i][j][4 * q + u]);
                    }
                }
            }
        } else {
            float* const o_base = EPI == TEPI_PARTIAL ? outf + (size_t)(it / total) * M * N : outf;
#pragma unroll
            for (int j = 0; j < TJ; ++j)
#pragma unroll
                for (int i = 0; i < TI; ++i) {
                    const int n = nwave + 32 * i + 4 * sc;
                    f32x4 old[4];
                    if (EPI == TEPI_RESID) {                      // requested before the turn-around
#pragma unroll
                        for (int p = 0; p < 4; ++p) {
                            const int m = mwave + 32 * j + 8 * p + sr;
                            old[p] = *reinterpret_cast<const f32x4*>(o_base + (size_t)min(m, M - 1) * N + min(n, N - 4));
                        }
                    }
                    __builtin_amdgcn_wave_barrier();
#pragma unroll
                    for (int q = 0; q < 4; ++q)
                        *reinterpret_cast<float4*>(stg + lr * 128 + (((2 * q + lh) ^ (lr & 7)) * 16)) =
                            make_float4(acc[i][j][4 * q], acc[i][j][4 * q + 1], acc[i][j][4 * q + 2], acc[i][j][4 * q + 3]);
                    __builtin_amdgcn_wave_barrier();
                    f32x4 o[4];
#pragma unroll
                    for (int p = 0; p < 4; ++p) {
                        const int r = 8 * p + sr;
                        o[p] = *reinterpret_cast<const f32x4*>(stg + r * 128 + ((sc ^ (r & 7)) * 16));
                    }
#pragma unroll
                    for (int p = 0; p < 4; ++p) {
                        const int m = mwave + 32 * j + 8 * p + sr;
                        if (EPI == TEPI_RESID) o[p] += old[p];
                        if (m < M && n < N) *reinterpret_cast<f32x4*>(o_base + (size_t)m * N + n) = o[p];
                    }
                }
        }
        __builtin_amdgcn_wave_barrier();
        // (the LM head's epilogue has other use for the registers of the next stage's first fragments, and they are read again here:
        // 40 bytes of spills otherwise, 874 instead of 860 us for 1280 x 151936 x 2048)
        if constexpr (EPI == TEPI_LMHEAD) read_frags(0, stage % ST, 0);
    }
}
