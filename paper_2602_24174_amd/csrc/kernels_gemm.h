// The tiled bf16 GEMM of forwards of more than 16 rows: out[M, N] = epilogue(A[M, K] W[N, K]^T), both operands k-contiguous.
//
// A workgroup computes BN (output features) x BM (rows) tiles with v_mfma_f32_32x32x16_bf16, the WEIGHT rows as the A operand,
// so a lane ends up with runs of 4 consecutive features of one row.  k advances in stages of 64; ST stages sit in LDS at once,
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
// Loads are buffer loads: a lane's offset from its tile's first row is the same for every item, k is a scalar beside it, and past the
// last item the buffer has no bytes, so the stream's end costs no traffic and the loop no branch.  They are spread over the k-blocks of
// a stage (the first two of them with two stages in LDS): all at once, behind the barrier, every wave waited for the others' (128 x 128 x 64 of a stage 0.78 us, 0.55 so).
// What bounds a 128 x 128 tile is that rate of lines into a compute unit: without the products 23.3 of 24.8 us for 576 x 1536 x 8960 in four slices
// with cold weights, 18.5 with warm ones, 18.4 without the loads.  In the forwards, one tile per compute unit through registers | so, us: down
// 1280 x 2048 x 11008 in six slices 61.5 | 59.0, 6336 x 1536 x 8960 195 | 189, output 1280 x 2048 x 2048 26.9 | 21.5, q/k/v of prompts 6336 x 2048 x 1536
// 80 | 54.
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

// silu(g) u, with a division's quotient in half its instructions: every matrix core waits for them.  The denominator lies in 1..2^128
// or is infinite, so what a division does for other ones is left out; a quarter of both keeps the reciprocal of the largest a normal number.
// Of all 2^32 g the quotient has other bits than g / (1 + exp(-g)) for those below 2^-124 alone, whose quarter is not a normal number: half of them, by one ulp.
// Gate/up 256 x 256, 1280 x 22016 x 2048: 107.5 us with a division, 105.3 so; 6336 x 17920 x 1536: 317, 305; 480 x 17920 x 1536: 44.8, 42.8.
__device__ __forceinline__ float silu_times(float g, float u) {
    const float d = fmaf(__expf(-g), 0.25f, 0.25f), n = 0.25f * g, r = __builtin_amdgcn_rcpf(d), q = n * r;
    return __builtin_amdgcn_div_fixupf(fmaf(fmaf(-d, q, n), r, q), d, n) * u;
}

// The rotation of a feature and its partner half a head on.  Which product is rounded first is written out: launches of different row counts
// rotate in different kernels, and a row has to have the same bits from all of them.
__device__ __forceinline__ void rope_turn(float a, float b, float cs, float sn, float& ra, float& rb) {
    ra = __builtin_fmaf(a, cs, -(b * sn));
    rb = __builtin_fmaf(b, cs, a * sn);
}

typedef float f32x4_u __attribute__((ext_vector_type(4), aligned(4)));    // four floats at any 4-byte address
typedef float f32x2_u __attribute__((ext_vector_type(2), aligned(4)));
typedef uint32_t u32x2_u __attribute__((ext_vector_type(2), aligned(4)));
typedef uint32_t u32x4_u __attribute__((ext_vector_type(4), aligned(4)));

constexpr int gemm_lds_bytes(int BN, int BM, int WN, int WM, int ST) { return ST * (BN + BM) * TG_BK * 2 + WN * WM * 4096; }

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
// TI x TJ MFMA tiles of 32 x 32; ST = stages in LDS; HD = head_dim (rotation only).
template <int EPI, int BN, int BM, int WN, int WM, int ST, int HD = 0>
__global__ __launch_bounds__(64 * WN * WM) __attribute__((amdgpu_waves_per_eu(1, 2)))
void k_gemm(const BF16* __restrict__ A, const BF16* __restrict__ W, int M, int N, int K, int slices, float* __restrict__ outf,
            BF16* __restrict__ outb, LmEpi lm, RopeEpi rp) {
#ifdef __HIP_DEVICE_COMPILE__                                     // (buffer resources are unknown to the host's pass)
    constexpr int NW = WN * WM;
    constexpr int SK = TG_BK;                                     // k per stage: whole cache lines of the operands' rows
    constexpr int SN = BN / WN, SM = BM / WM, TI = SN / 32, TJ = SM / 32, NS = SK / 16;
    constexpr int RB = SK * 2, CPR = SK / 8, RPI = 64 / CPR;      // bytes and 16-byte chunks of a tile row of one stage; rows per load instruction
    constexpr int NI = (BN + BM) / RPI, LPW = NI / NW;            // load instructions per stage, and per wave
    constexpr int STAGE = (BN + BM) * RB;
    static_assert(SN % 32 == 0 && SM % 32 == 0 && NI % NW == 0 && BN % RPI == 0, "tile shape");
    static_assert(LPW * (ST - 1) < 63, "the outstanding loads of a wave fit its counter");
    constexpr int SPREAD = ST > 2 ? NS : 2;                       // (two stages leave a load little time: 105.3 us over two k-blocks in the first case above, 106.8 at once)
    constexpr auto part = [](int x) { return x >= SPREAD ? LPW : x * LPW / SPREAD; };      // loads of a stage requested before k-block x
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
        return max(0, min(nk_all, kb + per) - kb);
    };

    // ---- loads: a wave instruction brings 64 chunks of 16 bytes, RPI tile rows, to 1 KB of LDS in lane order; chunk c of row
    // r is parked at place c ^ swz(r) of its row, which spreads the rows a fragment read touches over all banks.  A tile's buffer ends with
    // the matrix' last row: rows past it arrive as zeros, and what they produce is never stored.  The k of a load is the scalar offset, which need not
    // count for whether a load is inside: of a row inside it stays below the row's length, and past the last item it is 0.
    auto swz = [](int r) __attribute__((always_inline)) { return (r >> 1) & 7; };
    uint32_t loff[LPW];                                           // from the tile's first row: the same for every item
#pragma unroll
    for (int p = 0; p < LPW; ++p) {
        const int i = wave * LPW + p, r = (i < BN / RPI ? i : i - BN / RPI) * RPI + lane / CPR;
        loff[p] = (uint32_t)r * (uint32_t)(K * 2) + ((lane % CPR) ^ swz(r)) * 16;
    }
    __amdgpu_buffer_rsrc_t rs_w, rs_a;
    int l_it = x0 + blockIdx.x / 8, l_left = 0, issued = 0;       // item being loaded, its stages still to load, stages requested in all
    uint32_t l_k = 0, l_at = wave * (LPW * 1024);                 // its next k (bytes), and where that stage goes
    auto load_item = [&]() __attribute__((always_inline)) {       // the next item with stages; past the last one, loads of nothing
        while (l_it < x1 && (l_left = item_stages(l_it)) == 0) l_it += step;
        int n0 = 0, m0 = 0;
        const bool any = l_it < x1;
        if (any) tile_of(l_it, n0, m0);
        else l_left = 1;                                          // (so this comes again after every stage)
        l_k = any ? (uint32_t)(l_it / total) * per * (TG_BK * 2) : 0;
        rs_w = __builtin_amdgcn_make_buffer_rsrc((void*)(W + (size_t)n0 * K), 0, any ? min(BN, N - n0) * K * 2 : 0, 0x00027000);
        rs_a = __builtin_amdgcn_make_buffer_rsrc((void*)(A + (size_t)m0 * K), 0, any ? min(BM, M - m0) * K * 2 : 0, 0x00027000);
    };
    // requests loads P0 .. P1 of the next stage of the stream
    auto issue = [&]<int P0, int P1>() __attribute__((always_inline)) {
#pragma unroll
        for (int p = P0; p < P1; ++p)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(wave * LPW + p < BN / RPI ? rs_w : rs_a, (__attribute__((address_space(3))) void*)(lds + l_at + p * 1024),
                                                     16, loff[p], l_k, 0, 0);
    };
    auto advance = [&]() __attribute__((always_inline)) {
        ++issued;
        l_at += STAGE;
        if (l_at >= ST * STAGE) l_at -= ST * STAGE;
        l_k += RB;
        if (--l_left == 0) {
            l_it += step;
            load_item();
        }
    };
    load_item();
    if (l_it >= x1) return;                                       // no work at all
#pragma unroll 1
    for (int s = 0; s + 1 < ST; ++s) {
        issue.template operator()<0, LPW>();
        advance();
    }
    issue.template operator()<0, part(1)>();

    // ---- fragments: lane l reads the 8 k of half l / 32 of row l % 32 of its 32-row tile; double-buffered, one k-block of 16 ahead
    const int frow = lane & 31, fx = swz(frow);
    const unsigned char* fw_base = lds + (wn * SN + frow) * RB;
    const unsigned char* fa_base = lds + (BN + wm * SM + frow) * RB;
    bf16x8 fw[2][TI], fa[2][TJ];
    auto read_frags = [&](int set, int at, int ks) __attribute__((always_inline)) {
        const int off = at + ((2 * ks + (lane >> 5)) ^ fx) * 16;
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
    int stage = 0, landed = 0, at = 0;  // stage being multiplied and its place; every stage below `landed` is known to be in LDS
    asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"(LPW * (ST - 2) + part(1)) : "memory");
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
        // Rotation: where the lane's rows go, a chain of three dependent loads that ends under the first products
        int32_t r_pos[TJ], r_slot[TJ], r_page[TJ];                // table position, slot in its page (-1: appends nothing), page
        if constexpr (EPI == TEPI_ROPE) {
#pragma unroll
            for (int j = 0; j < TJ; ++j) {
                const int m = min(mwave + 32 * j + (lane & 31), M - 1), b = rp.gm.seq(m);
                const int ir = rp.gm.index(m, b), pos = rp.pos0[b] + ir;
                r_pos[j] = min(pos, rp.max_pos - 1);
                r_slot[j] = ir < rp.n_rows[b] && mwave + 32 * j + (lane & 31) < M ? pos % TASC_KV_BLOCK : -1;
                r_page[j] = r_slot[j] >= 0 ? rp.block_tab[(size_t)b * rp.gm.max_blocks + pos / TASC_KV_BLOCK] : 0;
            }
        }
        // One stage: the products of k-block ks run while the fragments of ks + 1 are read.  In front of the last k-block
        // every wave has read its last fragment of the stage and seen its own loads of the next stage land: after the barrier
        // the stage's buffer is refilled (ST stages ahead) and the next stage's first fragments are read under the last products.
        // The refill's loads are spread over SPREAD k-blocks from there on.
#pragma unroll 1
        for (int kt = item_stages(it); kt > 0; --kt) {
            auto block = [&]<int ks>() __attribute__((always_inline)) {
                read_frags((ks + 1) & 1, at, ks + 1);
                issue.template operator()<part(ks + 1), part(ks + 2)>();
                multiply(ks & 1);
                interleave<TI + TJ, TI * TJ, part(ks + 2) - part(ks + 1)>();
            };
            static_assert(NS == 4, "three k-blocks, and the last one behind the barrier");
            block.template operator()<0>();
            block.template operator()<1>();
            block.template operator()<2>();
            advance();
            // (loads return in order; the ones of the ST - 2 stages after the next may still be on their way)
            if (stage + 1 >= landed) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(LPW * (ST - 2)) : "memory");
            asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
            ++stage;
            at += STAGE;
            if (at >= ST * STAGE) at -= ST * STAGE;
            read_frags(0, at, 0);
            issue.template operator()<0, part(1)>();
            multiply((NS - 1) & 1);
            interleave<TI + TJ, TI * TJ, part(1)>();
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
                            o[u] = silu_times(g, up);
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
            // (half a head = 16, 32 or 64 features further on).
            const KvGeom& gm = rp.gm;
            // the q and k heads of 32 rows, up to 32 of the lane's factors at a time
            auto turn_rows = [&]<int j>() __attribute__((always_inline)) {
                constexpr int HALF = HD / 2, NX = HALF < 32 ? HALF / 8 : 4, STEP = HD == 32 ? 0 : HALF / 32;       // the partner: STEP tiles on, or 8 registers
#pragma unroll
                for (int x0 = 0; x0 < HALF / 8; x0 += NX) {
                    f32x4 cs[NX], sn[NX];
#pragma unroll
                    for (int x = 0; x < NX; ++x) {
                        cs[x] = *reinterpret_cast<const f32x4*>(rp.cosT + (size_t)r_pos[j] * HALF + 8 * (x0 + x) + 4 * lh);
                        sn[x] = *reinterpret_cast<const f32x4*>(rp.sinT + (size_t)r_pos[j] * HALF + 8 * (x0 + x) + 4 * lh);
                    }
#pragma unroll
                    for (int i = 0; i < TI; ++i) {
                        if ((32 * i) % HD != 8 * x0 || i + STEP >= TI || (nwave + 32 * i) / HD >= gm.H + gm.Hkv) continue;
                        f32x16 &a_ = acc[i][j], &b_ = acc[i + STEP < TI ? i + STEP : i][j];
#pragma unroll
                        for (int e = 0; e < 4 * NX; ++e) {
                            float ra, rb;
                            rope_turn(a_[e], b_[HD == 32 ? e + 8 : e], cs[e / 4][e % 4], sn[e / 4][e % 4], ra, rb);
                            a_[e] = ra;
                            b_[HD == 32 ? e + 8 : e] = rb;
                        }
                    }
                    __builtin_amdgcn_sched_barrier(0);
                }
            };
            static_assert(TJ <= 2 && HD <= SN, "rows of a wave; whole heads");
            turn_rows.template operator()<0>();
            if constexpr (TJ > 1) turn_rows.template operator()<1>();
#pragma unroll
            for (int j = 0; j < TJ; ++j) {
                const int m = mwave + 32 * j + lr, slot = r_slot[j];
                const bool active = slot >= 0;
                BF16* const page = rp.kv_layer + (size_t)r_page[j] * gm.page_elems;
#pragma unroll
                for (int i = 0; i < TI; ++i) {
                    const int n = nwave + 32 * i, head = n / HD, e0 = n % HD;
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
                        if (head < gm.H) { if (m < M) dst = outb + (size_t)m * gm.H * HD + n; }
                        else if (active) dst = page + (size_t)((head - gm.H) * TASC_KV_BLOCK + slot) * HD + e0;
                        __builtin_amdgcn_wave_barrier();
#pragma unroll
                        for (int p = 0; p < 2; ++p) {
                            const int r = 16 * p + (el >> 2), ch = el & 3;
                            const u32x4 o = *reinterpret_cast<const u32x4*>(stg + r * 64 + ((ch ^ (r & 3)) * 16));
                            const uint64_t d64 = (uint64_t)dst;
                            const uint64_t dr = (uint64_t)(uint32_t)__shfl((int)(uint32_t)d64, r) | ((uint64_t)(uint32_t)__shfl((int)(uint32_t)(d64 >> 32), r) << 32);
                            if (dr) *reinterpret_cast<u32x4*>(reinterpret_cast<BF16*>(dr) + 8 * ch) = o;
                        }
                    }
                }
            }
            // Values go transposed: [feature][32 rows] of two tiles in the wave's LDS, a feature a lane, and from there runs of rows that are
            // neighbours in a page, 8 slots, 2 or 1 at a time.  The columns of few workgroups hold all the values of a layer, so what they cost
            // is added to the launch (q/k/v of prompts, 6336 x 2048 x 1536: two-byte stores straight from the registers 80 us, so 54).
            if ((nwave + SN - 1) / HD >= gm.H + gm.Hkv && nwave < N) {
                static_assert(TI % 2 == 0, "tiles in pairs");
#pragma unroll 1
                for (int pass = 0; pass < TJ * TI / 2; ++pass) {
                    const int v0 = nwave + 64 * (pass % (TI / 2)) - (gm.H + gm.Hkv) * HD;      // the pair's first value feature
                    if (v0 <= -64) continue;
                    __builtin_amdgcn_wave_barrier();
#pragma unroll
                    for (int t = 0; t < TJ * TI / 2; ++t) {
                        if (t != pass) continue;
#pragma unroll
                        for (int ii = 0; ii < 2; ++ii)
#pragma unroll
                            for (int e = 0; e < 16; ++e) {
                                const int f = 32 * ii + tile_row(e, el);
                                *reinterpret_cast<uint16_t*>(stg + f * 64 + (((lr >> 3) ^ ((f >> 2) & 3)) * 16) + (lr & 7) * 2) =
                                    f2bf(acc[2 * (t % (TI / 2)) + ii][t / (TI / 2)][e]);
                            }
                    }
                    __builtin_amdgcn_wave_barrier();
                    int slot_l = r_slot[0], page_l = r_page[0];
                    if constexpr (TJ > 1) {
                        slot_l = pass < TI / 2 ? slot_l : r_slot[1];
                        page_l = pass < TI / 2 ? page_l : r_page[1];
                    }
                    // bit r: row r + 1 follows row r in its page.  (All lanes shuffle, before any condition: a lane that sits out reads as 0, and
                    // page 0 is a page.)
                    const int slot_n = __shfl(slot_l, (el + 1) & 63), page_n = __shfl(page_l, (el + 1) & 63);
                    const uint32_t on = (uint32_t)__ballot(lr < 31 && slot_l >= 0 && slot_n == slot_l + 1 && page_n == page_l);
                    if (v0 + el >= 0 && nwave + 64 * (pass % (TI / 2)) + el < N) {
                        BF16* const base = rp.kv_layer + (size_t)gm.Hkv * TASC_KV_BLOCK * HD + (size_t)(v0 + el) * TASC_KV_BLOCK;
                        uint32_t v[17];                              // the feature's 32 rows
#pragma unroll
                        for (int c = 0; c < 4; ++c) {
                            const u32x4 w = *reinterpret_cast<const u32x4*>(stg + el * 64 + ((c ^ ((el >> 2) & 3)) * 16));
#pragma unroll
                            for (int u = 0; u < 4; ++u) v[4 * c + u] = w[u];
                        }
                        v[16] = 0;
                        auto two = [&](int r) { return (r & 1) ? __builtin_amdgcn_alignbit(v[min(r / 2 + 1, 16)], v[min(r / 2, 16)], 16) : v[min(r / 2, 16)]; };
                        int next = 0;
#pragma unroll
                        for (int r = 0; r < 32; ++r) {
                            const int slot = __builtin_amdgcn_readlane(slot_l, r);
                            if (r < next || slot < 0) continue;
                            uint16_t* const dst = reinterpret_cast<uint16_t*>(base + (size_t)__builtin_amdgcn_readlane(page_l, r) * gm.page_elems) + slot;
                            if ((slot & 7) == 0 && ((on >> r) & 0x7F) == 0x7F) {             // (row 31 has no bit: never past the last row)
                                *reinterpret_cast<u32x4*>(dst) = u32x4{two(r), two(r + 2), two(r + 4), two(r + 6)};
                                next = r + 8;
                            } else if ((slot & 1) == 0 && ((on >> r) & 1)) {
                                *reinterpret_cast<uint32_t*>(dst) = two(r);
                                next = r + 2;
                            } else {
                                *dst = (uint16_t)(v[r / 2] >> (16 * (r & 1)));
                            }
                        }
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
        if constexpr (EPI == TEPI_LMHEAD || EPI == TEPI_ROPE) read_frags(0, at, 0);
    }
#endif
}
