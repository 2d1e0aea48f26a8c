// Type-generic (fp32 or bf16 storage, fp32 arithmetic) kernels of the target forward.  They are the
// fp32 path and the reference the MFMA kernels are checked against.  Every output row is reduced in
// an order that does not depend on how many rows a launch holds, so a token scored as row i of a
// speculative step gets bit-identical results to the same token scored alone by plain greedy decoding.
#pragma once
#include "tasc_internal.h"

struct BF16 { uint16_t v; };

__device__ inline float bf2f(uint32_t bits16) { return __uint_as_float(bits16 << 16); }
// fp32 -> bf16, round to nearest even: the hardware conversion of gfx950 (v_cvt_pk_bf16_f32), one instruction per pair
typedef __attribute__((ext_vector_type(2))) float tasc_f32x2;
typedef __attribute__((ext_vector_type(2))) __bf16 tasc_bf16x2;
__device__ inline uint32_t f2bf_pair(float lo, float hi) {
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(tasc_f32x2{lo, hi}, tasc_bf16x2));
}
__device__ inline uint16_t f2bf(float f) { return (uint16_t)(f2bf_pair(f, 0.f) & 0xFFFFu); }
__device__ inline float to_f(float v) { return v; }
__device__ inline float to_f(BF16 v) { return bf2f(v.v); }
template <typename T> __device__ inline T from_f(float f);
template <> __device__ inline float from_f<float>(float f) { return f; }
template <> __device__ inline BF16 from_f<BF16>(float f) { return BF16{f2bf(f)}; }

__device__ inline void load8(const float* __restrict__ p, float* o) {
    float4 a = *reinterpret_cast<const float4*>(p), b = *reinterpret_cast<const float4*>(p + 4);
    o[0] = a.x; o[1] = a.y; o[2] = a.z; o[3] = a.w; o[4] = b.x; o[5] = b.y; o[6] = b.z; o[7] = b.w;
}
__device__ inline void load8(const BF16* __restrict__ p, float* o) {
    uint4 u = *reinterpret_cast<const uint4*>(p);
    o[0] = bf2f(u.x & 0xFFFFu); o[1] = bf2f(u.x >> 16); o[2] = bf2f(u.y & 0xFFFFu); o[3] = bf2f(u.y >> 16);
    o[4] = bf2f(u.z & 0xFFFFu); o[5] = bf2f(u.z >> 16); o[6] = bf2f(u.w & 0xFFFFu); o[7] = bf2f(u.w >> 16);
}

__device__ inline void load4(const float* __restrict__ p, float* o) {
    const float4 a = *reinterpret_cast<const float4*>(p);
    o[0] = a.x; o[1] = a.y; o[2] = a.z; o[3] = a.w;
}
__device__ inline void load4(const BF16* __restrict__ p, float* o) {
    const uint2 u = *reinterpret_cast<const uint2*>(p);
    o[0] = bf2f(u.x & 0xFFFFu); o[1] = bf2f(u.x >> 16); o[2] = bf2f(u.y & 0xFFFFu); o[3] = bf2f(u.y >> 16);
}

template <int VEC, typename T>
__device__ inline void load_n(const T* __restrict__ p, float* o) {
    if constexpr (VEC == 8) load8(p, o);
    else load4(p, o);
}

__device__ inline float wave_sum(float v) {
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
    return v;
}
__device__ inline float wave_max(float v) {
    for (int o = 32; o > 0; o >>= 1) v = fmaxf(v, __shfl_xor(v, o));
    return v;
}

// Sum over the 64 lanes with DPP row operations (a few cycles each; the ds_bpermute path of __shfl_xor costs an LDS
// round trip per step).  The lanes are added in a fixed order, the same for every call.
__device__ __forceinline__ float wave_sum_dpp(float v) {
    v += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0xB1, 0xF, 0xF, false));    // quad_perm [1,0,3,2]
    v += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0x4E, 0xF, 0xF, false));    // quad_perm [2,3,0,1]
    v += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0x141, 0xF, 0xF, false));   // row_half_mirror
    v += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0x140, 0xF, 0xF, false));   // row_mirror
    // every lane now holds the sum of its row of 16; rows 0..3 are lanes 0-15, 16-31, 32-47, 48-63
    const float r0 = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), 0));
    const float r1 = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), 16));
    const float r2 = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), 32));
    const float r3 = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), 48));
    return (r0 + r1) + (r2 + r3);
}

// ---------------------------------------------------------------- rows of a verify step
// Row idx = (sequence idx / (k + 1), i = idx % (k + 1)): the pending token (i = 0) or draft i - 1.
struct StepRows {
    const int32_t* tokens;    // [B, max_len]; null: not a verify step, the rows have been made already
    const int32_t* n_tok;
    const int32_t* cached;
    const int32_t* drafts;    // [B, k]
    int32_t max_len, k, vocab;
    int32_t *row_tok, *row_seq, *row0, *n_rows, *pos0, *sel_rows, *sel_tok;
};
__device__ __forceinline__ int step_token(const StepRows& a, int idx) {
    const int nq = a.k + 1, b = idx / nq, i = idx % nq;
    if (i == 0) return a.tokens[(size_t)b * a.max_len + a.n_tok[b] - 1];
    const int t = a.drafts[b * a.k + i - 1];
    return t < 0 ? 0 : (t >= a.vocab ? a.vocab - 1 : t);     // a draft outside the vocabulary can only be rejected
}
__device__ __forceinline__ void step_row(const StepRows& a, int idx, int t) {
    const int nq = a.k + 1, b = idx / nq;
    if (idx % nq == 0) {
        a.n_rows[b] = nq;
        a.row0[b] = idx;
        a.pos0[b] = a.cached[b];
    }
    a.row_tok[idx] = t;
    a.row_seq[idx] = b;
    a.sel_rows[idx] = idx;
    a.sel_tok[idx] = t;
}
__global__ void k_prepare_verify(StepRows a, int rows) {
    const int idx = blockIdx.x * blockDim.x + threadIdx.x;
    if (idx < rows) step_row(a, idx, step_token(a, idx));
}

// ---------------------------------------------------------------- embedding gather
template <typename T>
__global__ void k_embed(const T* __restrict__ E, const int32_t* row_tok, int d, float* __restrict__ x, StepRows step) {
    const int r = blockIdx.x, t = step.tokens ? step_token(step, r) : row_tok[r];
    if (step.tokens && threadIdx.x == 0) step_row(step, r, t);
    const T* e = E + (size_t)t * d;
    for (int k = threadIdx.x * 8; k < d; k += blockDim.x * 8) {
        float v[8];
        load8(e + k, v);
        float* o = x + (size_t)r * d + k;
        *reinterpret_cast<float4*>(o) = make_float4(v[0], v[1], v[2], v[3]);
        *reinterpret_cast<float4*>(o + 4) = make_float4(v[4], v[5], v[6], v[7]);
    }
}

// ---------------------------------------------------------------- RMSNorm: h = x * g / sqrt(mean(x^2) + eps)
// One wave per row.  `sel` (nullable) gathers rows: output row r reads input row sel[r] (negative -> row 0).
template <typename T>
__global__ __launch_bounds__(64) void k_rmsnorm(const float* __restrict__ x, const float* __restrict__ g,
                                                const int32_t* __restrict__ sel, int d, float eps, T* __restrict__ h) {
    const int r = blockIdx.x, lane = threadIdx.x;
    int src = sel ? sel[r] : r;
    if (src < 0) src = 0;
    const float* xr = x + (size_t)src * d;
    float ss = 0.f;
    for (int k = lane * 4; k < d; k += 256) {
        float4 v = *reinterpret_cast<const float4*>(xr + k);
        ss += v.x * v.x + v.y * v.y + v.z * v.z + v.w * v.w;
    }
    ss = wave_sum(ss);
    const float rinv = 1.0f / sqrtf(ss / (float)d + eps);
    for (int k = lane * 4; k < d; k += 256) {
        float4 v = *reinterpret_cast<const float4*>(xr + k);
        float4 gg = *reinterpret_cast<const float4*>(g + k);
        T* o = h + (size_t)r * d + k;
        o[0] = from_f<T>(v.x * rinv * gg.x);
        o[1] = from_f<T>(v.y * rinv * gg.y);
        o[2] = from_f<T>(v.z * rinv * gg.z);
        o[3] = from_f<T>(v.w * rinv * gg.w);
    }
}

// Rows of a forward: sequence b has the n_rows[b] rows row0[b] .. row0[b] + n_rows[b] - 1, row_seq[r] = the sequence of row r.
// Rows that belong to no sequence (the persistent kernels' prompt chunks) have i >= n_rows[b].
struct KvGeom {
    int32_t H, Hkv, hd, max_blocks;
    size_t page_elems;        // elements of one page: K [Hkv][16][hd] then V^T [Hkv][hd][16]
    const int32_t* row_seq;   // of the launch's first row on
    const int32_t* row0;      // [B], counted over the whole forward
    int32_t first;            // the launch's first row in that count
    __device__ int seq(int r) const { return row_seq[r]; }
    __device__ int index(int r, int b) const { return r + first - row0[b]; }
};

// ---------------------------------------------------------------- generic GEMM  out[M, N] = A[M, K] W[N, K]^T
// EPI_RESID: outf += A W^T.  EPI_SWIGLU: outT = silu(gate) up, a wave per feature (weight rows in blocks of 16 gate, 16 up).
// EPI_ROPE: the fused q/k/v projection, a wave per pair of features half a head apart: q and k rotated at the row's position, q to
// outT, new k and v rows to their cache pages.
enum { EPI_RESID = 1, EPI_SWIGLU = 2, EPI_ROPE = 3 };

struct GenericRope {          // EPI_ROPE only
    const float* cosT;        // [max_pos][hd / 2]
    const float* sinT;
    const int32_t* n_rows;
    const int32_t* pos0;
    const int32_t* block_tab;
    KvGeom gm;
    int32_t max_pos, nq;      // nq: rows of every sequence, all active, in a verify step; 0: look them up
};

// Up to this width the norms ride along with the products behind them: a small model's launches are what it waits for.  Beyond, every
// column's wave would sum the squares and scale the weights again for nothing (verify steps, fp32, two layers, us, norms in launches of their
// own | along: 5 rows, d 128 73 | 67, 256 78 | 72, 384 103 | 95, 2048 275 | 281; 224 rows 254 | 280, 330 | 364, 566 | 622, 3960 | 4930).
constexpr int kNormAlong = 256;

// The products of up to 8 rows (R of them, from row0 on) with one weight row, or two, by one wave: every lane sums its own k-slices (VEC
// wide) in ascending order, then the 64 partial sums are added in the order of wave_sum_dpp.  Lane r < 8 returns with row r's.  NORM: A is the
// residual stream and the product is with its RMSNorm (gain g): the sum of squares is taken along with the products, of weights
// already multiplied by the gain.
struct RowDots { float v, u; };
template <typename T, typename AT, bool PAIR, bool NORM, int VEC>
__device__ __forceinline__ RowDots row_dots(const AT* __restrict__ A, int row0, int R, const T* __restrict__ w0, const T* __restrict__ w1, int K,
                                            const float* __restrict__ g, float eps, int lane) {
    float acc[8] = {0, 0, 0, 0, 0, 0, 0, 0}, acu[8] = {0, 0, 0, 0, 0, 0, 0, 0}, ss[8] = {0, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll 2
    for (int k = lane * VEC; k < K; k += 64 * VEC) {
        float wv[VEC], uv[VEC], gv[VEC];
        load_n<VEC>(w0 + k, wv);
        if (PAIR) load_n<VEC>(w1 + k, uv);
        if (NORM) {
            load_n<VEC>(g + k, gv);
#pragma unroll
            for (int e = 0; e < VEC; ++e) {
                wv[e] *= gv[e];
                if (PAIR) uv[e] *= gv[e];
            }
        }
#pragma unroll
        for (int r = 0; r < 8; ++r) {
            if (r < R) {
                float av[VEC];
                load_n<VEC>(A + (size_t)(row0 + r) * K + k, av);
#pragma unroll
                for (int e = 0; e < VEC; ++e) {
                    acc[r] = fmaf(av[e], wv[e], acc[r]);
                    if (PAIR) acu[r] = fmaf(av[e], uv[e], acu[r]);
                    if (NORM) ss[r] = fmaf(av[e], av[e], ss[r]);
                }
            }
        }
    }
    float v = 0.f, u = 0.f, q = 0.f;
#pragma unroll
    for (int r = 0; r < 8; ++r) {
        if (r < R) {
            const float a = wave_sum_dpp(acc[r]), b = PAIR ? wave_sum_dpp(acu[r]) : 0.f, c = NORM ? wave_sum_dpp(ss[r]) : 0.f;
            v = lane == r ? a : v;
            u = lane == r ? b : u;
            q = lane == r ? c : q;
        }
    }
    if (NORM) {
        const float rinv = 1.0f / sqrtf(q / (float)K + eps);
        v *= rinv;
        u *= rinv;
    }
    return RowDots{v, u};
}
// a row's pair of features (e0 and half a head on) of a q, k or v head -> its rotation, its place
template <typename T>
__device__ __forceinline__ void rope_store(const GenericRope& rp, int head, int e0, int row, int pos, T* page, RowDots d, float cs, float sn,
                                           T* __restrict__ q_out) {
    const KvGeom& gm = rp.gm;
    const int half = gm.hd / 2, slot = pos % TASC_KV_BLOCK;
    if (head < gm.H + gm.Hkv) {
        const float ra = fmaf(d.v, cs, -(d.u * sn)), rc = fmaf(d.u, cs, d.v * sn);
        T* o = head < gm.H ? q_out + ((size_t)row * gm.H + head) * gm.hd + e0
                           : page ? page + (size_t)((head - gm.H) * TASC_KV_BLOCK + slot) * gm.hd + e0 : nullptr;
        if (o) {
            o[0] = from_f<T>(ra);
            o[half] = from_f<T>(rc);
        }
    } else if (page) {
        T* vt = page + (size_t)gm.Hkv * TASC_KV_BLOCK * gm.hd + (size_t)((head - gm.H - gm.Hkv) * gm.hd + e0) * TASC_KV_BLOCK + slot;
        vt[0] = from_f<T>(d.v);
        vt[(size_t)half * TASC_KV_BLOCK] = from_f<T>(d.u);
    }
}

// One wave per output column (or pair), rows in chunks of 8, blockIdx.y and gridDim.y chunks on.
// Of a small model's step each launch is a few dependent loads and its own start and end (fp32, d 128, 5 rows: 4.6 to 5.4 us; 4.1 to
// 4.9 with norm, rotation and cache append as launches of 2.4 and 2.8 us beside it): so those ride along, and what an epilogue needs
// is requested before the products.  (The projection inside the attention's workgroups was slower: 22.8 us against 5.4 + 7.8.)
template <typename T, typename AT, int EPI, bool NORM, int VEC>
__global__ __launch_bounds__(256) void k_gemm_generic(const AT* __restrict__ A, const T* __restrict__ W, int M, int N, int K,
                                                      const float* __restrict__ g, float eps, float* outf, T* __restrict__ outT,
                                                      T* __restrict__ kv_layer, GenericRope rp) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int col = blockIdx.x * 4 + wave;
    if (col >= N) return;
    const KvGeom& gm = rp.gm;
    const int half = EPI == EPI_ROPE ? gm.hd / 2 : 1, head = col / half, e0 = col % half;        // EPI_ROPE: the pair's place
    const T *w0, *w1;
    if (EPI == EPI_SWIGLU) {
        w0 = W + (size_t)((col >> 4) * 32 + (col & 15)) * K;
        w1 = w0 + (size_t)16 * K;
    } else if (EPI == EPI_ROPE) {
        w0 = W + (size_t)(head * gm.hd + e0) * K;
        w1 = w0 + (size_t)half * K;
    } else {
        w0 = w1 = W + (size_t)col * K;
    }
    for (int r0 = 8 * blockIdx.y; r0 < M; r0 += 8 * gridDim.y) {
        // what lane r < 8 needs for row r0 + r at the end
        const int row = r0 + lane;
        const bool own = lane < 8 && row < M;
        float old = 0.f, cs = 1.f, sn = 0.f;
        T* page = nullptr;
        int pos = 0;
        if (own && EPI == EPI_RESID) old = outf[(size_t)row * N + col];
        if (own && EPI == EPI_ROPE) {
            const int b = rp.nq ? row / rp.nq : gm.seq(row), i = rp.nq ? row - b * rp.nq : gm.index(row, b);
            const bool active = rp.nq != 0 || i < rp.n_rows[b];
            pos = rp.pos0[b] + i;
            if (head < gm.H + gm.Hkv) {
                const int tpos = pos < rp.max_pos ? pos : rp.max_pos - 1;
                cs = rp.cosT[(size_t)tpos * half + e0];
                sn = rp.sinT[(size_t)tpos * half + e0];
            }
            if (active) page = kv_layer + (size_t)rp.block_tab[(size_t)b * gm.max_blocks + pos / TASC_KV_BLOCK] * gm.page_elems;
        }
        const RowDots d = row_dots<T, AT, EPI != EPI_RESID, NORM, VEC>(A, r0, min(8, M - r0), w0, w1, K, g, eps, lane);
        if (!own) continue;
        if (EPI == EPI_RESID) outf[(size_t)row * N + col] = old + d.v;
        if (EPI == EPI_SWIGLU) outT[(size_t)row * N + col] = from_f<T>(d.v / (1.0f + expf(-d.v)) * d.u);
        if (EPI == EPI_ROPE) rope_store<T>(rp, head, e0, row, pos, page, d, cs, sn, outT);
    }
}

// ---------------------------------------------------------------- generic attention over the paged cache
// One workgroup per (sequence, query head).  Keys are taken in tiles of 64 at absolute positions 0, 64, ...; a tile gives a row its
// maximum, the sum of its exponentials and their products with the values (a lane holds one dimension of the output and reads the 16
// tokens of a value page in one go, ahead of the scores), and the tiles are added in ascending order, rescaled to the larger
// maximum: the same arithmetic whoever computes a tile.  nq: rows of every sequence in a verify step, 0: look them up.  A wave takes
// whole rows, or, in a step whose rows would leave ATTN_GENERIC_IDLE waves or more without one at the end, or whose (row, tile) pairs
// are few, pairs of its own: the tiles of a row meet in LDS, as many of each row at a time as fit.  Latency bounds it (fp32, 32 dimensions,
// one sequence, us, a wave per row | pairs: 100 tokens and 5 rows 9.0 | 7.8, 2000 and 1 row 68 | 23, 3 rows 84 | 61, 9 rows 174 | 157; bf16, 128
// dimensions, 2000 tokens, 3 rows 204 | 108, 9 rows 372 | 300; with one or two waves idle the exchange costs more than they give).
#define ATTN_GENERIC_THREADS 512
#define ATTN_GENERIC_UNITS 32      // (row, tile) pairs that meet in LDS at a time
#define ATTN_GENERIC_ROWS 16       // most rows of a sequence that are taken by pairs
#define ATTN_GENERIC_IDLE 3
struct AttnTile {
    float m, l, acc[4];            // maximum, sum, output dimensions lane, lane + 64, ..
};
template <typename T>
__device__ __forceinline__ AttnTile attn_tile(const float* qi, const T* __restrict__ kv_layer, const int32_t* __restrict__ bt, int first_pages,
                                              const KvGeom& gm, int g, int t0, int L, float scale, int lane) {
    const int hd = gm.hd, key = t0 + lane, nk = min(64, L - t0);
    const size_t v_off = (size_t)gm.Hkv * TASC_KV_BLOCK * hd;
    const T* pages[4];
#pragma unroll
    for (int pg = 0; pg < 4; ++pg) {           // (pages past the row's position are not read, slots past it do not count)
        const int at = min(t0 + TASC_KV_BLOCK * pg, L - 1) / TASC_KV_BLOCK;
        pages[pg] = kv_layer + (size_t)(t0 < 64 * TASC_KV_BLOCK ? __builtin_amdgcn_readlane(first_pages, at & 63) : bt[at]) * gm.page_elems;
    }
    const T* mine = lane < 16 ? pages[0] : lane < 32 ? pages[1] : lane < 48 ? pages[2] : pages[3];
    const T* kp = mine + (size_t)(g * TASC_KV_BLOCK + (key < L ? key : L - 1) % TASC_KV_BLOCK) * hd;
    float v[4][TASC_KV_BLOCK];
    auto load_v = [&](int e) __attribute__((always_inline)) {
#pragma unroll
        for (int pg = 0; pg < 4; ++pg) {
            const T* vt = pages[pg] + v_off + (size_t)(g * hd + min(e, hd - 1)) * TASC_KV_BLOCK;
            load8(vt, v[pg]);
            load8(vt + 8, v[pg] + 8);
        }
    };
    load_v(lane);
    float dot = 0.f;
#pragma unroll 4
    for (int e = 0; e < hd; e += 8) {
        float kvv[8];
        load8(kp + e, kvv);
#pragma unroll
        for (int u = 0; u < 8; ++u) dot = fmaf(qi[e + u], kvv[u], dot);
    }
    AttnTile o;
    const float s = key < L ? dot * scale : -INFINITY;
    o.m = wave_max(s);
    const float p = key < L ? expf(s - (o.m == -INFINITY ? 0.f : o.m)) : 0.f;      // (every product of a tile can overflow to -inf: weights of 0)
    o.l = wave_sum_dpp(p);
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        o.acc[c] = 0.f;
        if (64 * c >= hd) continue;
        if (c > 0) load_v(lane + 64 * c);
#pragma unroll
        for (int pg = 0; pg < 4; ++pg) {
            if (TASC_KV_BLOCK * pg >= nk) break;
#pragma unroll
            for (int q = 0; q < TASC_KV_BLOCK; ++q) {
                const float vq = TASC_KV_BLOCK * pg + q < nk ? v[pg][q] : 0.f;
                o.acc[c] = fmaf(__int_as_float(__builtin_amdgcn_readlane(__float_as_int(p), TASC_KV_BLOCK * pg + q)), vq, o.acc[c]);
            }
        }
    }
    return o;
}
__device__ __forceinline__ void attn_add(float& m, float& l, float& acc, float tm, float tl, float ta) {
    const float mn = fmaxf(m, tm), at = mn == -INFINITY ? 0.f : mn, c1 = expf(m - at), c2 = expf(tm - at);
    l = fmaf(l, c1, tl * c2);
    acc = fmaf(acc, c1, ta * c2);
    m = mn;
}
template <typename T>
__global__ __launch_bounds__(ATTN_GENERIC_THREADS) void k_attn_generic(const T* __restrict__ q, const T* __restrict__ kv_layer,
                                                      const int32_t* __restrict__ n_rows, const int32_t* __restrict__ pos0,
                                                      const int32_t* __restrict__ block_tab, KvGeom gm, float scale, int nq,
                                                      T* __restrict__ att) {
    extern __shared__ float s_q[];             // [waves][hd], then [units][hd + 2]
    constexpr int NW = ATTN_GENERIC_THREADS / 64;
    const int b = blockIdx.x, j = blockIdx.y, g = (j * gm.Hkv) / gm.H;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int32_t* const bt = block_tab + (size_t)b * gm.max_blocks;
    const int first_pages = bt[min(lane, gm.max_blocks - 1)];          // in one go with the position
    const int hd = gm.hd, nr = nq ? nq : n_rows[b], p0 = pos0[b];
    const size_t row0 = nq ? (size_t)b * nq : (size_t)gm.row0[b];
    const size_t qstride = (size_t)gm.H * hd;
    float* const qi = s_q + wave * hd;         // the wave's own query row
    auto load_q = [&](int i) __attribute__((always_inline)) {
        __builtin_amdgcn_wave_barrier();
        for (int e = lane; e < hd; e += 64) qi[e] = to_f(q[(row0 + i) * qstride + j * hd + e]);
        __builtin_amdgcn_wave_barrier();
    };
    float* const s_part = s_q + NW * hd;
    const int tiles = (p0 + nr + 63) / 64;     // of the last row, the most of any
    auto pair = [&](int u, int i, int t0) __attribute__((always_inline)) {       // row i's tile at t0, to place u
        const int L = p0 + i + 1;
        if (t0 >= L) return;
        load_q(i);
        const AttnTile o = attn_tile(qi, kv_layer, bt, first_pages, gm, g, t0, L, scale, lane);
        float* part = s_part + u * (hd + 2);
#pragma unroll
        for (int c = 0; c < 4; ++c)
            if (lane + 64 * c < hd) part[lane + 64 * c] = o.acc[c];
        if (lane == 0) {
            part[hd] = o.m;
            part[hd + 1] = o.l;
        }
    };
    if (gridDim.z == 1 && nr * tiles <= ATTN_GENERIC_UNITS) {
        for (int u = wave; u < nr * tiles; u += NW) pair(u, u / tiles, 64 * (u % tiles));
        __syncthreads();
        for (int idx = threadIdx.x; idx < nr * hd; idx += ATTN_GENERIC_THREADS) {
            const int i = idx / hd, e = idx % hd;
            float m = -INFINITY, l = 0.f, acc = 0.f;
            for (int t = 0; 64 * t < p0 + i + 1; ++t) {
                const float* part = s_part + (i * tiles + t) * (hd + 2);
                attn_add(m, l, acc, part[hd], part[hd + 1], part[e]);
            }
            att[(row0 + i) * qstride + j * hd + e] = from_f<T>(acc / l);
        }
        return;
    }
    if (gridDim.z == 1 && (NW - nr % NW) % NW >= ATTN_GENERIC_IDLE) {            // (at most ATTN_GENERIC_ROWS rows, and one)
        const int per = ATTN_GENERIC_UNITS / nr;                                 // tiles of each row at a time
        constexpr int OWN = ATTN_GENERIC_ROWS * 256 / ATTN_GENERIC_THREADS;                     // (row, dimension) pairs of a thread
        float m[OWN], l[OWN], acc[OWN];
#pragma unroll
        for (int o = 0; o < OWN; ++o) {
            m[o] = -INFINITY;
            l[o] = acc[o] = 0.f;
        }
        for (int tp = 0; tp < tiles; tp += per) {
            const int np = min(per, tiles - tp);
            for (int u = wave; u < nr * np; u += NW) pair(u, u / np, 64 * (tp + u % np));
            __syncthreads();
#pragma unroll
            for (int o = 0; o < OWN; ++o) {
                const int idx = threadIdx.x + o * ATTN_GENERIC_THREADS, i = idx / hd, e = idx % hd;
                if (idx >= nr * hd) break;
                for (int t = 0; t < np && 64 * (tp + t) < p0 + i + 1; ++t) {
                    const float* part = s_part + (i * np + t) * (hd + 2);
                    attn_add(m[o], l[o], acc[o], part[hd], part[hd + 1], part[e]);
                }
            }
            if (tp + per < tiles) __syncthreads();
        }
#pragma unroll
        for (int o = 0; o < OWN; ++o) {
            const int idx = threadIdx.x + o * ATTN_GENERIC_THREADS, i = idx / hd, e = idx % hd;
            if (idx < nr * hd) att[(row0 + i) * qstride + j * hd + e] = from_f<T>(acc[o] / l[o]);
        }
        return;
    }
    for (int i = NW * blockIdx.z + wave; i < nr; i += NW * gridDim.z) {
        load_q(i);
        const int L = p0 + i + 1;
        float m = -INFINITY, l = 0.f, acc[4] = {0, 0, 0, 0};
        for (int t0 = 0; t0 < L; t0 += 64) {
            const AttnTile o = attn_tile(qi, kv_layer, bt, first_pages, gm, g, t0, L, scale, lane);
            const float m0 = m, l0 = l;
#pragma unroll
            for (int c = 0; c < 4; ++c) {      // (the same maximum and sum for every dimension)
                m = m0;
                l = l0;
                attn_add(m, l, acc[c], o.m, o.l, o.acc[c]);
            }
        }
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const int e = lane + 64 * c;
            if (e < hd) att[(row0 + i) * qstride + j * hd + e] = from_f<T>(acc[c] / l);
        }
    }
}

// ---------------------------------------------------------------- generic LM head with fused bias and partial argmax
struct BiasCsr {
    const int64_t* rowptr;
    const int32_t* col;
    const float* val;
    const float* base;
};

// x: NORM: [rows, d] residual stream, LM-head row r is the final RMSNorm (gain gf) of row sel[r] (negative: row 0); else the normalised
// rows themselves.  Row r was fed token tok[r] (its bias row).  WAVES waves take CW columns each, four at a time, and leave per row the
// best (value, index) of the workgroup's columns; index ties go to the lowest.  logits (nullable) receives every logit.
// LOOKUP, few columns a workgroup (vocabularies of few strips): one more wave looks up the rows' seen successors among the columns, eight
// lanes a row, while the others multiply, and leaves their bias in LDS: latency bounds it (512 columns in four workgroups of 16 waves, a
// binary search by one lane per row in front, took 24 us; 6.3 us so).  Else whole strips: the registers hold 16 waves a compute unit and
// no seventeenth, so eight of them look a row up each, in front, and a column's logits are taken as they come (d 2048, vocabulary of 32000,
// fp32, 5 rows 58 us, 62 with a binary search per lane, 70 with 8 waves beside one that looks up; bf16 43 and 69 of the latter two).
template <typename T, int WAVES, int CW, bool LOOKUP, bool NORM, int VEC>
__global__ __launch_bounds__(64 * (WAVES + LOOKUP)) void k_lmhead_generic(const float* __restrict__ x, const int32_t* __restrict__ sel,
                                                        const float* __restrict__ gf, float eps, const T* __restrict__ W,
                                                        const int32_t* __restrict__ tok, int n_rows, int V, int d,
                                                        BiasCsr bias, float* __restrict__ part_val,
                                                        int32_t* __restrict__ part_idx, int n_parts,
                                                        float* __restrict__ logits) {
    constexpr int CB = 4, COLS = WAVES * CW;                          // columns at a time, and of the workgroup
    __shared__ float s_bias[8][COLS];
    __shared__ float s_v[WAVES][8];
    __shared__ int32_t s_i[WAVES][8];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int first = blockIdx.x * COLS, c0 = first + wave * CW;
    for (int r0 = 0; r0 < n_rows; r0 += 8) {
        const int row = r0 + lane;
        const bool own = lane < 8 && row < n_rows;
        float best = -INFINITY;
        int32_t best_i = 0x7FFFFFFF;
        // the bias of row r0 + r at the workgroup's columns, by G lanes, this one number q
        auto row_bias = [&](int r, int q, auto group) __attribute__((always_inline)) {
            constexpr int G = decltype(group)::value;
            float base = 0.f;
            int64_t lo = 0, hi = 0, end = 0;
            if (bias.rowptr && r0 + r < n_rows) {
                const int u = tok[r0 + r];
                base = bias.base[u];
                lo = bias.rowptr[u];
                hi = end = bias.rowptr[u + 1];
            }
            for (int c = q; c < COLS; c += G) s_bias[r][c] = base;
            // first entry of the row with a column >= first: the range in G + 1 parts per look
            while (__ballot(hi - lo > 0) != 0) {
                const int64_t n = hi - lo, at = lo + n * (q + 1) / (G + 1);          // (below hi)
                const u64 below = __ballot(n > 0 && bias.col[at] < first) >> (lane - q);
                const int k = __popcll(G < 64 ? below & ((1ull << (G & 63)) - 1) : below);        // ascending: the first k are
                const int64_t from = k > 0 ? lo + n * k / (G + 1) + 1 : lo;
                if (k < G) hi = lo + n * (k + 1) / (G + 1);
                lo = n > 0 ? from : lo;
                hi = hi > lo ? hi : lo;
            }
            __builtin_amdgcn_wave_barrier();
            for (int64_t p = lo + q; p < end; p += G) {
                const int c = bias.col[p] - first;
                if (c >= COLS) break;
                s_bias[r][c] = bias.val[p];
            }
        };
        // lane r: row r0 + r's logits without bias at columns at .. at + CB - 1
        auto columns = [&](int at, float* z) __attribute__((always_inline)) {
            float acc[CB][8], ss[8];
#pragma unroll
            for (int r = 0; r < 8; ++r) {
                ss[r] = 0.f;
#pragma unroll
                for (int u = 0; u < CB; ++u) acc[u][r] = 0.f;
            }
            size_t from[8];
#pragma unroll
            for (int r = 0; r < 8; ++r) from[r] = (size_t)(NORM ? max(sel[min(r0 + r, n_rows - 1)], 0) : r0 + r) * d;
            for (int k = lane * VEC; k < d; k += 64 * VEC) {
                float wv[CB][VEC], gv[VEC];
                if (NORM) load_n<VEC>(gf + k, gv);
#pragma unroll
                for (int u = 0; u < CB; ++u) load_n<VEC>(W + (size_t)min(at + u, V - 1) * d + k, wv[u]);
#pragma unroll
                for (int u = 0; u < CB; ++u)
#pragma unroll
                    for (int e = 0; e < VEC; ++e)
                        if (NORM) wv[u][e] *= gv[e];
#pragma unroll
                for (int r = 0; r < 8; ++r) {
                    if (r0 + r < n_rows) {
                        float av[VEC];
                        load_n<VEC>(x + from[r] + k, av);
#pragma unroll
                        for (int e = 0; e < VEC; ++e) {
                            if (NORM) ss[r] = fmaf(av[e], av[e], ss[r]);
#pragma unroll
                            for (int u = 0; u < CB; ++u) acc[u][r] = fmaf(av[e], wv[u][e], acc[u][r]);
                        }
                    }
                }
            }
            float mine_s = 0.f;
#pragma unroll
            for (int u = 0; u < CB; ++u) z[u] = 0.f;
#pragma unroll
            for (int r = 0; r < 8; ++r) {
                if (NORM) {
                    const float q = wave_sum_dpp(ss[r]);
                    mine_s = lane == r ? q : mine_s;
                }
#pragma unroll
                for (int u = 0; u < CB; ++u) {
                    const float v = wave_sum_dpp(acc[u][r]);
                    z[u] = lane == r ? v : z[u];
                }
            }
            if (NORM) {
                const float rinv = 1.0f / sqrtf(mine_s / (float)d + eps);
#pragma unroll
                for (int u = 0; u < CB; ++u) z[u] *= rinv;
            }
        };
        auto take = [&](int c, float z) __attribute__((always_inline)) {
            if (!own || c >= V) return;
            const float y = z + s_bias[lane][c - first];
            if (logits) logits[(size_t)row * V + c] = y;
            if (y > best) { best = y; best_i = c; }
        };
        if constexpr (LOOKUP) {                            // one more wave looks the bias up meanwhile
            float z[CW];
            if (wave == WAVES) {
                row_bias(lane >> 3, lane & 7, std::integral_constant<int, 8>{});
            } else {
#pragma unroll
                for (int cb = 0; cb < CW; cb += CB) columns(c0 + cb, z + cb);
            }
            __syncthreads();
            if (wave < WAVES) {
#pragma unroll
                for (int u = 0; u < CW; ++u) take(c0 + u, z[u]);
            }
        } else {                                           // the first eight waves do, a row each, in front
            static_assert(WAVES >= 8, "a wave per row");
            if (wave < 8) row_bias(wave, lane, std::integral_constant<int, 64>{});
            __syncthreads();
#pragma unroll 1
            for (int cb = 0; cb < CW && c0 + cb < V; cb += CB) {
                float z[CB];
                columns(c0 + cb, z);
#pragma unroll
                for (int u = 0; u < CB; ++u) take(c0 + cb + u, z[u]);
            }
        }
        if (wave < WAVES && own) {
            s_v[wave][lane] = best;
            s_i[wave][lane] = best_i;
        }
        __syncthreads();
        if (wave == 0 && own) {
            for (int w = 1; w < WAVES; ++w)
                if (s_v[w][lane] > best) { best = s_v[w][lane]; best_i = s_i[w][lane]; }
            part_val[(size_t)row * n_parts + blockIdx.x] = best;
            part_idx[(size_t)row * n_parts + blockIdx.x] = best_i;
        }
    }
}

// Argmax over the strips of a row (lowest index among equal values) by one wave, the loads of 512 strips in flight at a time: a
// chain of round trips otherwise (576 rows of 1187 strips: 6.2 us, 11.9 with one pair of loads at a time).
__device__ __forceinline__ int32_t strips_argmax(const float* __restrict__ pv, const int32_t* __restrict__ pi, int n_strips, int lane) {
    float bv = -INFINITY;
    int32_t bi = 0x7FFFFFFF;
    for (int s0 = lane; s0 < n_strips; s0 += 512) {
        float v[8];
        int32_t i[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {                     // (past the end the last strip again: it changes nothing)
            const int s = min(s0 + 64 * u, n_strips - 1);
            v[u] = pv[s];
            i[u] = pi[s];
        }
#pragma unroll
        for (int u = 0; u < 8; ++u)
            if (v[u] > bv || (v[u] == bv && i[u] < bi)) { bv = v[u]; bi = i[u]; }
    }
    for (int o = 32; o > 0; o >>= 1) {
        const float v = __shfl_xor(bv, o);
        const int32_t i = __shfl_xor(bi, o);
        if (v > bv || (v == bv && i < bi)) { bv = v; bi = i; }
    }
    return bi == 0x7FFFFFFF ? 0 : bi;                     // all-NaN row: still a valid token id
}
// amax[r] = argmax of row r: the prompt forward's selected rows
__global__ __launch_bounds__(64) void k_argmax_reduce(const float* __restrict__ part_val, const int32_t* __restrict__ part_idx,
                                                      int n_strips, int32_t* __restrict__ amax) {
    const size_t r = blockIdx.x;
    const int32_t t = strips_argmax(part_val + r * n_strips, part_idx + r * n_strips, n_strips, threadIdx.x);
    if (threadIdx.x == 0) amax[r] = t;
}

// The end of a verify step, one workgroup per sequence: a wave per row finds its argmax, then the first wave accepts greedily:
// the longest prefix of the drafts equal to the target's argmax, plus the bonus token; rollback = the cached length only grows by
// the accepted rows.  Latency bounds it (two or three dependent loads); as two launches with the acceptance in one thread
// per sequence they took 4.7 + 4.6 us.
struct AcceptArgs {
    const float* part_val;    // [B (k + 1), n_strips]
    const int32_t* part_idx;
    int32_t n_strips, k, max_len;
    const int32_t* drafts;    // [B, k]
    int32_t *tokens, *n_tok, *cached, *n_emit;
    u64* counters;
    int32_t* accept_len;      // nullable [B]
    int32_t* emitted;         // nullable [B, k + 1]
    int32_t* trace_step;      // nullable [B, 2 k + 3]
};
#define ACCEPT_THREADS(nq) (64 * (nq))       // at most 16 rows a sequence
static_assert(TASC_MAX_K + 1 <= 16, "a wave per row");
__global__ __launch_bounds__(1024) void k_argmax_accept(AcceptArgs a) {
    __shared__ int32_t s_am[16];
    const int b = blockIdx.x, nq = a.k + 1, k = a.k, lane = threadIdx.x & 63, i = threadIdx.x >> 6;
    const int N = a.n_tok[b], emit = a.n_emit[b], cached = a.cached[b], max_new = (int)a.counters[TASC_CTR_MAX_NEW];
    const int draft = lane < k ? a.drafts[b * k + lane] : 0;
    const size_t r = (size_t)b * nq + i;
    const int32_t t = strips_argmax(a.part_val + r * a.n_strips, a.part_idx + r * a.n_strips, a.n_strips, lane);
    if (lane == 0) s_am[i] = t;
    __syncthreads();
    if (i != 0) return;
    const int32_t am = lane < nq ? s_am[lane] : 0;
    const bool frozen = emit >= max_new;
    const u64 differ = __ballot(lane >= k || draft != am);
    const int m = frozen ? 0 : __ffsll((unsigned long long)differ) - 1;
    const int32_t own = lane < m ? draft : am;             // the token that lane <= m emits
    if (!frozen && lane <= m) a.tokens[(size_t)b * a.max_len + N + lane] = own;
    if (a.emitted && lane < nq) a.emitted[b * nq + lane] = frozen || lane > m ? -1 : own;
    if (a.trace_step) {
        int32_t* tr = a.trace_step + (size_t)b * (2 * k + 3);
        if (lane < k) tr[1 + lane] = draft;
        if (lane < nq) tr[1 + k + lane] = am;
        if (lane == 0) {
            tr[0] = N;
            tr[2 * k + 2] = frozen ? -1 : m;
        }
    }
    if (lane != 0) return;
    if (a.accept_len) a.accept_len[b] = m;
    if (!frozen) {
        a.n_tok[b] = N + m + 1;
        a.cached[b] = cached + m + 1;
        a.n_emit[b] = emit + m + 1;
        if (emit + m + 1 >= max_new) atomicAdd(&a.counters[0], 1ull);
        atomicAdd(&a.counters[3], (u64)m);
        atomicAdd(&a.counters[4], (u64)k);
        atomicAdd(&a.counters[8 + m], 1ull);
    }
    if (b == 0) atomicAdd(&a.counters[2], 1ull);
}
