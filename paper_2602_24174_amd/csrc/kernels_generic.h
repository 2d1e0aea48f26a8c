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

__device__ inline float wave_sum(float v) {
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
    return v;
}
__device__ inline float wave_max(float v) {
    for (int o = 32; o > 0; o >>= 1) v = fmaxf(v, __shfl_xor(v, o));
    return v;
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
__global__ void k_embed(const T* __restrict__ E, const int32_t* __restrict__ row_tok, int d, float* __restrict__ x) {
    const int r = blockIdx.x;
    const T* e = E + (size_t)row_tok[r] * d;
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

// ---------------------------------------------------------------- generic GEMM  out[M, N] = A[M, K] W[N, K]^T
enum { EPI_STORE = 0, EPI_RESID = 1, EPI_SWIGLU = 2 };

// One wave per output column (per FFN feature for EPI_SWIGLU), rows in chunks of 8.  Every lane sums
// its own k-slices in ascending order, then a butterfly adds the 64 partial sums.
template <typename T, int EPI>
__global__ __launch_bounds__(256) void k_gemm_generic(const T* __restrict__ A, const T* __restrict__ W, int M, int N, int K,
                                                      float* __restrict__ outf, T* __restrict__ outT) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int col = blockIdx.x * 4 + wave;
    if (col >= N) return;
    const T* w0;
    const T* w1 = nullptr;
    if (EPI == EPI_SWIGLU) {
        w0 = W + (size_t)((col >> 4) * 32 + (col & 15)) * K;
        w1 = w0 + (size_t)16 * K;
    } else {
        w0 = W + (size_t)col * K;
    }
    for (int r0 = 0; r0 < M; r0 += 8) {
        float acc[8] = {0, 0, 0, 0, 0, 0, 0, 0}, acu[8] = {0, 0, 0, 0, 0, 0, 0, 0};
        for (int k = lane * 8; k < K; k += 512) {
            float wv[8], uv[8];
            load8(w0 + k, wv);
            if (EPI == EPI_SWIGLU) load8(w1 + k, uv);
#pragma unroll
            for (int r = 0; r < 8; ++r) {
                if (r0 + r < M) {
                    float av[8];
                    load8(A + (size_t)(r0 + r) * K + k, av);
#pragma unroll
                    for (int e = 0; e < 8; ++e) {
                        acc[r] = fmaf(av[e], wv[e], acc[r]);
                        if (EPI == EPI_SWIGLU) acu[r] = fmaf(av[e], uv[e], acu[r]);
                    }
                }
            }
        }
        float mine = 0.f, mine_u = 0.f;
#pragma unroll
        for (int r = 0; r < 8; ++r) {
            float v = wave_sum(acc[r]);
            if (lane == r) mine = v;
            if (EPI == EPI_SWIGLU) {
                float u = wave_sum(acu[r]);
                if (lane == r) mine_u = u;
            }
        }
        const int row = r0 + lane;
        if (lane < 8 && row < M) {
            if (EPI == EPI_STORE) outf[(size_t)row * N + col] = mine;
            if (EPI == EPI_RESID) outf[(size_t)row * N + col] += mine;
            if (EPI == EPI_SWIGLU) outT[(size_t)row * N + col] = from_f<T>(mine / (1.0f + expf(-mine)) * mine_u);
        }
    }
}

// ---------------------------------------------------------------- RoPE + KV append
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

// Row r = (sequence b, i) sits at position pos0[b] + i.  q is rotated into `q_out`; k is rotated and
// written to the K half of its page, v to the transposed V half.  Rows beyond n_rows[b] write nothing.
// `qkv` may be n_slices partial sums [n_slices][rows][nqkv] (slice_stride elements apart), added here in slice order.
template <typename T>
__global__ void k_rope_kv(const float* __restrict__ qkv, const float* __restrict__ cosT, const float* __restrict__ sinT,
                          int max_pos, const int32_t* __restrict__ n_rows, const int32_t* __restrict__ pos0,
                          const int32_t* __restrict__ block_tab, KvGeom gm, T* __restrict__ q_out, T* __restrict__ kv_layer,
                          int n_slices = 1, size_t slice_stride = 0) {
    const int r = blockIdx.x, b = gm.seq(r), i = gm.index(r, b);
    const bool active = i < n_rows[b];
    const int pos = pos0[b] + i;
    const int tpos = pos < max_pos ? pos : max_pos - 1;
    const int half = gm.hd / 2, nqkv = (gm.H + 2 * gm.Hkv) * gm.hd;
    const float* src = qkv + (size_t)r * nqkv;
    T* page = nullptr;
    const int slot = pos % TASC_KV_BLOCK;
    if (active) page = kv_layer + (size_t)block_tab[(size_t)b * gm.max_blocks + pos / TASC_KV_BLOCK] * gm.page_elems;
    for (int idx = threadIdx.x; idx < (gm.H + 2 * gm.Hkv) * half; idx += blockDim.x) {
        const int head = idx / half, e = idx % half;
        float a = src[head * gm.hd + e], c = src[head * gm.hd + e + half];
        for (int sl = 1; sl < n_slices; ++sl) {            // k-slices of a split projection, added in slice order
            a += src[(size_t)sl * slice_stride + head * gm.hd + e];
            c += src[(size_t)sl * slice_stride + head * gm.hd + e + half];
        }
        if (head < gm.H + gm.Hkv) {
            const float cs = cosT[(size_t)tpos * half + e], sn = sinT[(size_t)tpos * half + e];
            const float ra = a * cs - c * sn, rc = c * cs + a * sn;
            if (head < gm.H) {
                q_out[(size_t)r * gm.H * gm.hd + head * gm.hd + e] = from_f<T>(ra);
                q_out[(size_t)r * gm.H * gm.hd + head * gm.hd + e + half] = from_f<T>(rc);
            } else if (active) {
                const int g = head - gm.H;
                page[(size_t)(g * TASC_KV_BLOCK + slot) * gm.hd + e] = from_f<T>(ra);
                page[(size_t)(g * TASC_KV_BLOCK + slot) * gm.hd + e + half] = from_f<T>(rc);
            }
        } else if (active) {
            const int g = head - gm.H - gm.Hkv;
            T* vt = page + (size_t)gm.Hkv * TASC_KV_BLOCK * gm.hd;
            vt[(size_t)(g * gm.hd + e) * TASC_KV_BLOCK + slot] = from_f<T>(a);
            vt[(size_t)(g * gm.hd + e + half) * TASC_KV_BLOCK + slot] = from_f<T>(c);
        }
    }
}

// ---------------------------------------------------------------- generic attention over the paged cache
// One workgroup per (sequence, query head); a wave per query row.  Keys are visited in tiles of 64 at
// absolute positions 0, 64, ...; running max / sum (online softmax) in fp32.  A lane holds one dimension of the output and
// reads the 16 tokens of a value page in one go (they are contiguous), all pages of the tile ahead of the first product: with a
// load per key, one sequence of 100 tokens took 46 us, nearly all of it waiting.
#define ATTN_GENERIC_THREADS 512
template <typename T>
__global__ __launch_bounds__(ATTN_GENERIC_THREADS) void k_attn_generic(const T* __restrict__ q, const T* __restrict__ kv_layer,
                                                      const int32_t* __restrict__ n_rows, const int32_t* __restrict__ pos0,
                                                      const int32_t* __restrict__ block_tab, KvGeom gm, float scale,
                                                      T* __restrict__ att) {
    extern __shared__ float s_q[];   // [most rows of a sequence][hd]
    const int b = blockIdx.x, j = blockIdx.y, g = (j * gm.Hkv) / gm.H;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int hd = gm.hd, nr = n_rows[b], p0 = pos0[b];
    const size_t qstride = (size_t)gm.H * hd, row0 = gm.row0[b];
    for (int idx = threadIdx.x; idx < nr * hd; idx += blockDim.x) {
        const int i = idx / hd, e = idx % hd;
        s_q[idx] = to_f(q[(row0 + i) * qstride + j * hd + e]);
    }
    __syncthreads();
    const int32_t* bt = block_tab + (size_t)b * gm.max_blocks;
    const size_t v_off = (size_t)gm.Hkv * TASC_KV_BLOCK * hd;
    for (int i = wave; i < nr; i += ATTN_GENERIC_THREADS / 64) {
        T* out = att + (row0 + i) * qstride + j * hd;
        const float* qi = s_q + i * hd;
        const int L = p0 + i + 1;
        float m = -INFINITY, l = 0.f, acc[4] = {0, 0, 0, 0};
        for (int t0 = 0; t0 < L; t0 += 64) {
            const int key = t0 + lane;
            float s = -INFINITY;
            if (key < L) {
                const T* kp = kv_layer + (size_t)bt[key / TASC_KV_BLOCK] * gm.page_elems +
                              (size_t)(g * TASC_KV_BLOCK + key % TASC_KV_BLOCK) * hd;
                float dot = 0.f;
#pragma unroll 4
                for (int e = 0; e < hd; e += 8) {
                    float kvv[8];
                    load8(kp + e, kvv);
#pragma unroll
                    for (int u = 0; u < 8; ++u) dot = fmaf(qi[e + u], kvv[u], dot);
                }
                s = dot * scale;
            }
            const float m_new = fmaxf(m, wave_max(s));
            const float corr = expf(m - m_new);
            const float p = key < L ? expf(s - m_new) : 0.f;
            l = l * corr + wave_sum(p);
            m = m_new;
            const int nk = min(64, L - t0);
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                acc[c] *= corr;
                const int e = lane + 64 * c;
                if (64 * c >= hd) break;
                // (pages past the row's position are not read, slots past it do not count)
                float v[4][TASC_KV_BLOCK];
#pragma unroll
                for (int pg = 0; pg < 4; ++pg) {
                    const int kpos = min(t0 + TASC_KV_BLOCK * pg, L - 1);
                    const T* vt = kv_layer + (size_t)bt[kpos / TASC_KV_BLOCK] * gm.page_elems + v_off + (size_t)(g * hd + min(e, hd - 1)) * TASC_KV_BLOCK;
                    load8(vt, v[pg]);
                    load8(vt + 8, v[pg] + 8);
                }
#pragma unroll
                for (int pg = 0; pg < 4; ++pg) {
                    if (TASC_KV_BLOCK * pg >= nk) break;
#pragma unroll
                    for (int q = 0; q < TASC_KV_BLOCK; ++q) {
                        const float vq = TASC_KV_BLOCK * pg + q < nk ? v[pg][q] : 0.f;
                        acc[c] = fmaf(__int_as_float(__builtin_amdgcn_readlane(__float_as_int(p), TASC_KV_BLOCK * pg + q)), vq, acc[c]);
                    }
                }
            }
        }
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const int e = lane + 64 * c;
            if (e < hd) out[e] = from_f<T>(acc[c] / l);
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

// h: [n_rows, d] normalised hidden rows; row r was fed token tok[r] (bias row).  A workgroup covers a
// strip of TASC_LM_STRIP vocabulary columns, 8 per wave, and leaves, per row, the best (value, index)
// of its strip; index ties go to the lowest column.  logits (nullable) receives every logit.  Four columns
// at a time: the 32 sums over the wave are independent chains (one column at a time and 32 columns a wave, a vocabulary of
// 512 took 50 us, all of it the chains' latency).
#define LM_GENERIC_WAVES 16
template <typename T>
__global__ __launch_bounds__(64 * LM_GENERIC_WAVES) void k_lmhead_generic(const T* __restrict__ h, const T* __restrict__ W,
                                                        const int32_t* __restrict__ tok, int n_rows, int V, int d,
                                                        BiasCsr bias, float* __restrict__ part_val,
                                                        int32_t* __restrict__ part_idx, int n_strips,
                                                        float* __restrict__ logits) {
    constexpr int CW = TASC_LM_STRIP / LM_GENERIC_WAVES, CB = 4;      // columns of a wave, and at a time
    __shared__ float s_v[LM_GENERIC_WAVES][8];
    __shared__ int32_t s_i[LM_GENERIC_WAVES][8];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int strip = blockIdx.x;
    const int c0 = strip * TASC_LM_STRIP + wave * CW;
    for (int r0 = 0; r0 < n_rows; r0 += 8) {
        const int row = r0 + lane;
        const bool own = lane < 8 && row < n_rows;
        float best = -INFINITY;
        int32_t best_i = 0x7FFFFFFF;
        int64_t bp = 0, be = 0;
        float base = 0.f;
        if (own && bias.rowptr) {
            const int u = tok[row];
            int64_t lo = bias.rowptr[u];
            be = bias.rowptr[u + 1];
            int64_t hi = be;
            while (lo < hi) {   // first entry of the row with column >= c0
                int64_t mid = (lo + hi) >> 1;
                if (bias.col[mid] < c0) lo = mid + 1; else hi = mid;
            }
            bp = lo;
            base = bias.base[u];
        }
        for (int cb = c0; cb < c0 + CW && cb < V; cb += CB) {
            float acc[CB][8];
#pragma unroll
            for (int u = 0; u < CB; ++u)
#pragma unroll
                for (int r = 0; r < 8; ++r) acc[u][r] = 0.f;
            for (int k = lane * 8; k < d; k += 512) {
                float wv[CB][8];
#pragma unroll
                for (int u = 0; u < CB; ++u) load8(W + (size_t)min(cb + u, V - 1) * d + k, wv[u]);
#pragma unroll
                for (int r = 0; r < 8; ++r) {
                    if (r0 + r < n_rows) {
                        float av[8];
                        load8(h + (size_t)(r0 + r) * d + k, av);
#pragma unroll
                        for (int u = 0; u < CB; ++u)
#pragma unroll
                            for (int e = 0; e < 8; ++e) acc[u][r] = fmaf(av[e], wv[u][e], acc[u][r]);
                    }
                }
            }
            float mine[CB];
#pragma unroll
            for (int u = 0; u < CB; ++u) mine[u] = 0.f;
#pragma unroll
            for (int r = 0; r < 8; ++r)
#pragma unroll
                for (int u = 0; u < CB; ++u) {
                    const float v = wave_sum(acc[u][r]);
                    if (lane == r) mine[u] = v;
                }
#pragma unroll
            for (int u = 0; u < CB; ++u) {
                const int c = cb + u;
                if (own && c < V) {
                    float z = mine[u];
                    if (bias.rowptr) {
                        if (bp < be && bias.col[bp] == c) z += bias.val[bp++];
                        else z += base;
                    }
                    if (logits) logits[(size_t)row * V + c] = z;
                    if (z > best) { best = z; best_i = c; }
                }
            }
        }
        if (lane < 8) { s_v[wave][lane] = best; s_i[wave][lane] = best_i; }
        __syncthreads();
        if (wave == 0 && own) {
            float bv = s_v[0][lane];
            int32_t bi = s_i[0][lane];
            for (int w = 1; w < LM_GENERIC_WAVES; ++w)
                if (s_v[w][lane] > bv) { bv = s_v[w][lane]; bi = s_i[w][lane]; }
            part_val[(size_t)row * n_strips + strip] = bv;
            part_idx[(size_t)row * n_strips + strip] = bi;
        }
        __syncthreads();
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
