// One target forward over M rows, at most nq of a sequence, against the paged KV cache, ending (optionally) in the
// LM head with fused bias and argmax.  Used by the prompt forward (nq = chunk length) and by the
// verify step (nq = k + 1; paper, subsection "Speculative Decoding": the drafted tokens are verified
// in parallel via a single forward pass).
//
// The order in which a row is reduced depends on the model and the session only, never on data or on the
// other rows of the call (whose number chooses tile shapes, which do not change it), so plain greedy decoding
// (k = 0) and speculative decoding of one session agree bit for bit, and a prompt's cache and first token do not
// depend on the prompts beside it.
#include "tasc_internal.h"
#include "kernels_generic.h"
#include "kernels_small.h"
#include "kernels_pipe.h"
#include "kernels_tiled.h"
#include <algorithm>
#include <type_traits>
#include <utility>

TascConfig g_tasc_config = {/*small_path*/ 2, /*small_grid*/ 0, /*layer_wgs*/ 0, /*layer_stride*/ 0, /*tiled_path*/ 1, /*xcd_local*/ 1,
                             /*layer_workers*/ 0, /*small_kernel*/ 1, /*pipe_share*/ 1, /*chains*/ 0, /*step_graph*/ 1, /*build_list_kib*/ 8 << 20,
                             /*enrich_wait*/ 1 << 20};
// One-time set-up (kernel attributes, the compute-unit count) is kept per device and done under a lock, so that calls
// from several host threads, or sessions on different devices of one process, each find their own device prepared.
#include <mutex>
namespace {
struct DevState { bool tiled_ready = false, small_ready = false, pipe_ready = false; int cu_count = 0; };
DevState g_dev[16];
std::mutex g_dev_mu;
DevState& dev_state() {
    int dev = 0;
    (void)hipGetDevice(&dev);
    return g_dev[dev & 15];
}
}  // namespace
static u64* g_phase_ts = nullptr;
static int64_t g_phase_ts_cap = 0;

extern "C" tasc_status tasc_profile_phases(uint64_t* device_buf, int64_t capacity) {
    TASC_REQUIRE(capacity >= 0 && (device_buf || capacity == 0), "profile_phases: bad buffer");
    g_phase_ts = (u64*)device_buf;
    g_phase_ts_cap = device_buf ? capacity : 0;
    return TASC_OK;
}

extern "C" tasc_status tasc_config_set(int32_t key, int32_t value) {
    if (key == TASC_CFG_SMALL_PATH) {
        TASC_REQUIRE(value >= 0 && value <= 2, "config_set: small path %d outside [0, 2]", value);
        g_tasc_config.small_path = value;
    } else if (key == TASC_CFG_SMALL_GRID) {
        TASC_REQUIRE(value >= 0 && value <= 4096, "config_set: grid %d outside [0, 4096]", value);
        g_tasc_config.small_grid = value;
    } else if (key == TASC_CFG_TILED_PATH) {
        TASC_REQUIRE(value == 0 || value == 1, "config_set: tiled path %d outside [0, 1]", value);
        g_tasc_config.tiled_path = value;
    } else if (key == TASC_CFG_SMALL_LAYER_WGS) {
        TASC_REQUIRE(value >= 0 && value <= 4096, "config_set: layer workgroups %d outside [0, 4096]", value);
        g_tasc_config.layer_wgs = value;
    } else if (key == TASC_CFG_SMALL_LAYER_STRIDE) {
        TASC_REQUIRE(value >= 0 && value <= 64, "config_set: layer stride %d outside [0, 64]", value);
        g_tasc_config.layer_stride = value;
    } else if (key == TASC_CFG_SMALL_LAYER_WORKERS) {
        TASC_REQUIRE(value >= 0 && value <= 64, "config_set: layer workers %d outside [0, 64]", value);
        g_tasc_config.layer_workers = value;
    } else if (key == TASC_CFG_SMALL_KERNEL) {
        TASC_REQUIRE(value == 0 || value == 1, "config_set: small kernel %d outside [0, 1]", value);
        g_tasc_config.small_kernel = value;
    } else if (key == TASC_CFG_STEP_GRAPH) {
        TASC_REQUIRE(value == 0 || value == 1, "config_set: step graph %d outside [0, 1]", value);
        g_tasc_config.step_graph = value;
    } else if (key == TASC_CFG_CHAINS) {
        TASC_REQUIRE(value >= 0 && value <= TASC_MAX_CHAINS, "config_set: chains %d outside [0, %d]", value, TASC_MAX_CHAINS);
        g_tasc_config.chains = value;
    } else if (key == TASC_CFG_BUILD_LIST_KIB) {
        TASC_REQUIRE(value >= 0, "config_set: build list size %d KiB", value);
        g_tasc_config.build_list_kib = value;
    } else if (key == TASC_CFG_KEEP_SCRATCH_KIB) {
        TASC_REQUIRE(value >= 0 && value <= 2 << 20, "config_set: kept scratch %d KiB outside [0, %d]", value, 2 << 20);
        tasc_scratch_limit((size_t)value << 10);
    } else if (key == TASC_CFG_ENRICH_WAIT) {
        TASC_REQUIRE(value >= 0, "config_set: enrichment wait %d", value);
        g_tasc_config.enrich_wait = value;
    } else if (key == TASC_CFG_PIPE_SHARE) {
        TASC_REQUIRE(value >= 1 && value <= 3, "config_set: pipeline share %d outside [1, 3]", value);
        g_tasc_config.pipe_share = value;
    } else if (key == TASC_CFG_SMALL_XCD_LOCAL) {
        TASC_REQUIRE(value == 0 || value == 1, "config_set: XCD-local switch %d outside [0, 1]", value);
        g_tasc_config.xcd_local = value;
    } else {
        tasc_set_error("config_set: unknown key %d", key);
        return TASC_EINVAL;
    }
    return TASC_OK;
}

namespace {

#define PROF(cls) TascProfScope _ps(cls, st)

StepRows step_rows(const tasc_model* m, const tasc_session* s, const TascVerifyTail* tail) {
    const TascSessDev& d = s->d;
    if (!tail) return StepRows{};
    return StepRows{d.tokens, d.n_tok, d.cached, tail->drafts, s->max_len, tail->k, m->desc.vocab, d.row_tok, d.row_seq, d.row0, d.n_rows, d.pos0,
                    d.sel_rows, d.sel_tok};
}
tasc_status prepare_verify(const tasc_model* m, const tasc_session* s, const TascVerifyTail* tail, hipStream_t st) {
    if (!tail) return TASC_OK;
    const int rows = s->batch * (tail->k + 1);
    k_prepare_verify<<<dim3((rows + 255) / 256), dim3(256), 0, st>>>(step_rows(m, s, tail), rows);
    TASC_LAUNCH_CHECK();
    return TASC_OK;
}
// the LM head's partial maxima -> argmax of the selected rows (a prompt forward), or the acceptance of a verify step
tasc_status finish_rows(const tasc_session* s, int n_sel, int n_parts, const float* part_val, const int32_t* part_idx, const TascVerifyTail* tail,
                        hipStream_t st) {
    const TascSessDev& d = s->d;
    PROF(TASC_KC_ACCEPT);
    if (tail)
        k_argmax_accept<<<dim3(s->batch), dim3(ACCEPT_THREADS(tail->k + 1)), 0, st>>>(
            AcceptArgs{part_val, part_idx, n_parts, tail->k, s->max_len, tail->drafts, d.tokens, d.n_tok, d.cached, d.n_emit, d.counters,
                       tail->accept_len, tail->emitted, tail->trace_step});
    else k_argmax_reduce<<<dim3(n_sel), dim3(64), 0, st>>>(part_val, part_idx, n_parts, d.amax);
    TASC_LAUNCH_CHECK();
    return TASC_OK;
}

template <typename T>
tasc_status forward_generic(const tasc_model* m, tasc_session* s, int nq, int M, int n_sel, float* logits_dbg, const TascVerifyTail* tail, hipStream_t st) {
    const tasc_model_desc& c = m->desc;
    const TascSessDev& d = s->d;
    const int D = c.d_model, H = c.n_heads, Hkv = c.n_kv_heads, hd = c.head_dim, F = c.d_ffn;
    const int pairs = (H + 2 * Hkv) * (hd / 2), nqo = H * hd;
    const KvGeom gm{H, Hkv, hd, s->max_blocks, s->page_elems, d.row_seq, d.row0, 0};
    const GenericRope rope{m->rope_cos, m->rope_sin, d.n_rows, d.pos0, d.block_tab, gm, c.max_pos, tail ? nq : 0};
    const float scale = 1.0f / sqrtf((float)hd);
    const size_t att_lds = ((size_t)(ATTN_GENERIC_THREADS / 64) * hd + (size_t)ATTN_GENERIC_UNITS * (hd + 2)) * sizeof(float);
    const unsigned chunks = (unsigned)std::min((M + 7) / 8, 64);      // chunks of rows side by side
    {
        PROF(TASC_KC_PREPARE);
        k_embed<T><<<dim3(M), dim3(64), 0, st>>>((const T*)m->embed, d.row_tok, D, d.x, step_rows(m, s, tail));
    }
    TASC_LAUNCH_CHECK();
    // a product of the residual stream's norm, or of `in`; lanes take 8 columns at a time where that leaves none of them out
    const bool along = D <= kNormAlong;
    float* const h = (float*)d.h;
    auto product = [&](auto epi, const auto* in, const float* gain, const void* weights, int n, int k, float* outf, T* outT, T* kv_layer, const GenericRope& rp) {
        constexpr int EPI = decltype(epi)::value;
        using AT = std::remove_cv_t<std::remove_pointer_t<decltype(in)>>;
        const dim3 grid((n + 3) / 4, chunks);
        if (gain && along) {
            if constexpr (std::is_same_v<AT, float>)
                k_gemm_generic<T, AT, EPI, true, 4><<<grid, dim3(256), 0, st>>>(in, (const T*)weights, M, n, k, gain, c.rms_eps, outf, outT, kv_layer, rp);
        } else if (k < 512) {
            k_gemm_generic<T, AT, EPI, false, 4><<<grid, dim3(256), 0, st>>>(in, (const T*)weights, M, n, k, nullptr, 0.f, outf, outT, kv_layer, rp);
        } else {
            k_gemm_generic<T, AT, EPI, false, 8><<<grid, dim3(256), 0, st>>>(in, (const T*)weights, M, n, k, nullptr, 0.f, outf, outT, kv_layer, rp);
        }
    };
    auto norm = [&](const float* gain, const int32_t* sel, int rows) {
        if (along) return;
        PROF(TASC_KC_NORM);
        k_rmsnorm<float><<<dim3(rows), dim3(64), 0, st>>>(d.x, gain, sel, D, c.rms_eps, h);
    };
    const float* const rows_in = along ? d.x : h;
    for (int l = 0; l < c.n_layers; ++l) {
        const TascLayerW& w = m->layers[l];
        T* kv_layer = (T*)s->kv_pool + (size_t)l * s->kv_layer_stride;
        norm(w.g1, nullptr, M);
        {
            PROF(TASC_KC_GEMM_QKV);
            product(std::integral_constant<int, EPI_ROPE>{}, rows_in, w.g1, w.wqkv, pairs, D, nullptr, (T*)d.q, kv_layer, rope);
        }
        {
            PROF(TASC_KC_ATTN);
            k_attn_generic<T><<<dim3(s->batch, H, nq <= ATTN_GENERIC_ROWS ? 1 : (nq + 7) / 8), dim3(ATTN_GENERIC_THREADS), att_lds, st>>>(
                (const T*)d.q, kv_layer, d.n_rows, d.pos0, d.block_tab, gm, scale, tail ? nq : 0, (T*)d.att);
        }
        {
            PROF(TASC_KC_GEMM_O);
            product(std::integral_constant<int, EPI_RESID>{}, (const T*)d.att, nullptr, w.wo, D, nqo, d.x, nullptr, nullptr, GenericRope{});
        }
        norm(w.g2, nullptr, M);
        {
            PROF(TASC_KC_GEMM_GU);
            product(std::integral_constant<int, EPI_SWIGLU>{}, rows_in, w.g2, w.wgu, F, D, nullptr, (T*)d.act, nullptr, GenericRope{});
        }
        {
            PROF(TASC_KC_GEMM_D);
            product(std::integral_constant<int, EPI_RESID>{}, (const T*)d.act, nullptr, w.wd, D, F, d.x, nullptr, nullptr, GenericRope{});
        }
        TASC_LAUNCH_CHECK();
    }
    if (n_sel > 0) {
        const BiasCsr bias{m->bias_rowptr, m->bias_col, m->bias_val, m->bias_base};
        const int split = tasc_generic_lm_split(s->n_strips, D), parts = s->n_strips * split;
        norm(m->gf, d.sel_rows, n_sel);
        {
            PROF(TASC_KC_LMHEAD);
            auto head = [&](auto kernel, int threads) {
                kernel<<<dim3(parts), dim3(threads), 0, st>>>(rows_in, d.sel_rows, m->gf, c.rms_eps, (const T*)m->lm_head, d.sel_tok, n_sel, c.vocab, D, bias,
                                                             d.part_val, d.part_idx, parts, logits_dbg);
            };
            constexpr int strip = TASC_LM_STRIP;
            if (split == 8) along ? head(&k_lmhead_generic<T, 4, strip / 32, true, true, 4>, 320) : D < 512 ? head(&k_lmhead_generic<T, 4, strip / 32, true, false, 4>, 320)
                                                                                                  : head(&k_lmhead_generic<T, 4, strip / 32, true, false, 8>, 320);
            else along ? head(&k_lmhead_generic<T, 16, strip / 16, false, true, 4>, 1024) : D < 512 ? head(&k_lmhead_generic<T, 16, strip / 16, false, false, 4>, 1024)
                                                                                        : head(&k_lmhead_generic<T, 16, strip / 16, false, false, 8>, 1024);
        }
        TASC_LAUNCH_CHECK();
        return finish_rows(s, n_sel, parts, d.part_val, d.part_idx, tail, st);
    }
    return TASC_OK;
}

// the LDS-tiled MFMA kernels serve bf16 forwards of any row count with these shapes
}  // namespace
bool tasc_tiled_fits(const tasc_model_desc& c) {
    return c.dtype == TASC_BF16 && c.d_model % 64 == 0 && (c.n_heads * c.head_dim) % 64 == 0 && c.d_ffn % 64 == 0 &&
           (c.head_dim == 32 || c.head_dim == 64 || c.head_dim == 128);
}
namespace {

// Tile shapes (output features x rows, waves along each): 128 x 128, and 256 x 256 or 256 x 192 for row counts where the GEMMs are
// MFMA-bound.  All reduce every output element over k in the same order, so the choice may depend on the row count.
#define TILE_SMALL 128, 128, 2, 2
#define TILE_MID 256, 192, 4, 2        // 192 rows per tile where that leaves fewer padded rows than 256 (576 = 3 x 192)
#define TILE_NARROW 64, 128, 1, 4      // few rows and a narrow output: twice the workgroups of the small tile
// k_gemm (kernels_gemm.h) takes all launches but these, which fill their LDS through registers (kernels_tiled.h): one round of tiles over at
// most kFewRows rows, whose weights come from memory for a few row tiles only and are fetched further ahead there (us, registers | straight to
// LDS: gate/up 576 x 17920 x 1536 in 256 x 192 tiles 38.4 | 42.8, 224 x 9728 x 896 in 128 x 128 ones 12.3 | 12.7, 224 x 896 x 4864 in
// six slices of 64 x 128 ones 8.5 | 8.8; with more row tiles gate/up 1000 x 9728 x 896 27.2 | 26.8, output 6336 x 1536 x 1536 46.4 | 42.2; one round of
// 256 x 192 tiles, N 2048 to 17920, warm operands: straight to LDS takes 0.998 to 1.015 of the time at 384 to 768 rows, 0.94 to 1.02 at 832 to 1152), the
// narrow tile, and the 128 x 128 tile's SwiGLU, rotation and k-slices in one round.  The first two have spans of 64 or 128 features a wave, and so
// four waves of 64 x 64; the other epilogues take eight of 32 x 64 (us, four waves through registers | eight straight to LDS: 1280 x 2048 x 2048
// with residual 25.4 | 21.5, 3072 x 1536 x 8960 151 | 134; slices in one round: 1137 x 896 x 4864 in four 16.3 | 17.8 and the reduction behind them
// 5.7 | 7.9, 576 x 1536 x 8960 in four 23.8 | 24.1, 576 x 2048 x 1536 in two 11.1 | 10.5; in more than one 1280 x 2048 x 11008 in six 89 | 81).
// Stages of 64 of k, two in LDS for the large tiles, four for the small one: a stage of 32 of k is half a cache line of a row, and each half is
// a request of its own (128 x 128, 1280 x 2560 x 2048, eight stages of 32 | four of 64: 29.4 | 23.1).  (So for the LM head's large tile: 1280 x 49152 x 2048 without
// logits, four stages of 32 | two of 64: 245 | 219, 1280 x 151936 x 2048 705 | 654.)
#define GEMM_SMALL 128, 128, 4, 2, 4
#define GEMM_SMALL_GU 128, 128, 2, 4, 4
#define GEMM_SMALL_ROPE 128, 128, 1, 4, 4
#define GEMM_LARGE 256, 256, 2, 4, 2
#define GEMM_MID 256, 192, 4, 2, 2
constexpr int kFewRows = 768;
constexpr int kLargeTileRows = 384;

// kernel and LDS; the head size is the rotation's only
template <int EPI, int HD>
constexpr auto gemm_large() {
    return std::pair(&k_gemm<EPI, GEMM_LARGE, HD>, gemm_lds_bytes(GEMM_LARGE));
}
template <int EPI, int HD>
constexpr auto gemm_small() {
    if constexpr (EPI == TEPI_SWIGLU) return std::pair(&k_gemm<EPI, GEMM_SMALL_GU>, gemm_lds_bytes(GEMM_SMALL_GU));
    else if constexpr (EPI == TEPI_ROPE) return std::pair(&k_gemm<EPI, GEMM_SMALL_ROPE, HD>, gemm_lds_bytes(GEMM_SMALL_ROPE));
    else return std::pair(&k_gemm<EPI, GEMM_SMALL>, gemm_lds_bytes(GEMM_SMALL));
}
// f(head_dim as a type), 0 where the epilogue has no use for it
template <int EPI>
auto with_head_dim(int hd, auto f) {
    if constexpr (EPI != TEPI_ROPE) return f(std::integral_constant<int, 0>{});
    else return hd == 128 ? f(std::integral_constant<int, 128>{}) : hd == 64 ? f(std::integral_constant<int, 64>{}) : f(std::integral_constant<int, 32>{});
}
constexpr bool small_in_registers(int epi) { return epi == TEPI_SWIGLU || epi == TEPI_ROPE || epi == TEPI_PARTIAL; }

template <int EPI>
tasc_status tiled_attrs() {
    auto lds = [](auto kernel, int bytes) { return hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, bytes); };
    for (int hd : {32, 64, 128})
        TASC_HIP(with_head_dim<EPI>(hd, [&](auto h) {
            constexpr auto large = gemm_large<EPI, decltype(h)::value>();
            const hipError_t rc = lds(large.first, large.second);
            if constexpr (EPI == TEPI_LMHEAD) return rc;
            else {
                constexpr auto small = gemm_small<EPI, decltype(h)::value>();
                return rc != hipSuccess ? rc : lds(small.first, small.second);
            }
        }));
    if constexpr (EPI != TEPI_ROPE) TASC_HIP(lds(&k_gemm<EPI, GEMM_MID>, gemm_lds_bytes(GEMM_MID)));
    if constexpr (EPI == TEPI_LMHEAD || small_in_registers(EPI)) TASC_HIP(lds(&k_gemm_tiled<EPI, TILE_SMALL>, TG_LDS_BYTES(128, 128)));
    if constexpr (EPI != TEPI_LMHEAD) {
        TASC_HIP(lds(&k_gemm_tiled<EPI, TILE_NARROW>, TG_LDS_BYTES(64, 128)));
        TASC_HIP(lds(&k_gemm_tiled<EPI, TILE_MID>, TG_LDS_BYTES(256, 192)));
    }
    return TASC_OK;
}

// launches out = epilogue(A W^T) with the tile shape that suits M; `slices` > 1 only for TEPI_PARTIAL
template <int EPI>
void launch_gemm(const BF16* A, const void* Wm, int M, int N, int K, float* outf, BF16* outb, const LmEpi& lm, int slices,
                 hipStream_t st, int cus, const RopeEpi& rp = RopeEpi{}) {
    // large tiles need enough of them to fill the chip: narrow outputs stay on the small tile (the k order, and so
    // every row's result, is the same for both shapes)
    const long large_wgs = (long)((M + 255) / 256) * ((N + 255) / 256) * slices;
    const long small_wgs = (long)((M + 127) / 128) * ((N + 127) / 128) * slices;
    // ... a very wide output takes them from 129 rows on: one row tile then reads every weight tile once, and the activations
    // are re-read per 256 instead of per 128 output features.  The LM head takes the streaming kernel as soon as the small tiles
    // are more than one per compute unit: it stores logits as whole row segments and hides the weights' latency (us of a whole
    // verify step of one layer, with logits, small | streaming: 160 x 49152 x 896 156 | 115, 224 x 49152 x 2048 224 | 181,
    // 301 x 16384 x 896 133 | 116, 64 x 49152 x 896 123 | 109; one per compute unit: 224 x 16384 x 896 106 | 125,
    // 128 x 32768 x 2048 131 | 146; us of the launch alone without logits, as in the decode loop, with the bias of a corpus of 32 M
    // tokens: 40 x 49152 x 896 59 | 36, 128 x 49152 x 2048 102 | 89, 64 x 151936 x 896 127 | 123, of 80 M: 64 x 151936 x 1536
    // 188 | 175, of 0.5 M: 40 x 49152 x 896 46 | 31, 64 x 151936 x 1536 152 | 142; it loses where one row tile is half padding
    // and the lists are long: 96 x 151936 x 1536 180 | 200 at 32 M, 156 | 147 at 0.5 M).  Up to 32 rows its tiles are mostly
    // padding (25 x 49152 x 896 106 | 108, 25 x 151936 x 896 165 | 169).
    const bool large = EPI == TEPI_LMHEAD ? M > 32 && small_wgs > cus : (M >= kLargeTileRows && large_wgs >= 128) || (M > 128 && large_wgs >= 512);
    if (large) {
        // Tiles of 192 rows where their rounds over the compute units are shorter in all (the tile shape never changes a row's result):
        // fewer padded rows (576 = 3 x 192), a last round that larger tiles would leave half empty, or idle units in the only one.
        // They read the weights more often, so they have to win by a twelfth.  165 products of 384 to 8192 rows, all epilogues,
        // by the rounds of 192 / 256 rows: as many of both 1.06 to 1.34 times as fast (us, 256 | 192: down 6336 x 1536 x 8960 187 | 174; 3072 x 2048 x
        // 11008 in four slices 121 | 100), 6 / 5 1.11 times (gate and up 3072 x 22016 x 2048 223 | 201), but 5 / 4 between 0.92 (6336 x 2048 x
        // 11008 in four slices 270 | 295) and 1.07.  LM head, 200 and 256 rows x 16640 to 32768, 480 to 700 rows x 12288 to 20480: 1.01
        // to 1.12 times (200 x 16640 x 1536 53.8 | 48.8, 256 x 32768 x 2048 73.6 | 72.2).
        const int mt256 = (M + 255) / 256, mt192 = (M + 191) / 192;
        const int nt = (N + 255) / 256;
        auto rounds = [&](int mt) { return ((long)mt * nt * slices + cus - 1) / cus; };
        const bool mid = rounds(mt192) * 192 * 12 < rounds(mt256) * 256 * 11;
        if (mid) {
            if constexpr (EPI != TEPI_LMHEAD) {
                // (the other kernel's rotation needs whole heads in a wave's features: 128, not 64)
                if (EPI == TEPI_ROPE || ((long)mt192 * nt * slices <= cus && M <= kFewRows)) {
                    k_gemm_tiled<EPI, TILE_MID><<<dim3((unsigned)(mt192 * nt), (unsigned)slices), dim3(512), TG_LDS_BYTES(256, 192), st>>>(
                        A, (const BF16*)Wm, M, N, K, outf, outb, lm, rp);
                    return;
                }
            }
            if constexpr (EPI != TEPI_ROPE) {
                k_gemm<EPI, GEMM_MID><<<dim3((unsigned)cus), dim3(512), gemm_lds_bytes(GEMM_MID), st>>>(A, (const BF16*)Wm, M, N, K, slices, outf, outb, lm, rp);
                return;
            }
        }
        with_head_dim<EPI>(rp.gm.hd, [&](auto h) {
            constexpr auto k = gemm_large<EPI, decltype(h)::value>();
            k.first<<<dim3((unsigned)cus), dim3(512), k.second, st>>>(A, (const BF16*)Wm, M, N, K, slices, outf, outb, lm, rp);
        });
        return;
    }
    if constexpr (EPI == TEPI_LMHEAD) {
        dim3 g((unsigned)(((M + 127) / 128) * ((N + 127) / 128)), 1);
        k_gemm_tiled<EPI, TILE_SMALL><<<g, dim3(256), TG_LDS_BYTES(128, 128), st>>>(A, (const BF16*)Wm, M, N, K, outf, outb, lm, rp);
    } else {
        // (the rotation epilogue needs whole heads inside a tile)
        if (small_wgs <= 128 && !(EPI == TEPI_ROPE && rp.gm.hd > 64)) {         // half of the compute units idle: halve the tile's width (a workgroup each, still)
            dim3 g((unsigned)(((M + 127) / 128) * ((N + 63) / 64)), (unsigned)slices);
            k_gemm_tiled<EPI, TILE_NARROW><<<g, dim3(256), TG_LDS_BYTES(64, 128), st>>>(A, (const BF16*)Wm, M, N, K, outf, outb, lm, rp);
            return;
        }
        if constexpr (small_in_registers(EPI)) {
            if (small_wgs <= cus) {
                const dim3 g((unsigned)(((M + 127) / 128) * ((N + 127) / 128)), (unsigned)slices);
                k_gemm_tiled<EPI, TILE_SMALL><<<g, dim3(256), TG_LDS_BYTES(128, 128), st>>>(A, (const BF16*)Wm, M, N, K, outf, outb, lm, rp);
                return;
            }
        }
        with_head_dim<EPI>(rp.gm.hd, [&](auto h) {
            constexpr auto k = gemm_small<EPI, decltype(h)::value>();
            const dim3 grid((unsigned)std::min<long>(small_wgs, cus)), threads(EPI == TEPI_ROPE ? 256 : 512);
            k.first<<<grid, threads, k.second, st>>>(A, (const BF16*)Wm, M, N, K, slices, outf, outb, lm, rp);
        });
    }
}

// one-off set-up of the tiled kernels; *cus = the device's compute units
tasc_status tiled_ready(int* cus) {
    std::lock_guard<std::mutex> lock(g_dev_mu);
    DevState& ds = dev_state();
    if (ds.cu_count == 0) {
        int dev = 0;
        TASC_HIP(hipGetDevice(&dev));
        TASC_HIP(hipDeviceGetAttribute(&ds.cu_count, hipDeviceAttributeMultiprocessorCount, dev));
    }
    *cus = ds.cu_count;
    if (ds.tiled_ready) return TASC_OK;
    tasc_status rc;
    if ((rc = tiled_attrs<TEPI_STORE>()) != TASC_OK) return rc;
    if ((rc = tiled_attrs<TEPI_RESID>()) != TASC_OK) return rc;
    if ((rc = tiled_attrs<TEPI_SWIGLU>()) != TASC_OK) return rc;
    if ((rc = tiled_attrs<TEPI_LMHEAD>()) != TASC_OK) return rc;
    if ((rc = tiled_attrs<TEPI_PARTIAL>()) != TASC_OK) return rc;
    if ((rc = tiled_attrs<TEPI_ROPE>()) != TASC_OK) return rc;
    TASC_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(k_attn_staged<2>), hipFuncAttributeMaxDynamicSharedMemorySize, TA_LDS_BYTES(64) + 4 * TA_MAX_BLOCKS));
    TASC_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(k_attn_staged<4>), hipFuncAttributeMaxDynamicSharedMemorySize, TA_LDS_BYTES(128) + 4 * TA_MAX_BLOCKS));
    TASC_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(k_attn_prompt<2>), hipFuncAttributeMaxDynamicSharedMemorySize, TA_LDS_BYTES(64) + 4 * TA_MAX_BLOCKS));
    TASC_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(k_attn_prompt<4>), hipFuncAttributeMaxDynamicSharedMemorySize, TA_LDS_BYTES(128) + 4 * TA_MAX_BLOCKS));
    ds.tiled_ready = true;
    return TASC_OK;
}


// how many ranges of sequences run the layers side by side when the caller leaves the choice to the library
int tiled_auto_chains(const tasc_model_desc& c, int batch, int nq) {
    (void)c; (void)batch; (void)nq;
    return 1;
}

tasc_status forward_tiled(const tasc_model* m, tasc_session* s, int nq, int M_all, int n_sel, float* logits_dbg, const TascVerifyTail* tail, hipStream_t st) {
    const bool decode = tail != nullptr;
    const tasc_model_desc& c = m->desc;
    const TascSessDev& d = s->d;
    int cus = 0;
    {
        const tasc_status rc = tiled_ready(&cus);
        if (rc != TASC_OK) return rc;
    }
    const int D = c.d_model, H = c.n_heads, Hkv = c.n_kv_heads, hd = c.head_dim, F = c.d_ffn;
    const int nqkv = (H + 2 * Hkv) * hd, nqo = H * hd;
    LmEpi none{};
    // Narrow outputs (few column tiles) are computed in k-slices.  The slice count fixes the order in which a row's
    // products are added, so it must be the same for every DECODE forward of a session (a greedy step and a verify step
    // of one session differ in their row count, and speculative decoding must reproduce greedy decoding bit for bit): it
    // depends on N, K and the session's batch only, never on the rows of the call; rows_ref = 5 rows per sequence
    // stands for the verify steps the session is sized for.  A prompt forward is the same computation in the
    // speculative and in the greedy run whatever its slice count, so it takes the count that suits the many rows of its
    // chunks (they fill the chip without slices, and every slice is a pass over rows x N partial sums) -- but not the rows this
    // call happens to have, which are the other prompts' as well: prompt_ref, a session constant.
    const int rows_ref = decode ? s->batch * 5 : s->prompt_ref;
    auto slices = [&](int N, int K) {
        const int n_nt = (N + 127) / 128, nk = K / TG_BK;
        if (n_nt >= 32) return 1;
        // many sequences, short k: the small tiles of one slice already fill the chip, and every slice would cost a
        // pass over rows x N partial sums
        if (nk <= 40 && n_nt * ((rows_ref + 127) / 128) >= 128) return 1;
        int ks;
        if (rows_ref >= kLargeTileRows && nk > 40) {
            // long k on large tiles: as many slices as fit the compute units in one round
            const int tiles = ((rows_ref + 255) / 256) * ((N + 255) / 256);
            ks = 256 / tiles;
        } else {
            // few rows: one slice per 12 k-steps, or enough for about 24 (column tile, slice) pairs if that is more
            // (measured on the qkv / output / down projections of the 0.5B and 1.5B shapes)
            ks = nk / 12 > (24 + n_nt - 1) / n_nt ? nk / 12 : (24 + n_nt - 1) / n_nt;
        }
        // beyond two 128-row tiles every slice's pass over rows x N partial sums costs more than the shorter k loop
        // gains (the 1.5B shape's down projection in the step: 4 slices 4.40 ms per verify step, 8 slices 4.52 ms)
        if (rows_ref > 256 && rows_ref < kLargeTileRows && ks > 4) ks = 4;
        ks = ks < nk / 4 ? ks : nk / 4;                       // slices of at least 4 k-steps
        ks = ks < TG_MAX_SLICES ? ks : TG_MAX_SLICES;
        if (!decode && ks > s->prompt_slices) ks = s->prompt_slices;
        if (ks < 1) return 1;
        // no empty slice at the end: fewer of the same length (k_gemm has no stage to begin with in one)
        return (nk + (nk + ks - 1) / ks - 1) / ((nk + ks - 1) / ks);
    };
    // Key chunks of the attention: two workgroups per compute unit in one round, but no more than 4 partial results to merge.
    // A session constant, since it fixes the order in which a row's keys are added; the one for prompts counts the row passes of
    // prompt_ref rows too, so that long chunks need no merge.
    const int att_passes = decode ? 1 : (s->prompt_ref / s->batch * (H / Hkv) + 63) / 64;
    int att_chunks = 512 / (s->batch * Hkv * att_passes);
    att_chunks = att_chunks < 1 ? 1 : (att_chunks > 4 ? 4 : att_chunks);
    // Prompt chunks that need no key chunks go 128 (row, head) pairs a workgroup where that is a workgroup per compute unit; a session
    // constant as well (the two kernels' sums are not the same bits).  2 layers of the 0.5B, 1.5B and 3B shapes, 64 | 128 pairs: from 256
    // workgroups on 0.99 to 1.32 times as fast (1 prompt of 8192: 1479 | 1119, 2610 | 2141, 3667 | 3085 us; 32 of 64: 320 | 321, 531 | 534,
    // 798 | 793), with 146 to 224 of them 0.98 to 1.02 times (4 of 512: 354 | 354, 558 | 564, 811 | 825; 1 of 2048: 423 | 414, 725 | 712, 955 | 932).
    const int prompt_passes = (s->prompt_ref / s->batch * (H / Hkv) + TAP_ROWS - 1) / TAP_ROWS;
    const bool prompt_attn = !decode && att_chunks == 1 && s->batch * Hkv * prompt_passes >= cus;
    const BiasCursors bc{BiasCsr{m->bias_rowptr, m->bias_col, m->bias_val, m->bias_base}, d.sel_tok,
                         m->bias_rowptr ? n_sel * (s->n_strips + 1) : 0, s->n_strips, d.bias_ptr, d.bias_first, d.bias_base};
    const unsigned bias_wgs = (unsigned)((bc.n + 255) / 256);
    {
        PROF(TASC_KC_PREPARE);
        if (D <= RRN_MAX_D) {
            k_embed_norm<<<dim3(M_all + bias_wgs), dim3(256), 0, st>>>((const BF16*)m->embed, d.row_tok, m->layers[0].g1, M_all, D, c.rms_eps,
                                                                      d.x, (BF16*)d.h, bc, step_rows(m, s, tail));
        } else {
            const tasc_status rc = prepare_verify(m, s, tail, st);
            if (rc != TASC_OK) return rc;
            k_embed<BF16><<<dim3(M_all), dim3(64), 0, st>>>((const BF16*)m->embed, d.row_tok, D, d.x, StepRows{});
            if (bias_wgs) k_bias_ptr<<<dim3(bias_wgs), dim3(256), 0, st>>>(bc);
        }
    }
    TASC_LAUNCH_CHECK();
    // A verify step's LM-head rows are its rows, so the last layer's reduction can normalise them as well.  (Of a decode forward
    // only, and whether it does depends on the slices alone: a row's bits are the same in steps of any row count.)
    const bool all_rows = decode && n_sel == M_all;
    bool final_normed = false;

    // The layers of sequences [b0, b0 + nb) on stream `st`: every kernel below computes a row from that row's own data
    // (and its sequence's cache), in an order fixed by the session, so the layers may run for several ranges of
    // sequences side by side ("chains", each on a stream of its own with its own share of every buffer) without
    // changing a bit of any row.
    auto run_layers = [&](int b0, int nb, hipStream_t st) -> tasc_status {
        const int M = nb == s->batch ? M_all : nb * nq;          // (ranges of sequences only where all have nq rows)
        const size_t r0 = (size_t)b0 * nq;
        const KvGeom gm{H, Hkv, hd, s->max_blocks, s->page_elems, d.row_seq + r0, d.row0, (int32_t)r0};
        float* const x = d.x + r0 * D;
        BF16* const h = (BF16*)d.h + r0 * D;
        BF16* const q = (BF16*)d.q + r0 * nqo;
        BF16* const att = (BF16*)d.att + r0 * nqo;
        BF16* const act = (BF16*)d.act + r0 * F;
        float* const part = d.att_part + r0 * 8 * (size_t)(nqkv > D ? nqkv : D);   // (r0 > 0 only among the batch x max_rows rows the scratch has 8 slices for)
        const int32_t* const n_rows = d.n_rows;
        const int32_t* const pos0 = d.pos0;
        const int32_t* const block_tab = d.block_tab;
        // out (+)= A W^T through k-slices and the ordered reduction.  With `norm_g` the RMSNorm of the updated rows (gain
        // norm_g, into h) is fused into the reduction; returns false if the caller still has to run it (no slices).
        auto gemm_sliced = [&](const BF16* A, const void* Wm, int N, int K, float* out, bool resid, const float* norm_g) {
            const int ks = slices(N, K);
            if (ks == 1) {
                if (resid) launch_gemm<TEPI_RESID>(A, Wm, M, N, K, out, nullptr, none, 1, st, cus);
                else launch_gemm<TEPI_STORE>(A, Wm, M, N, K, out, nullptr, none, 1, st, cus);
                return false;
            }
            launch_gemm<TEPI_PARTIAL>(A, Wm, M, N, K, part, nullptr, none, ks, st, cus);
            const size_t mn = (size_t)M * N;
            if (resid && norm_g && N == D && D <= RRN_MAX_D) {
                bool fused = true;
                switch (ks) {
#define RRN_CASE(NS) case NS: k_reduce_resid_norm<NS><<<dim3(M), dim3(256), 0, st>>>(part, mn, out, norm_g, D, c.rms_eps, h); break;
                    RRN_CASE(2) RRN_CASE(3) RRN_CASE(4) RRN_CASE(5) RRN_CASE(6) RRN_CASE(7) RRN_CASE(8)
#undef RRN_CASE
                    default: fused = false;
                }
                if (fused) return true;
            }
            const unsigned blocks = (unsigned)((mn / 4 + 255) / 256);
            if (resid) k_splitk_reduce<true><<<dim3(blocks), dim3(256), 0, st>>>(part, ks, mn, out);
            else k_splitk_reduce<false><<<dim3(blocks), dim3(256), 0, st>>>(part, ks, mn, out);
            return false;
        };
        const int rows_pass = 32;
        const dim3 attn_grid(nb * Hkv, (nq * (H / Hkv) + rows_pass - 1) / rows_pass);
        bool h_ready = D <= RRN_MAX_D;        // h already holds the layer's normalised input
        for (int l = 0; l < c.n_layers; ++l) {
            const TascLayerW& w = m->layers[l];
            BF16* kv_layer = (BF16*)s->kv_pool + (size_t)l * s->kv_layer_stride;
            if (!h_ready) {
                PROF(TASC_KC_NORM);
                if (D <= RRN_MAX_D) k_rmsnorm_row<<<dim3(M), dim3(256), 0, st>>>(x, w.g1, D, c.rms_eps, h);
                else k_rmsnorm<BF16><<<dim3(M), dim3(64), 0, st>>>(x, w.g1, nullptr, D, c.rms_eps, h);
            }
            const int ks_qkv = slices(nqkv, D);
            {
                // one slice: rotation and cache append ride in the projection's epilogue
                PROF(TASC_KC_GEMM_QKV);
                if (ks_qkv == 1)
                    launch_gemm<TEPI_ROPE>(h, w.wqkv, M, nqkv, D, nullptr, q, none, 1, st, cus,
                                           RopeEpi{m->rope_cos, m->rope_sin, n_rows, pos0, block_tab, kv_layer, gm, c.max_pos});
                else launch_gemm<TEPI_PARTIAL>(h, w.wqkv, M, nqkv, D, part, nullptr, none, ks_qkv, st, cus);
            }
            if (ks_qkv > 1) {
                // the k-slices of a split projection are added inside the rotation kernel (same order as the reduction kernel)
                PROF(TASC_KC_ROPE_KV);
                switch (ks_qkv) {
#define ROPE_CASE(NS) case NS: k_rope_kv<NS><<<dim3(M), dim3(256), 0, st>>>(part, m->rope_cos, m->rope_sin, c.max_pos, n_rows, pos0, block_tab, gm, \
                                                                          decode ? nq : 0, q, kv_layer, (size_t)M * nqkv); break;
                    ROPE_CASE(2) ROPE_CASE(3) ROPE_CASE(4) ROPE_CASE(5) ROPE_CASE(6) ROPE_CASE(7)
                    default: ROPE_CASE(8)
#undef ROPE_CASE
                }
            }
            {
                PROF(TASC_KC_ATTN);
                AttnArgs aa{q, att, kv_layer, n_rows, pos0, block_tab, d.row0, b0, (int32_t)r0, M, nq, H, Hkv,
                            s->max_blocks, decode ? 1 : 0, s->page_elems, 1.0f / sqrtf((float)hd)};
                if (hd == 32 || s->max_blocks > TA_MAX_BLOCKS) {
                    if (hd == 64) k_attn_tiled<2><<<attn_grid, dim3(SMALL_THREADS), 0, st>>>(aa);
                    else if (hd == 128) k_attn_tiled<4><<<attn_grid, dim3(SMALL_THREADS), 0, st>>>(aa);
                    else k_attn_tiled<1><<<attn_grid, dim3(SMALL_THREADS), 0, st>>>(aa);
                } else if (prompt_attn) {
                    const dim3 grid(nb * Hkv, (nq * (H / Hkv) + TAP_ROWS - 1) / TAP_ROWS);
                    if (hd == 64) k_attn_prompt<2><<<grid, dim3(TAP_THREADS), TA_LDS_BYTES(64) + 4 * s->max_blocks, st>>>(aa);
                    else k_attn_prompt<4><<<grid, dim3(TAP_THREADS), TA_LDS_BYTES(128) + 4 * s->max_blocks, st>>>(aa);
                } else {
                    // keys and values staged in LDS, 64 rows per pass; the key tiles are dealt to att_chunks workgroups, a
                    // number fixed by the session's batch (it sets the order in which a row's keys are added)
                    const size_t rows_all = (size_t)M;
                    AttnStagedArgs sa{aa, part, part + (size_t)att_chunks * rows_all * H * hd, att_chunks};
                    const dim3 grid(nb * Hkv, (nq * (H / Hkv) + 63) / 64, att_chunks);
                    if (hd == 64) k_attn_staged<2><<<grid, dim3(SMALL_THREADS), TA_LDS_BYTES(64) + 4 * s->max_blocks, st>>>(sa);
                    else k_attn_staged<4><<<grid, dim3(SMALL_THREADS), TA_LDS_BYTES(128) + 4 * s->max_blocks, st>>>(sa);
                    if (att_chunks > 1) {
                        const size_t n = rows_all * H * hd / 4;
                        const dim3 mg((unsigned)((n + 255) / 256));
                        if (att_chunks == 2) k_attn_merge<2><<<mg, dim3(256), 0, st>>>(sa.part_o, sa.part_ml, rows_all, H, hd, att);
                        else if (att_chunks == 3) k_attn_merge<3><<<mg, dim3(256), 0, st>>>(sa.part_o, sa.part_ml, rows_all, H, hd, att);
                        else k_attn_merge<4><<<mg, dim3(256), 0, st>>>(sa.part_o, sa.part_ml, rows_all, H, hd, att);
                    }
                }
            }
            bool normed;
            {
                PROF(TASC_KC_GEMM_O);
                normed = gemm_sliced(att, w.wo, D, nqo, x, true, w.g2);
            }
            if (!normed) {
                PROF(TASC_KC_NORM);
                if (D <= RRN_MAX_D) k_rmsnorm_row<<<dim3(M), dim3(256), 0, st>>>(x, w.g2, D, c.rms_eps, h);
                else k_rmsnorm<BF16><<<dim3(M), dim3(64), 0, st>>>(x, w.g2, nullptr, D, c.rms_eps, h);
            }
            {
                PROF(TASC_KC_GEMM_GU);
                launch_gemm<TEPI_SWIGLU>(h, w.wgu, M, 2 * F, D, nullptr, act, none, 1, st, cus);
            }
            {
                // the next layer's first RMSNorm rides on this reduction
                PROF(TASC_KC_GEMM_D);
                h_ready = gemm_sliced(act, w.wd, D, F, x, true, l + 1 < c.n_layers ? m->layers[l + 1].g1 : all_rows ? m->gf : nullptr);
            }
            TASC_LAUNCH_CHECK();
        }
        final_normed = h_ready;
        return TASC_OK;
    };

    // chains: few rows leave the layer kernels short of workgroups and bound by their own start-up and dependent
    // memory round trips; ranges of sequences that run side by side fill the compute units.  Each reads the weights
    // again (from the caches when the chains keep pace), so the count stays small.
    // (Not for prompt chunks of more than batch x max_rows rows: a chain's share of the partial sums below is 8 slices of its
    // rows, and beyond batch x max_rows the scratch may hold 4.)
    const int chains = M_all == s->batch * nq && nq <= s->max_rows ? tasc_forward_chains(m, s, nq) : 1;
    if (chains <= 1) {
        const tasc_status rc = run_layers(0, s->batch, st);
        if (rc != TASC_OK) return rc;
    } else {
        TASC_HIP(hipEventRecord(s->chain_fork, st));
        for (int ch = 0; ch < chains; ++ch) {
            const int b0 = (int)((long)s->batch * ch / chains), b1 = (int)((long)s->batch * (ch + 1) / chains);
            hipStream_t cs = ch == 0 ? st : s->chain_st[ch - 1];
            if (ch > 0) TASC_HIP(hipStreamWaitEvent(cs, s->chain_fork, 0));
            const tasc_status rc = run_layers(b0, b1 - b0, cs);
            if (rc != TASC_OK) return rc;
            if (ch > 0) {
                TASC_HIP(hipEventRecord(s->chain_join[ch - 1], cs));
                TASC_HIP(hipStreamWaitEvent(st, s->chain_join[ch - 1], 0));
            }
        }
    }
    if (n_sel > 0) {
        if (!final_normed) {
            PROF(TASC_KC_NORM);
            k_rmsnorm<BF16><<<dim3(n_sel), dim3(64), 0, st>>>(d.x, m->gf, d.sel_rows, D, c.rms_eps, (BF16*)d.h);
        }
        LmEpi lm{bc.bias, d.bias_ptr, d.bias_first, d.bias_base, d.part_val, d.part_idx, logits_dbg, s->n_strips};
        {
            PROF(TASC_KC_LMHEAD);
            launch_gemm<TEPI_LMHEAD>((const BF16*)d.h, m->lm_head, n_sel, c.vocab, D, nullptr, nullptr, lm, 1, st, cus);
        }
        TASC_LAUNCH_CHECK();
        return finish_rows(s, n_sel, s->n_strips, d.part_val, d.part_idx, tail, st);
    }
    return TASC_OK;
}

// the fused small-batch kernel serves a bf16 forward of at most 16 rows with these shapes
bool small_path_fits(const tasc_model* m, int batch, int nq, int max_blocks) {
    const tasc_model_desc& c = m->desc;
    return m->lm_head_f != nullptr && c.dtype == TASC_BF16 && batch * nq <= SMALL_ROWS && c.n_layers <= SMALL_MAX_LAYERS && batch * max_blocks <= SMALL_MAX_BT && c.d_model <= SMALL_KC && c.d_model % 32 == 0 &&
           (c.head_dim == 32 || c.head_dim == 64 || c.head_dim == 128) && c.d_ffn % 32 == 0 && c.vocab >= 16 &&
           (nq * (c.n_heads / c.n_kv_heads)) >= 1;
}


tasc_status forward_small(const tasc_model* m, tasc_session* s, int nq, int n_sel, float* logits_dbg, const TascVerifyTail* tail,
                          hipStream_t st) {
    const tasc_model_desc& c = m->desc;
    const TascSessDev& d = s->d;
    tasc_status prc = prepare_verify(m, s, tail, st);
    if (prc != TASC_OK) return prc;
    DevState& ds = dev_state();
    if (std::lock_guard<std::mutex> lock(g_dev_mu); !ds.small_ready) {
        int dev = 0, cus = 0;
        TASC_HIP(hipGetDevice(&dev));
        TASC_HIP(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev));
        int per_cu = 0;
        TASC_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(k_small_step<1>), hipFuncAttributeMaxDynamicSharedMemorySize,
                                     SMALL_LDS_BYTES));
        TASC_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(k_small_step<2>), hipFuncAttributeMaxDynamicSharedMemorySize,
                                     SMALL_LDS_BYTES));
        TASC_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(k_small_step<4>), hipFuncAttributeMaxDynamicSharedMemorySize,
                                     SMALL_LDS_BYTES));
        TASC_HIP(hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, k_small_step<4>, SMALL_THREADS, SMALL_LDS_BYTES));
        if (cus < 1 || per_cu < 1) {
            tasc_set_error("forward: the persistent kernel does not fit the device (%d compute units, %d blocks each)", cus, per_cu);
            return TASC_EHIP;
        }
        ds.cu_count = cus;
        ds.small_ready = true;
    }
    SmallArgs a;
    a.layers = m->d_layers;
    a.embed = (const BF16*)m->embed;
    a.lm_head = (const BF16*)m->lm_head_f;
    a.gf = m->gf;
    a.rope_cos = m->rope_cos;
    a.rope_sin = m->rope_sin;
    a.bias = BiasCsr{m->bias_rowptr, m->bias_col, m->bias_val, m->bias_base};
    a.n_layers = c.n_layers; a.D = c.d_model; a.H = c.n_heads; a.Hkv = c.n_kv_heads; a.hd = c.head_dim; a.F = c.d_ffn;
    a.V = c.vocab; a.max_pos = c.max_pos; a.eps = c.rms_eps; a.scale = 1.0f / sqrtf((float)c.head_dim);
    a.kv_pool = (BF16*)s->kv_pool; a.kv_layer_stride = s->kv_layer_stride; a.page_elems = s->page_elems;
    a.B = s->batch; a.nq = nq; a.M = s->batch * nq; a.max_blocks = s->max_blocks; a.max_len = s->max_len;
    a.n_strips = s->n_strips; a.max_new = s->max_new;
    a.row_tok = d.row_tok; a.n_rows = d.n_rows; a.pos0 = d.pos0; a.block_tab = d.block_tab; a.sel_rows = d.sel_rows;
    a.sel_tok = d.sel_tok; a.n_sel = n_sel;
    {
        const TascSmallWs w = tasc_small_ws_layout(c);
        a.x = (float*)(d.small_ws + w.x_off); a.x_stride = w.x_stride;
        a.q = (BF16*)(d.small_ws + w.q_off); a.att = (BF16*)(d.small_ws + w.att_off); a.q_stride = w.q_stride;
        a.act = (BF16*)(d.small_ws + w.act_off); a.act_stride = w.act_stride;
    }
    a.part_val = d.part_val; a.part_idx = d.part_idx; a.amax = d.amax; a.logits_dbg = logits_dbg;
    a.k = tail ? tail->k : -1;
    a.drafts = tail ? tail->drafts : nullptr;
    a.tokens = d.tokens; a.n_tok = d.n_tok; a.cached = d.cached; a.n_emit = d.n_emit; a.counters = d.counters;
    a.accept_len = tail ? tail->accept_len : nullptr;
    a.emitted = tail ? tail->emitted : nullptr;
    a.trace_step = tail ? tail->trace_step : nullptr;
    a.bar_flags = (u32*)&d.counters[TASC_CTR_FLAGS];
    a.barb_counter = &d.counters[TASC_CTR_BARB];
    a.bar_error = (u32*)&d.counters[TASC_CTR_BAR_ERR];
    a.xcc_mask = (u32*)&d.counters[TASC_CTR_XCC];
    a.xcd_local = g_tasc_config.xcd_local;
    a.bias_ptr = d.bias_ptr;
    const int n_phases = 3 + 5 * c.n_layers, n_lg_phases = 1 + 5 * c.n_layers;
    a.phase_ts = g_phase_ts;
    a.phase_ts_wgs = g_phase_ts ? (int32_t)(g_phase_ts_cap / (2 * (int64_t)n_phases)) : 0;
    const int last = n_sel > 0 ? n_phases : n_lg_phases;   // without LM-head rows the step ends after the last layer
    int grid = g_tasc_config.small_grid > 0 ? g_tasc_config.small_grid : ds.cu_count;
    grid = grid < ds.cu_count ? grid : ds.cu_count;            // every workgroup must be resident: at most one per compute unit
    // Layer group.  The dispatcher deals workgroup ids round-robin over the 8 XCDs, so by default the group is
    // every 8th workgroup, 32 of them: one XCD's worth, which lets the 150 latency-bound layer phases hand
    // their activations over through that XCD's L2 (the kernel checks where it really runs and falls back
    // to agent-scope barriers otherwise).  With XCD-local barriers off, or a grid too small for that, the
    // group is the first 48 workgroups, spread over all XCDs.  The LM head always uses the whole grid.
    const bool one_xcd = g_tasc_config.xcd_local != 0 && g_tasc_config.small_path == 2 && grid >= 8 * 32;
    int stride = g_tasc_config.layer_stride > 0 ? g_tasc_config.layer_stride : (one_xcd ? 8 : 1);
    int lg = g_tasc_config.layer_wgs > 0 ? g_tasc_config.layer_wgs : (one_xcd && g_tasc_config.layer_stride <= 0 ? 32 : 48);
    if (stride > grid) stride = grid;
    if (lg > (grid + stride - 1) / stride) lg = (grid + stride - 1) / stride;
    if (lg > SMALL_MAX_GROUP) lg = SMALL_MAX_GROUP;
    a.lg_stride = stride;
    a.lg_count = lg;
    a.lg_workers = g_tasc_config.layer_workers > 0 ? g_tasc_config.layer_workers : lg;
    a.bar_epoch = s->bar_epoch;
    a.barb_base = s->barb_base;
    s->ll_armed = false;       // this kernel writes the first copy of the buffers the pipeline kernel expects untouched
    PROF(TASC_KC_LAYERS);
    auto launch = [&](int p0, int p1) {
        if (c.head_dim == 32) k_small_step<1><<<dim3(grid), dim3(SMALL_THREADS), SMALL_LDS_BYTES, st>>>(a, p0, p1);
        else if (c.head_dim == 64) k_small_step<2><<<dim3(grid), dim3(SMALL_THREADS), SMALL_LDS_BYTES, st>>>(a, p0, p1);
        else k_small_step<4><<<dim3(grid), dim3(SMALL_THREADS), SMALL_LDS_BYTES, st>>>(a, p0, p1);
    };
    if (g_tasc_config.small_path == 2) {
        launch(0, last);
        s->bar_epoch += (u32)(n_lg_phases - 1);
        s->barb_base += (u64)(last - n_lg_phases) * grid;
    } else {
        for (int ph = 0; ph < last; ++ph) {
            // a launch of one phase crosses no barrier
            launch(ph, ph + 1);
        }
    }
    TASC_LAUNCH_CHECK();
    return TASC_OK;
}

// ---------------------------------------------------------------- the spatial-pipeline kernel
__global__ void k_fill_sentinel(u64* p, size_t units16) {
    for (size_t u = (size_t)blockIdx.x * blockDim.x + threadIdx.x; u < units16; u += (size_t)gridDim.x * blockDim.x) {
        p[2 * u] = ~0ull;
        p[2 * u + 1] = ~0ull;
    }
}

// Deals the workgroups of the grid to the five roles: every role gets enough of them that a workgroup's share of the
// role's items (16-feature tiles, or (sequence, head) pairs) stays within what one pass holds in registers.  Returns
// false if the grid is too small for the model.
bool pipe_roles(const tasc_model_desc& c, int batch, int grid, int32_t (&base)[PIPE_N_ROLES], int32_t (&count)[PIPE_N_ROLES]) {
    const bool wide = c.d_model > 768;                     // 6 fragments per tile row and lane: one item per pass
    const int items[PIPE_N_ROLES] = {(c.n_heads + 2 * c.n_kv_heads) * (c.head_dim / 32), batch * c.n_heads, c.d_model / 16,
                                     c.d_ffn / 16, c.d_model / 16};
    const int max_share[PIPE_N_ROLES] = {wide ? 1 : 3, 1 << 20, 3, wide ? 1 : 3, 3};
    int share[PIPE_N_ROLES] = {1, 1, 1, 1, 1};
    for (int r = 0; r < PIPE_N_ROLES; ++r)
        if (r != PIPE_ATTN) share[r] = g_tasc_config.pipe_share > max_share[r] ? max_share[r] : (g_tasc_config.pipe_share < 1 ? 1 : g_tasc_config.pipe_share);
    auto wgs = [&](int r) { return (items[r] + share[r] - 1) / share[r]; };
    share[PIPE_ATTN] = (items[PIPE_ATTN] + 15) / 16;       // at most 16 workgroups on attention
    for (;;) {
        int total = 0;
        for (int r = 0; r < PIPE_N_ROLES; ++r) total += wgs(r);
        if (total <= grid) break;
        int pick = -1;
        for (int r = 0; r < PIPE_N_ROLES; ++r)
            if (share[r] < max_share[r] && (pick < 0 || wgs(r) > wgs(pick))) pick = r;
        if (pick < 0) return false;
        ++share[pick];
    }
    int at = 0;
    for (int r = 0; r < PIPE_N_ROLES; ++r) {
        base[r] = at;
        count[r] = wgs(r);
        at += count[r];
    }
    return true;
}

bool pipe_path_fits(const tasc_model* m, int batch, int nq, int max_blocks, int grid) {
    const tasc_model_desc& c = m->desc;
    int32_t b[PIPE_N_ROLES], n[PIPE_N_ROLES];
    return c.d_model % 64 == 0 && grid >= 8 && pipe_roles(c, batch, grid, b, n);
}

template <int NKS, int WKS>
tasc_status pipe_attr() {
    TASC_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(k_pipe_step<NKS, WKS>), hipFuncAttributeMaxDynamicSharedMemorySize,
                                 PIPE_LDS_BYTES));
    return TASC_OK;
}

tasc_status forward_pipe(const tasc_model* m, tasc_session* s, int nq, int n_sel, float* logits_dbg, const TascVerifyTail* tail, int grid,
                         hipStream_t st) {
    const tasc_model_desc& c = m->desc;
    const TascSessDev& d = s->d;
    tasc_status prc = prepare_verify(m, s, tail, st);
    if (prc != TASC_OK) return prc;
    if (std::lock_guard<std::mutex> lock(g_dev_mu); !dev_state().pipe_ready) {
        tasc_status rc;
        if ((rc = pipe_attr<1, 3>()) != TASC_OK || (rc = pipe_attr<2, 3>()) != TASC_OK || (rc = pipe_attr<4, 3>()) != TASC_OK ||
            (rc = pipe_attr<1, 6>()) != TASC_OK || (rc = pipe_attr<2, 6>()) != TASC_OK || (rc = pipe_attr<4, 6>()) != TASC_OK)
            return rc;
        dev_state().pipe_ready = true;
    }
    if (!s->ll_armed) {
        tasc_status rc = tasc_pipe_arm(s, st);
        if (rc != TASC_OK) return rc;
    }
    const TascSmallWs w = tasc_small_ws_layout(c);
    char* cur = d.small_ws + (size_t)s->ll_copy * w.bytes;
    char* other = d.small_ws + (size_t)(1 - s->ll_copy) * w.bytes;
    PipeArgs pa;
    SmallArgs& a = pa.a;
    a.layers = m->d_layers;
    a.embed = (const BF16*)m->embed;
    a.lm_head = (const BF16*)m->lm_head_f;
    a.gf = m->gf;
    a.rope_cos = m->rope_cos;
    a.rope_sin = m->rope_sin;
    a.bias = BiasCsr{m->bias_rowptr, m->bias_col, m->bias_val, m->bias_base};
    a.n_layers = c.n_layers; a.D = c.d_model; a.H = c.n_heads; a.Hkv = c.n_kv_heads; a.hd = c.head_dim; a.F = c.d_ffn;
    a.V = c.vocab; a.max_pos = c.max_pos; a.eps = c.rms_eps; a.scale = 1.0f / sqrtf((float)c.head_dim);
    a.kv_pool = (BF16*)s->kv_pool; a.kv_layer_stride = s->kv_layer_stride; a.page_elems = s->page_elems;
    a.B = s->batch; a.nq = nq; a.M = s->batch * nq; a.max_blocks = s->max_blocks; a.max_len = s->max_len;
    a.n_strips = s->n_strips; a.max_new = s->max_new;
    a.row_tok = d.row_tok; a.n_rows = d.n_rows; a.pos0 = d.pos0; a.block_tab = d.block_tab; a.sel_rows = d.sel_rows;
    a.sel_tok = d.sel_tok; a.n_sel = n_sel;
    a.x = (float*)(cur + w.x_off); a.x_stride = w.x_stride;
    a.q = (BF16*)(cur + w.q_off); a.att = (BF16*)(cur + w.att_off); a.q_stride = w.q_stride;
    a.act = (BF16*)(cur + w.act_off); a.act_stride = w.act_stride;
    pa.kvn = (BF16*)(cur + w.kvn_off); pa.kvn_stride = w.kvn_stride;
    pa.pv = (float*)(cur + w.pv_off); pa.pi = (int32_t*)(cur + w.pi_off);
    a.part_val = d.part_val; a.part_idx = d.part_idx; a.amax = d.amax; a.logits_dbg = logits_dbg;
    a.k = tail ? tail->k : -1;
    a.drafts = tail ? tail->drafts : nullptr;
    a.tokens = d.tokens; a.n_tok = d.n_tok; a.cached = d.cached; a.n_emit = d.n_emit; a.counters = d.counters;
    a.accept_len = tail ? tail->accept_len : nullptr;
    a.emitted = tail ? tail->emitted : nullptr;
    a.trace_step = tail ? tail->trace_step : nullptr;
    a.bar_flags = (u32*)&d.counters[TASC_CTR_FLAGS];
    a.barb_counter = &d.counters[TASC_CTR_BARB];
    a.bar_error = (u32*)&d.counters[TASC_CTR_BAR_ERR];
    a.xcc_mask = (u32*)&d.counters[TASC_CTR_XCC];
    a.xcd_local = 0;
    a.bias_ptr = d.bias_ptr;
    a.lg_stride = 1; a.lg_count = 0; a.lg_workers = 0; a.bar_epoch = 0; a.barb_base = 0;
    const int n_phases = 3 + 5 * c.n_layers, n_lg_phases = 1 + 5 * c.n_layers;
    a.phase_ts = g_phase_ts;
    a.phase_ts_wgs = g_phase_ts ? (int32_t)(g_phase_ts_cap / (2 * (int64_t)n_phases)) : 0;
    if (!pipe_roles(c, s->batch, grid, pa.role_base, pa.role_count)) {
        tasc_set_error("forward: the pipeline kernel does not fit %d workgroups", grid);
        return TASC_EINVAL;
    }
    const int last = n_sel > 0 ? n_phases : n_lg_phases;
    PROF(TASC_KC_LAYERS);
    auto launch = [&](int p0, int p1) {
        pa.rearm = p0 == 0 ? (u64*)other : nullptr;
        pa.rearm_units = p0 == 0 ? w.bytes / 16 : 0;
        const bool wide = c.d_model > 768;
#define PIPE_LAUNCH(NKS)                                                                                                 \
        if (wide) k_pipe_step<NKS, 6><<<dim3(grid), dim3(SMALL_THREADS), PIPE_LDS_BYTES, st>>>(pa, p0, p1);               \
        else k_pipe_step<NKS, 3><<<dim3(grid), dim3(SMALL_THREADS), PIPE_LDS_BYTES, st>>>(pa, p0, p1)
        if (c.head_dim == 32) { PIPE_LAUNCH(1); }
        else if (c.head_dim == 64) { PIPE_LAUNCH(2); }
        else { PIPE_LAUNCH(4); }
#undef PIPE_LAUNCH
    };
    if (g_tasc_config.small_path == 2) {
        launch(0, last);
    } else {
        for (int ph = 0; ph < last; ++ph) launch(ph, ph + 1);
    }
    TASC_LAUNCH_CHECK();
    s->ll_copy = 1 - s->ll_copy;
    return TASC_OK;
}

}  // namespace

tasc_status tasc_pipe_arm(tasc_session* s, hipStream_t st) {
    const tasc_model_desc& c = s->model->desc;
    if (c.dtype != TASC_BF16) return TASC_OK;
    const size_t units = tasc_small_ws_bytes(c) / 16;
    k_fill_sentinel<<<dim3(1024), dim3(256), 0, st>>>((u64*)s->d.small_ws, units);
    TASC_LAUNCH_CHECK();
    s->ll_armed = true;
    return TASC_OK;
}

extern "C" tasc_status tasc_calibration_gemm(int32_t M, int32_t N, int32_t K, int32_t epilogue, int32_t slices, int32_t iters,
                                             void* stream, double* us_per_launch) {
    TASC_REQUIRE(us_per_launch && M >= 1 && M <= 65536 && N >= 128 && N <= (1 << 20) && N % 128 == 0 && K >= 64 && K <= 65536 && K % 64 == 0,
                 "calibration_gemm: 1 <= M <= 65536, N a multiple of 128 up to 2^20, K a multiple of 64 up to 65536");
    TASC_REQUIRE(epilogue == TEPI_STORE || epilogue == TEPI_RESID || epilogue == TEPI_SWIGLU || epilogue == TEPI_PARTIAL,
                 "calibration_gemm: epilogue %d is none of store (0), residual add (1), SwiGLU (2), k-slice partial sums (4)", epilogue);
    TASC_REQUIRE(slices >= 1 && slices <= TG_MAX_SLICES && (slices == 1 || epilogue == TEPI_PARTIAL) && K / 64 >= slices,
                 "calibration_gemm: 1 .. %d k-slices, more than one only with the partial-sum epilogue", TG_MAX_SLICES);
    TASC_REQUIRE(iters >= 1 && iters <= 10000, "calibration_gemm: 1 .. 10000 launches");
    hipStream_t st = (hipStream_t)stream;
    int cus = 0;
    tasc_status rc = tiled_ready(&cus);
    if (rc != TASC_OK) return rc;
    const size_t a_bytes = (size_t)M * K * 2, w_bytes = (size_t)N * K * 2, o_bytes = (size_t)M * N * 4 * slices;
    struct Tmp { void* p[3] = {nullptr, nullptr, nullptr}; ~Tmp() { for (void* q : p) if (q) (void)hipFree(q); } } t;
    TASC_ALLOC(&t.p[0], a_bytes);
    TASC_ALLOC(&t.p[1], w_bytes);
    TASC_ALLOC(&t.p[2], o_bytes);
    TASC_HIP(hipMemsetAsync(t.p[0], 0x3c, a_bytes, st));       // bf16 0x3c3c = 0.0115: finite sums and SwiGLU arguments
    TASC_HIP(hipMemsetAsync(t.p[1], 0x3c, w_bytes, st));
    TASC_HIP(hipMemsetAsync(t.p[2], 0, o_bytes, st));
    LmEpi none{};
    auto launch = [&]() {
        const BF16* A = (const BF16*)t.p[0];
        if (epilogue == TEPI_STORE) launch_gemm<TEPI_STORE>(A, t.p[1], M, N, K, (float*)t.p[2], nullptr, none, 1, st, cus);
        else if (epilogue == TEPI_RESID) launch_gemm<TEPI_RESID>(A, t.p[1], M, N, K, (float*)t.p[2], nullptr, none, 1, st, cus);
        else if (epilogue == TEPI_SWIGLU) launch_gemm<TEPI_SWIGLU>(A, t.p[1], M, N, K, nullptr, (BF16*)t.p[2], none, 1, st, cus);
        else launch_gemm<TEPI_PARTIAL>(A, t.p[1], M, N, K, (float*)t.p[2], nullptr, none, slices, st, cus);
    };
    struct Ev { hipEvent_t e[2] = {nullptr, nullptr}; ~Ev() { for (hipEvent_t q : e) if (q) (void)hipEventDestroy(q); } } ev;
    TASC_HIP(hipEventCreate(&ev.e[0]));
    TASC_HIP(hipEventCreate(&ev.e[1]));
    for (int i = 0; i < 3; ++i) launch();
    TASC_LAUNCH_CHECK();
    TASC_HIP(hipEventRecord(ev.e[0], st));
    for (int i = 0; i < iters; ++i) launch();
    TASC_HIP(hipEventRecord(ev.e[1], st));
    TASC_LAUNCH_CHECK();
    TASC_HIP(hipEventSynchronize(ev.e[1]));
    float ms = 0.f;
    TASC_HIP(hipEventElapsedTime(&ms, ev.e[0], ev.e[1]));
    *us_per_launch = (double)ms * 1e3 / iters;
    return TASC_OK;
}

int tasc_forward_chains(const tasc_model* m, const tasc_session* s, int32_t nq) {
    int chains = g_tasc_config.chains > 0 ? g_tasc_config.chains : tiled_auto_chains(m->desc, s->batch, nq);
    chains = chains < s->batch ? chains : s->batch;
    chains = chains < TASC_MAX_CHAINS ? chains : TASC_MAX_CHAINS;
    if (tasc_prof_any() || !s->chain_ready) chains = 1;       // the per-class timers bracket launches on one stream
    return chains;
}

bool tasc_forward_is_small(const tasc_model* m, const tasc_session* s, int32_t nq) {
    const int decode_rows = s->max_rows < SMALL_ROWS ? s->max_rows : SMALL_ROWS;
    return g_tasc_config.small_path != 0 && nq <= SMALL_ROWS && small_path_fits(m, s->batch, decode_rows, s->max_blocks);
}

bool tasc_forward_is_tiled(const tasc_model* m, const tasc_session* s, int32_t nq) {
    if (tasc_forward_is_small(m, s, nq)) return false;
    return g_tasc_config.tiled_path != 0 && tasc_tiled_fits(m->desc);
}

tasc_status tasc_forward_rows(const tasc_model* m, tasc_session* s, int32_t nq, int32_t n_rows, int32_t n_sel, float* logits_dbg,
                              const TascVerifyTail* tail, hipStream_t st) {
    // The kernel family of a decode step (nq <= 16 rows per sequence) is a property of the session, not of the
    // call's row count, so that a greedy step and a speculative step of one session use the same kernels and
    // reduce every row in the same order.  Prompt chunks of sessions with max_rows > 16 never
    // take the persistent kernels, however few rows the last one has (the prefill asks for 17 a sequence at least).
    const int decode_rows = s->max_rows < SMALL_ROWS ? s->max_rows : SMALL_ROWS;
    if (tasc_forward_is_small(m, s, nq)) {
        if (g_tasc_config.small_kernel != 0) {
            int cus = 0;
            {
                std::lock_guard<std::mutex> lock(g_dev_mu);
                DevState& ds = dev_state();
                if (ds.cu_count == 0) {
                    int dev = 0;
                    TASC_HIP(hipGetDevice(&dev));
                    TASC_HIP(hipDeviceGetAttribute(&ds.cu_count, hipDeviceAttributeMultiprocessorCount, dev));
                }
                cus = ds.cu_count;
            }
            int grid = g_tasc_config.small_grid > 0 ? g_tasc_config.small_grid : cus;
            grid = grid < cus ? grid : cus;      // every workgroup must be resident: at most one per compute unit
            if (pipe_path_fits(m, s->batch, decode_rows, s->max_blocks, grid)) return forward_pipe(m, s, nq, n_sel, logits_dbg, tail, grid, st);
        }
        return forward_small(m, s, nq, n_sel, logits_dbg, tail, st);
    }
    if (g_tasc_config.tiled_path != 0 && tasc_tiled_fits(m->desc)) return forward_tiled(m, s, nq, n_rows, n_sel, logits_dbg, tail, st);
    if (m->desc.dtype == TASC_F32) return forward_generic<float>(m, s, nq, n_rows, n_sel, logits_dbg, tail, st);
    return forward_generic<BF16>(m, s, nq, n_rows, n_sel, logits_dbg, tail, st);
}
