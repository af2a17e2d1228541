// Internal declarations shared by the translation units of libhh (not installed).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "../../include/hh.h"

namespace hh {

// ---- model dimensions derived from hh_cfg
struct Dims {
  int L, D, V;
  int Hm, P, N, d_inner, conv_dim, d_in_proj, ring_w;  // ring_w = conv_dim + Hm (raw xBC inputs | raw dt)
  int Hq, Hkv, Dh, dq, dkv, dqkv;
  int ldzx;         // row stride of the projection buffer: d_in_proj + dqkv (z | xBC | dt | q | k | v)
  int F;
  // Ring of raw conv inputs: what is read back are the 3 positions before a pass and the positions of a round, so that a bank of
  // ring_rows slots (a power of two, at least 16 and d_conv-1 + max_draft+1) holds it whatever the length of a prefill pass, of which the
  // last 3 positions are kept.  Passes of up to 509 positions have one bank that holds all of theirs; behind longer ones there are two banks:
  // pass p writes the one while it reads the positions before it from the other (ring_pass = 2^32 / prefill chunk rounded up; 0: one bank).
  int ring_rows, ring_slots;   // ring_slots: of all banks
  uint32_t ring_pass;
  int page_tokens, pages_per_seq, n_pages;
  int Bmax, Tmax, Gmax, Kmax, max_seq;
  int bf16;         // storage type of matrices and KV
  float eps, rope_base;
  int flags;        // hh_cfg.kernel_flags (HH_KF_* bits)
};

// ---- per-layer device pointers (an array of these lives in the workspace)
// slot of a position in the ring (before position 0: that of position 0)
__device__ __forceinline__ int ring_slot(const Dims& d, int pos) {
  const uint32_t p = (uint32_t)(pos > 0 ? pos : 0);
  return (int)((p & (uint32_t)(d.ring_rows - 1)) + (__umulhi(p, d.ring_pass) & 1u) * (uint32_t)d.ring_rows);
}
// first of a pass's nt positions that is kept in the ring
__device__ __forceinline__ int ring_first(const Dims& d, int nt) { return nt + 3 <= d.ring_rows ? 0 : nt - 3; }

struct LayerDev {
  const float *norm1, *conv_w, *conv_b, *a_log, *d_skip, *dt_bias, *gnorm, *norm2;
  const void *w_in, *w_out, *w_q, *w_k, *w_v, *w_o, *w_gate, *w_up, *w_down;
  void* w_inqkv;   // library-owned copy [d_in_proj + dqkv][D]: rows of w_in, w_q, w_k, w_v stacked
  float* S;        // committed SSM state of this layer   [B][Hm][P][N]
  float* S_draft;  // draft scratch state                 [B][Hm][P][N]
  float* ring;     // raw conv inputs, ring over positions [B][ring_slots][ring_w]
  void* kpool;     // K pages [n_pages][Hkv][page_tokens][Dh]
  void* vpool;     // V pages
};

// ---- skinny GEMM: Y[m][n] (op)= sum_k norm(X)[m][k] * W[n][k]
enum { EPI_STORE = 0, EPI_ADD = 1, EPI_SWIGLU = 2 };
// A bf16 matrix as the matrix-core kernels read it: scaled float16 tiles (packed_weight_elems 16-bit values) and its factors
// (scaled_tiles_floats): scale[0] for the activations of a many-row product and its inverse scale[1], scale[kScaleHead + n] the
// inverse of the factor that row n is held times.
constexpr int kScaleHead = 4;
struct HalfTiles { uint16_t* tiles; float* scale; };
struct GemvSeg {
  const void* W;    // [n_rows][K]
  const void* W2;   // EPI_SWIGLU: the "up" matrix paired row by row with W (gate)
  float* Y;         // [M][ldy], row n of this segment lands in column n
  int n_rows, ldy;
  HalfTiles H, H2;  // the same matrices for the matrix cores (bf16 weights only)
};
struct GemvArgs {
  const float* X; int ldx; int M; int K;
  const float* X2;                         // optional second addend of the input, same shape as X: X' = X + X2
  const float* R2;                         // EPI_ADD: optional second residual [M][ldy] added with the old Y
  const float* norm_w; float eps;          // rmsnorm prologue when norm_w != nullptr
  GemvSeg seg[4]; int n_seg;
  int epi;
  unsigned long long* best;                // optional per-block argmax partials [M][gridDim.x]
  int bf16;
  int flags;                               // hh_cfg.kernel_flags (HH_KF_* bits)
  int no_store;                            // EPI_STORE with an argmax output: only the argmax is wanted, Y need not be written
  unsigned long long* row_best;            // EPI_STORE, many-row kernels: per-row argmax keys [M] (zeroed by the caller), or nullptr
  // hand-over between two many-row products without a float32 round trip (see gemm_hands_over_planes):
  const uint16_t* planes_in;               // X already split into planes (X itself is not read)
  uint16_t* planes_out;                    // EPI_SWIGLU: the result goes out as split planes [gemm_planes_elems(M, N)] instead of Y
  // The SwiGLU result and the down projection that it goes to.  Its size goes with the square of the input's, so that no bound from
  // the weights alone comes near it: column j is held divided by act_factors_kernel's power of two (which the down projection's
  // tiles hold their column times), and in a many-row pass each row times a power of two from the norm of its normed input.
  const float* out_factor;                 // EPI_SWIGLU on the vector unit: inverse factor per column, or nullptr (the matrix-core kernels have it in H2's factors)
  float* row_factors_out;                  // EPI_SWIGLU, many rows: the rows' factors [M], written by the split; those of planes_out
  const float* row_weights;                // with row_factors_out: launch_act_input's weighted [K]
  const float* row_factors;                // many rows: the factors of X's rows or planes_in's, or nullptr (seg[0].H.scale[0])
  // Rows that the kernel and its K split are chosen for, where that is not M (0: M).  A prefill pass over prompts of unequal
  // length says batch x positions here: the order of its sums, and with it the bits of a sequence's results, then does not
  // depend on how long the other prompts are (chosen for the rows that exist it is no faster: two 3B blocks, 64 prompts of 224 to
  // 448 tokens and four rounds 39.29 against 39.35 ms, five prompts of 151 to 301 tokens no difference).
  int plan_rows;
};
inline int plan_rows(const GemvArgs& a) { return a.plan_rows > 0 ? a.plan_rows : a.M; }
hipError_t launch_gemv(const GemvArgs& a, int* n_blocks_out, hipStream_t s);
int gemv_max_blocks();   // upper bound on gridDim.x of launch_gemv (size of the argmax partial rows)

// ---- the same product for 1..16 activation rows on the matrix cores (bf16 weights; activations split in-kernel)
size_t packed_weight_elems(int N, int K);
bool skinny_mfma_fits(const GemvArgs& a);
hipError_t launch_skinny_mfma(const GemvArgs& a, float* partial, int* n_blocks_out, hipStream_t s);
// row_best (EPI_STORE only): per-row argmax keys [M], zeroed by the caller, raised with atomic maxima; store = 0: Y is not written
// f, f2: factors of the weight rows of each matrix
hipError_t launch_gemm_reduce(int epi, float* partial, int ksplit, int M, int N, const float* f, const float* f2, float* Y, int ldy, const float* R2,
                              const float* ssq, int ssq_ld, float rnorm_k, float eps, unsigned long long* row_best, int store,
                              hipStream_t s);

// ---- the same product for 17..96 activation rows on the matrix cores (weights from seg[0].H / H2,
// activations split in-kernel per K window; partial: scratch of gemm_partial_elems() floats)
bool mid_mfma_fits(const GemvArgs& a);
hipError_t launch_mid_mfma(const GemvArgs& a, float* partial, hipStream_t s);

// ---- two independent products of the same rows in one launch (and one reduction): a adds onto its output, b (no longer rows
// than a) stores.  b is split as a is, so that its sums may be grouped otherwise than in a launch of its own.
struct ReduceJob { float* partial; int ksplit; const float* f; float* Y; int ldy; const float* R2; const float* ssq; int ssq_ld; float rnorm_k, eps; };
hipError_t launch_gemm_reduce_pair(const ReduceJob& a, const ReduceJob& b, int M, int N, hipStream_t s);
bool gemv_pair_fits(const GemvArgs& a, const GemvArgs& b);
hipError_t launch_gemv_pair(const GemvArgs& a, const GemvArgs& b, hipStream_t s);
bool skinny_pair_fits(const GemvArgs& a, const GemvArgs& b);
hipError_t launch_skinny_pair(const GemvArgs& a, const GemvArgs& b, hipStream_t s);
bool mid_pair_fits(const GemvArgs& a, const GemvArgs& b);
hipError_t launch_mid_pair(const GemvArgs& a, const GemvArgs& b, float* partial_a, float* partial_b, hipStream_t s);

// ---- the same product on the matrix cores (weights as scaled float16 tiles, more than a few activation rows)
size_t gemm_planes_elems(int M, int K);   // 16-bit elements of scratch for the split activations
size_t scaled_tiles_floats(int N);
// tiles and factors (but for those of the activations) of W [N][K], column k times col[k] (nullptr: as it is); norms: the
// 2-norms of its rows [N rounded up to 16], columns times norm_col[k] (nullptr: as they are)
hipError_t launch_scaled_tiles(const void* W, int N, int K, size_t ldw, const float* col, const HalfTiles& h, const float* norm_col, float* norms, hipStream_t s);
// norm weights of the gate/up product's input times column factors u, and 1 / u (see column_max_kernel); scratch [16][K]
hipError_t launch_act_input(const void* gate, const void* up, int N, int K, const float* norm_w, float* scratch, float* weighted, float* inverse, hipStream_t s);
// factors of the SwiGLU result's columns, from the 2-norms of the gate's and the up matrix's rows: col[j] (the down projection's
// columns), inverse[j], and the up matrix's row factors times inverse[j] in up_out (its other values are up's)
hipError_t launch_act_factors(const float* n_gate, const float* n_up, int F, const float* up, float* up_out, float* col, float* inverse, hipStream_t s);
// factors of the activations, K columns normed with norm_w or products of them (see input_bound_kernel)
enum { BOUND_NORMED = 0, BOUND_VALUES = 1, BOUND_ACT = 2 };
hipError_t launch_input_bound(const float* norm_w, int K, int kind, const float* norms, int rows, const HalfTiles& h, hipStream_t s);
size_t gemm_partial_elems();              // float elements of scratch for split-K partial products
hipError_t launch_gemm_mfma(const GemvArgs& a, uint16_t* planes, float* partial, hipStream_t s);
// whether launch_gemm_mfma honours a.planes_out for these arguments (SwiGLU product through the LDS-staged
// kernel without a K split, result columns a multiple of 32): the caller then passes the same buffer as
// planes_in of the product that consumes the result
bool gemm_hands_over_planes(const GemvArgs& a);
// the most rows, up to `rows`, whose SwiGLU product (K columns, N results) does not hand its result over
int gemm_rows_without_hand_over(int rows, int K, int N, int flags);

// ---- SSM branch: causal conv + selective scan over up to T positions per sequence
struct SsmArgs {
  const LayerDev* layers; int layer0; int n_layers_z;  // blockIdx.z = (layer - layer0) * B + b
  LayerDev one;        // used instead of the table when layers == nullptr (single-layer launch)
  const float* zx;     // [B*T][ldzx] projections of this pass (nullptr: inputs come from the ring only)
  float* g;            // [B*T][d_inner]  y * silu(z)  (nullptr: no output)
  const int* pos0;     // [B] position of the first token of this pass
  const int* n_tok;    // [B] valid positions (<= T); nullptr: T for all
  const int* row0;     // [B] first row of each sequence in zx and g; nullptr: b * T (passes of more than 16 positions only)
  const int* n_acc;    // [B] rebuild mode: positions = n_acc[b] + 1
  const int* skip;     // [B] nonzero: leave this sequence untouched (may be nullptr)
  int T, B;
  int state_in, state_out;   // in: 0 committed S, 1 S_draft, 2 zeros.  out: 0 none, 1 S, 2 S_draft
  int write_ring;
  float* seg_scratch;        // ssd_segment_elems() floats for the segmented form of long passes over few sequences (nullptr: not available)
  float* ssd_shared;         // ssd_shared_elems() floats for the matmul form (nullptr: not available)
};
hipError_t launch_ssm(const Dims& d, const SsmArgs& a, hipStream_t s);
// the kernel for up to 9 positions on aligned shapes: whether it takes the pass, its position count (1, 3, 5, 9), and
// whether 16 lanes share a row (else 8)
bool ssm_small_fits(const Dims& d, const SsmArgs& a);
int ssm_small_tmax(int T);
bool ssm_small_wide(const Dims& d, const SsmArgs& a);
// matmul-form kernel for passes with many positions (ssd_mfma.hip); true if it took the pass
size_t ssd_segment_elems(const Dims& d);
size_t ssd_shared_elems(const Dims& d);
bool launch_ssd_mfma(const Dims& d, const SsmArgs& a, hipStream_t s, hipError_t* err);

// ---- attention branch
struct AttnArgs {
  void* kpool; void* vpool;  // this layer's K and V pages
  const float* qkv;       // [B*T][ldzx] (offset to the q column): raw q | k | v of this pass
  float* o;               // [B*T][dq]
  const int* pos0; const int* n_tok; const int* page_table;  // [B], [B], [B][pages_per_seq]
  const int* row0;        // [B] first row of each sequence in qkv and o; nullptr: b * T (one key slice only)
  const float* rope;      // [max_seq][Dh/2][2] (cos, sin)
  float* part_o; float* part_ml;  // split scratch: [B*T*Hq][S][Dh], [B*T*Hq][S][2]
  int* counters;          // [B][Hkv][row chunks], zero between launches: tickets of the key slices
  int T, B, n_splits;
  int keys;               // most keys that a sequence of the pass attends over (as far as the host knows)
};
int attention_row_chunks(const Dims& d, int T);
hipError_t launch_attention(const Dims& d, const AttnArgs& a, hipStream_t s);
bool attention_uses_mfma(const Dims& d);
int attention_mfma_row_chunks(const Dims& d, int T);
bool attention_mfma_fuses_append(const Dims& d, int T);
// bf16 cache, new keys already appended: the matrix-core kernel alone
hipError_t launch_attention_mfma(const Dims& d, const AttnArgs& a, hipStream_t s);
bool attention_mfma_accepts(const Dims& d, const AttnArgs& a);
int attention_mfma_row_tiles(const Dims& d, int T);
bool attention_mfma_two_kernels(const Dims& d, const AttnArgs& a);
hipError_t launch_attention_merge(const Dims& d, const AttnArgs& a, hipStream_t s);

// ---- both branches of a block in one launch (branches.hip): attention and scan of a pass of few positions
bool branches_fit(const Dims& d, int B, int T);
int branches_scan_blocks(const Dims& d, int B, int T);   // workgroups of the scan there
bool branches_take(const Dims& d, const AttnArgs& at, const SsmArgs& ss);   // whether launch_branches accepts the pass
hipError_t launch_branches(const Dims& d, const AttnArgs& at, const SsmArgs& ss, hipStream_t s);

// First row of sequence b in the buffers of a pass: b * T, or, in a prefill pass over prompts of unequal length, where the rows
// of the sequences before it end (only positions that exist have a row; then row0[b] + T <= (b + 1) * T, so that a read of up to T
// rows stays in the buffer, but a write past the valid positions would hit the next sequence).
__device__ __forceinline__ size_t first_row(const int* row0, int b, int T) { return row0 != nullptr ? (size_t)row0[b] : (size_t)b * T; }

// ---- small kernels
// first launch of a pass: tokens, embedding, positions, cleared argmax keys (see begin_pass_kernel)
enum { PASS_DRAFT = 0, PASS_VERIFY = 1, PASS_PROMPT = 2 };
struct PassArgs {
  const void* embed; int bf16, D, V;
  float* h;                                    // [B*T][D]
  const int *pending, *drafts, *prompt, *n_tok, *kv_len;
  int* pos0;
  int kmax, T, mode, step, row_stride, off;
  const int* row0;                             // PASS_PROMPT: [B] first row of each sequence in h, its n_tok rows alone; nullptr: b * T
  unsigned long long* clear;                   // [B*T] keys to clear, or nullptr
};
hipError_t launch_begin_pass(const PassArgs& a, int B, hipStream_t s);
hipError_t launch_argmax_finish(const unsigned long long* best, int n_part, int M, int* out, int out_stride,
                                int out_off, int T, const PassArgs* next, hipStream_t s);
struct CommitArgs {
  const int* drafts; const int* targets; const int* forced;  // [B][kmax], [B][kmax+1], [B] or nullptr
  int *committed, *last_n, *pending, *out_tok, *n_acc, *skip, *adv;
  unsigned long long* acc_stats;   // [2] running sums over rounds and active sequences: accepted drafts, tested drafts
  int B, k, kmax, G, out_stride;
};
hipError_t launch_accept(const CommitArgs& a, hipStream_t s);
hipError_t launch_advance(int* kv_len, const int* n, int B, hipStream_t s);
hipError_t launch_prefill_tail(const float* h, int T, int D, const int* n_tok, const int* row0, const int* is_last, float* lasth,
                               int* kv_len, int B, hipStream_t s);
hipError_t launch_prefill_finish(const int* first_tok, int* pending, int* out_tok, int out_stride, int* committed,
                                 int* last_n, int B, hipStream_t s);
// ---- token choice at temperature > 0 (rejection test of the round and its draws)
struct SamplingParams { float inv_t; uint32_t pad; uint64_t seed; };   // lives in device memory
// one row per sequence b at logits + b * row_stride -> out[b * out_stride + out_off];
// stream position of the drawn token: (idx_base ? idx_base[b] : 0) + idx_off.
// Parameters: *prm (device memory) when prm != nullptr, else prm_val.
hipError_t launch_sample_rows(const float* logits, size_t row_stride, int V, int B, const SamplingParams* prm,
                              SamplingParams prm_val, const int* idx_base, int idx_off, int purpose, int* out,
                              int out_stride, int out_off, hipStream_t s);
// logits_d [B][kmax][V], logits_v [B][k+1][V], stats: scratch of B * (2 * kmax + 1) * 2 floats
hipError_t launch_spec_targets(const float* logits_d, const float* logits_v, int V, int B, int k, int kmax,
                               const SamplingParams* prm, SamplingParams prm_val, float* stats, const int* drafts,
                               const int* committed, int* targets, hipStream_t s);
// device address and size of the current GPU's file-scope statistics array (no allocation)
hipError_t static_accept_scratch(float** ptr, size_t* n_floats);
hipError_t launch_fill_i32(int* p, int v, size_t n, hipStream_t s);
hipError_t launch_fill_f32(float* p, float v, size_t n, hipStream_t s);
hipError_t launch_export_state(const Dims& d, const LayerDev* layer, const int* kv_len, int B, float* conv_out,
                               hipStream_t s);
hipError_t launch_export_kv(const Dims& d, const LayerDev* layer, const int* page_table, int seq, int tok0,
                            int n_tokens, float* k, float* v, hipStream_t s);

}  // namespace hh
