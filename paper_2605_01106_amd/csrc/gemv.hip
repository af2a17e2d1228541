// Skinny GEMM for the dense projections (in/out/QKV/MLP/LM head) when only a few
// rows of activations meet each weight: Y[m][n] = sum_k X'[m][k] * W[n][k].
//
// The weights are streamed from HBM exactly once per launch, so the kernel is bound by HBM
// bandwidth and, for the small matrices of a batch-1 decode step, by latency.  Hence:
//   * a wavefront owns R output rows and up to 2048 of their columns and issues all of its
//     16-byte weight loads at once, BEFORE it touches the activations; rows longer than
//     that are split between the wavefronts of a workgroup and added through LDS;
//   * many small workgroups (2 to 8 wavefronts resident per SIMD, fewer the longer the rows, whose
//     activations are requested in one go) rather than deep software pipelines: measured on MI355X this streams at 5.4-5.8 TB/s;
//   * the activation rows are staged once per workgroup in LDS in float32 and never rounded:
//     a bf16 weight times a float32 activation, accumulated in float32;
//   * RMSNorm is fused as a prologue in one pass: LDS holds x[k] * w[k], and the scalar
//     1 / sqrt(mean(x^2) + eps) multiplies the finished dot product;
//   * epilogues: plain store, in-place residual add (the old value is fetched with the first
//     loads), SwiGLU (gate and up matrices paired row by row: silu(gate) * up), and
//     per-workgroup argmax partials for the LM head (largest value, lowest index on ties).
#include <stdlib.h>

#include "gemv_kernel.h"

namespace hh {

static constexpr int kMaxBlocks = 1 << 15;
static constexpr size_t kLdsBudget = 150 * 1024;

int gemv_max_blocks() { return kMaxBlocks; }

// rows of a launch: `left` rows, or fewer where their activations do not fit in LDS
static int row_tile(int K, int left) {
  const int Kpad = (K + 511) & ~511;
  int mt_cap = 8;
  while (mt_cap > 1 && (size_t)mt_cap * Kpad * 4 + 4096 > kLdsBudget) --mt_cap;
  mt_cap = mt_cap >= 8 ? 8 : mt_cap >= 5 ? 5 : mt_cap >= 3 ? 3 : 1;
  const int mt = left > 5 ? 8 : left > 3 ? 5 : left > 1 ? 3 : 1;
  return mt > mt_cap ? mt_cap : mt;
}

static void set_blocks(const GemvArgs& a, GemvPlan& p) {
  const int rgb = kGemvWaves / p.KS, nrg = a.seg[0].n_rows / p.R;
  // several row groups per workgroup, so that staging the activations (MT * K floats per
  // workgroup, from L2) stays small next to the weights it meets
  constexpr int target = 1024;
  const int per = (nrg + rgb - 1) / rgb;
  p.iters = (per + target - 1) / target;
  if (p.iters < 1) p.iters = 1;
  if (p.iters > 64) p.iters = 64;
  p.blocks = (nrg + rgb * p.iters - 1) / (rgb * p.iters);
  const int pn = (a.epi == EPI_SWIGLU ? 2 : 1) * p.R * p.MT;
  p.lds = ((size_t)p.MT * ((a.K + 511) & ~511) + kGemvWaves * p.MT + 2 * kGemvWaves * pn + 4) * sizeof(float);
}

static bool make_plan(const GemvArgs& a, int MT, GemvPlan& p) {
  const int N = a.seg[0].n_rows;
  const int Kpad = (a.K + 511) & ~511;
  const int nch = Kpad >> 9;
  p.MT = MT; p.tiles = 1;
  // column split: each wavefront takes NCW chunks, KS wavefronts per row group
  if (nch <= 2) { p.NCW = 2; p.KS = 1; }
  else if (nch <= 4) { p.NCW = 2; p.KS = 2; }
  else if (nch <= 8) { p.NCW = 2; p.KS = 4; }
  else if (nch <= 16) { p.NCW = 4; p.KS = 4; }
  else return false;
  // rows per wavefront: R * NCW (* 2 for SwiGLU) loads of 16 bytes in flight per lane
  int rmax = 4;
  if (a.epi == EPI_SWIGLU || MT > 5) rmax = 2;
  if (!a.bf16) rmax = 1;
  p.R = rmax;
  const int rgb = kGemvWaves / p.KS;
  // R must divide N; use fewer rows per wavefront while that is needed to cover the CUs
  constexpr int min_blocks = 256;
  while (p.R > 1 && (N % p.R || N / p.R / rgb < min_blocks)) p.R >>= 1;
  set_blocks(a, p);
  return p.blocks <= kMaxBlocks;
}

// The plan of a pair: b takes the split of a (the longer rows); wavefronts behind the end of b's rows re-read its last columns
// and meet zero activations.
bool gemv_pair_plan(const GemvArgs& a, const GemvArgs& b, GemvPlan& pa, GemvPlan& pb) {
  if (a.epi != EPI_ADD || b.epi != EPI_STORE || a.M != b.M || a.M < 1 || a.bf16 != b.bf16 || a.n_seg != 1 || b.n_seg != 1 ||
      a.best != nullptr || b.best != nullptr || b.K > a.K || a.K % 8 != 0 || b.K % 8 != 0 || b.K < 8 || a.ldx % 4 != 0 || b.ldx % 4 != 0 ||
      a.seg[0].n_rows <= 0 || b.seg[0].n_rows <= 0)
    return false;
  const int mt = row_tile(a.K, a.M);
  if (a.M > mt || !make_plan(a, mt, pa) || b.seg[0].n_rows % pa.R != 0) return false;
  pb = pa;
  set_blocks(b, pb);
  return pa.blocks + pb.blocks <= kMaxBlocks;
}

hipError_t launch_gemv(const GemvArgs& a, int* n_blocks_out, hipStream_t s) {
  if (a.K % 8 != 0 || a.K < 8 || a.ldx % 4 != 0 || a.n_seg != 1) return hipErrorInvalidValue;
  if (a.seg[0].n_rows <= 0 || a.M <= 0) return hipSuccess;
  int mt_first = 0;
  for (int m0 = 0; m0 < a.M;) {
    int mt = row_tile(a.K, a.M - m0);
    // the argmax partials of all row tiles share one layout: keep one launch shape
    if (a.best != nullptr) { if (mt_first == 0) mt_first = mt; mt = mt_first; }
    GemvPlan p;
    if (!make_plan(a, mt, p)) return hipErrorInvalidValue;
    if (n_blocks_out) *n_blocks_out = p.blocks;
    // All row tiles of this shape in one launch: a tile's workgroups alone leave most of the chip idle, and float32 models take
    // this kernel at every row count.  Tiny float32 model, a launch per tile and now: prefill of 500 tokens 3.67 -> 1.33 ms, of 64
    // prompts of 900 tokens 288 -> 28 ms; round of 48 sequences at k = 4 2490 -> 577 us, of 8 at k = 2 297 -> 223.
    p.tiles = a.best != nullptr ? (a.M - m0 + mt - 1) / mt : (a.M - m0) / mt;
    if (p.tiles < 1) p.tiles = 1;
    hipError_t e;
    switch (a.epi) {
      case EPI_STORE: e = gemv_dispatch_store(a, m0, p, s); break;
      case EPI_ADD: e = gemv_dispatch_add(a, m0, p, s); break;
      case EPI_SWIGLU: e = gemv_dispatch_swiglu(a, m0, p, s); break;
      default: e = hipErrorInvalidValue;
    }
    if (e != hipSuccess) return e;
    m0 += mt * p.tiles;
  }
  return hipSuccess;
}

}  // namespace hh
