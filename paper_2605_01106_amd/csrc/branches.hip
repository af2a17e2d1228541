// Both branches of a block (attention and selective scan, Eq. 2) in one launch, for passes of up to 9 positions.  The branches
// only share their input; on streams of their own they would fork and join the captured graph in every layer (about 20 us).
// Each workgroup belongs to one branch and does what the branch's own kernel does, so the results are the same bits.
#include "attn_mfma_body.h"
#include "ssm_small_body.h"

namespace hh {

// Operands of the attention that fit 256 registers: two workgroups per compute unit (the cap also keeps the accumulators
// out of the second register file, with 16 to 44 moves less per step).
static constexpr bool two_per_cu(int rt, int ks) { return rt * ks <= 4 || (rt == 3 && ks == 2); }

// grid: the n_attn workgroups of the attention (slice fastest, then KV head, then sequence), then those of the scan (row
// group fastest, then head, then sequence); 256 threads
template <int RT, int KS, int NV, int SUBS, int TMAX>
__global__ __launch_bounds__(256, two_per_cu(RT, KS) ? 2 : 1) void branches_kernel(const Dims d, const AttnArgs at, const SsmArgs ss, const int n_attn, const int ssm_x) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  __shared__ int s_last;
  const int i = blockIdx.x;
  if (i < n_attn) {
    const int x = i % at.n_splits, r = i / at.n_splits;
    attn_mfma_body<RT, KS, true, 4>(d, at, 1, x, r % d.Hkv, r / d.Hkv, smem_raw, s_last);
  } else {
    const int j = i - n_attn, x = j % ssm_x, r = j / ssm_x;
    ssm_small_body<NV, SUBS, TMAX, 1, 4, true>(d, ss, x, r % d.Hm, r / d.Hm, reinterpret_cast<float*>(smem_raw));
  }
}

template <int RT, int KS, int NV, int SUBS, int TMAX>
static hipError_t launch_one(const Dims& d, const AttnArgs& at, const SsmArgs& ss, hipStream_t s) {
  constexpr int rows = 64 / SUBS * 4;
  const int n_attn = at.n_splits * d.Hkv * at.B, ssm_x = (d.P + rows - 1) / rows;
  size_t lds = attn_mfma_lds<RT, KS, true, 4>(at.n_splits);
  const size_t lds_ssm = (size_t)TMAX * 2 * NV * SUBS * sizeof(float);
  if (lds_ssm > lds) lds = lds_ssm;
  static size_t lds_enabled = 48 * 1024;
  if (lds > lds_enabled) {
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(branches_kernel<RT, KS, NV, SUBS, TMAX>),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    lds_enabled = lds;
  }
  hipLaunchKernelGGL((branches_kernel<RT, KS, NV, SUBS, TMAX>), dim3(n_attn + ssm_x * d.Hm * ss.B), dim3(256), lds, s, d, at, ss, n_attn, ssm_x);
  return hipGetLastError();
}

template <int KS, int NV, int SUBS>
static hipError_t launch_rows(const Dims& d, const AttnArgs& at, const SsmArgs& ss, int rt, hipStream_t s) {
  switch (ssm_small_tmax(ss.T) * 16 + rt) {
    case 0x11: return launch_one<1, KS, NV, SUBS, 1>(d, at, ss, s);
    case 0x31: return launch_one<1, KS, NV, SUBS, 3>(d, at, ss, s);
    case 0x51: return launch_one<1, KS, NV, SUBS, 5>(d, at, ss, s);
    case 0x52: return launch_one<2, KS, NV, SUBS, 5>(d, at, ss, s);
    case 0x92: return launch_one<2, KS, NV, SUBS, 9>(d, at, ss, s);
    case 0x93: return launch_one<3, KS, NV, SUBS, 9>(d, at, ss, s);
  }
  return hipErrorInvalidValue;
}
template <int KS>
static hipError_t launch_state(const Dims& d, const AttnArgs& at, const SsmArgs& ss, int rt, hipStream_t s) {
  const bool wide = ssm_small_wide(d, ss);
  if (d.N == 128) return wide ? launch_rows<KS, 8, 16>(d, at, ss, rt, s) : launch_rows<KS, 16, 8>(d, at, ss, rt, s);
  if (d.N == 256) return wide ? launch_rows<KS, 16, 16>(d, at, ss, rt, s) : launch_rows<KS, 32, 8>(d, at, ss, rt, s);
  return hipErrorInvalidValue;
}

static int scan_rows(const Dims& d, const SsmArgs& ss) { return ssm_small_wide(d, ss) ? 16 : 32; }   // state rows per workgroup
static SsmArgs one_layer(int B, int T) {
  SsmArgs ss{};
  ss.n_layers_z = 1; ss.B = B; ss.T = T;
  return ss;
}
int branches_scan_blocks(const Dims& d, int B, int T) {
  const int rows = scan_rows(d, one_layer(B, T));
  return (d.P + rows - 1) / rows * d.Hm * B;
}

// A launch of its own costs about 4 us, and the shorter branch hides behind the longer one; but the scan, bound by the HBM
// stream of its state, gets the registers of the attention: one or two workgroups per compute unit instead of five.  It stays
// hidden up to 1.5 rounds of workgroups with one per compute unit, up to 4 rounds with two.  Four blocks of the 3B shape (per
// call, before and after): two per compute unit, 640 workgroups 4208 -> 4070 us, 1280 2570 -> 2502, 1920 2010 -> 1853, but
// 5120 2843 -> 2860; one per compute unit, 320 workgroups 6230 -> 6078, but 640 8650 -> 8780.
// The kernels that exist are those of the shapes that were measured, not all that could gain: state sizes 128 and 256, head
// dimensions 33 to 128, and the row tiles that 3 to 5 query heads per KV head give (one tile up to three positions, one or two up
// to five, two or three up to nine).  Others, as 8 query heads per KV head at three positions or 1 at nine, launch the branches apart.
bool branches_fit(const Dims& d, int B, int T) {
  const SsmArgs ss = one_layer(B, T);
  if (!attention_uses_mfma(d) || !attention_mfma_fuses_append(d, T) || !ssm_small_fits(d, ss) || (d.N != 128 && d.N != 256)) return false;
  const int ks = (d.Dh + 31) / 32, rt = attention_mfma_row_tiles(d, T), tmax = ssm_small_tmax(T);
  const bool shape = tmax == 1 ? rt == 1 : tmax == 3 ? rt == 1 : tmax == 5 ? rt <= 2 : rt == 2 || rt == 3;
  if (ks < 2 || ks > 4 || !shape) return false;
  return branches_scan_blocks(d, B, T) <= (two_per_cu(rt, ks == 2 ? 2 : 4) ? 2048 : 384);
}

bool branches_take(const Dims& d, const AttnArgs& at, const SsmArgs& ss) {
  return branches_fit(d, at.B, at.T) && attention_mfma_accepts(d, at) && ss.n_layers_z == 1 && ss.T == at.T && ss.B == at.B;
}

hipError_t launch_branches(const Dims& d, const AttnArgs& at_in, const SsmArgs& ss, hipStream_t s) {
  AttnArgs at = at_in;
  if (!branches_take(d, at, ss)) return hipErrorInvalidValue;
  // (by ticket the last workgroups' fences would wait for all that the scan writes: 24 sequences 1913 -> 2975 us per call)
  const bool two_kernels = attention_mfma_two_kernels(d, at);
  if (two_kernels) at.counters = nullptr;
  const int rt = attention_mfma_row_tiles(d, at.T);
  const hipError_t e = d.Dh <= 64 ? launch_state<2>(d, at, ss, rt, s) : launch_state<4>(d, at, ss, rt, s);
  return e == hipSuccess && two_kernels ? launch_attention_merge(d, at, s) : e;
}

}  // namespace hh
