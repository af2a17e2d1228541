// Launches of the attention branch over a bf16 cache (attn_mfma_body.h: the kernel's description), and the merge of its key
// slices.
#include "attn_mfma_body.h"

namespace hh {

// grid: x = row_chunks * n_splits, y = Hkv, z = B
template <int RT, int KS, bool FUSE, int NW>
__global__ __launch_bounds__(64 * NW, RT * KS <= 4 || (RT == 3 && KS == 2) ? 2 : 1) void attn_mfma_kernel(const Dims d, const AttnArgs a, const int row_chunks) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  __shared__ int s_last;
  attn_mfma_body<RT, KS, FUSE, NW>(d, a, row_chunks, blockIdx.x, blockIdx.y, blockIdx.z, smem_raw, s_last);
}

// Merge of the key slices as a kernel of its own, for launches with many workgroups (there the
// device-wide fence of the ticket scheme costs more than a kernel boundary) or with much partial
// data per row chunk (one workgroup would pull all of it through one compute unit).
// grid: x = T * G rows, y = Hkv, z = B; one workgroup per output row.  Thread = (slice group sg,
// float4 column c4): it sums the slices sg, sg + SG, ... of its column; the groups meet in LDS.
__global__ __launch_bounds__(256) void attn_merge_kernel(const Dims d, const AttnArgs a) {
  __shared__ float2 gm[64];        // (maximum, sum) of every slice
  __shared__ float4 red[256];
  const int tid = threadIdx.x;
  const int rr = blockIdx.x, kvh = blockIdx.y, b = blockIdx.z;
  const int Dh = d.Dh, G = d.Hq / d.Hkv, S = a.n_splits, d4n = Dh >> 2;
  const int SG = min(256 / d4n, S), sg = tid / d4n, c4 = tid - sg * d4n;
  const bool active = sg < SG;
  const int j = rr / G, hq = kvh * G + rr % G;
  const size_t rid = ((size_t)b * a.T + j) * d.Hq + hq;
  const float* prow = a.part_o + rid * S * Dh + 4 * c4;
  float4 pv[4];                    // the first pass of loads does not wait for the statistics
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    const int sl = sg + u * SG;
    pv[u] = active && sl < S ? *reinterpret_cast<const float4*>(prow + (size_t)sl * Dh) : make_float4(0.f, 0.f, 0.f, 0.f);
  }
  if (tid < S) gm[tid] = reinterpret_cast<const float2*>(a.part_ml)[rid * S + tid];
  __syncthreads();
  float M = -INFINITY;
  for (int sl = 0; sl < S; ++sl) M = fmaxf(M, gm[sl].x);
  float4 out = make_float4(0.f, 0.f, 0.f, 0.f);
  for (int s0 = 0; s0 < S; s0 += 4 * SG) {
    if (s0 > 0) {
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int sl = s0 + sg + u * SG;
        pv[u] = active && sl < S ? *reinterpret_cast<const float4*>(prow + (size_t)sl * Dh) : make_float4(0.f, 0.f, 0.f, 0.f);
      }
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int sl = s0 + sg + u * SG;
      if (active && sl < S) {
        const float mx = gm[sl].x;
        const float w = mx == -INFINITY ? 0.f : ex2(mx - M);
        out.x = fmaf(w, pv[u].x, out.x); out.y = fmaf(w, pv[u].y, out.y);
        out.z = fmaf(w, pv[u].z, out.z); out.w = fmaf(w, pv[u].w, out.w);
      }
    }
  }
  red[tid] = out;
  __syncthreads();
  if (sg != 0) return;
  for (int q = 1; q < SG; ++q) {                           // fixed order: deterministic
    const float4 v = red[q * d4n + c4];
    out.x += v.x; out.y += v.y; out.z += v.z; out.w += v.w;
  }
  float L = 0.f;
  for (int sl = 0; sl < S; ++sl) {
    const float2 ml = gm[sl];
    L = fmaf(ml.x == -INFINITY ? 0.f : ex2(ml.x - M), ml.y, L);
  }
  const int nt = a.n_tok != nullptr ? a.n_tok[b] : a.T;
  const float inv = j < nt && L > 0.f ? 1.0f / L : 0.f;    // positions past the valid ones give zeros
  *reinterpret_cast<float4*>(a.o + ((size_t)b * a.T + j) * d.dq + (size_t)hq * Dh + 4 * c4) =
      make_float4(out.x * inv, out.y * inv, out.z * inv, out.w * inv);
}

template <int RT, int KS, bool FUSE, int NW>
static hipError_t launch_w(const Dims& d, const AttnArgs& a, int row_chunks, hipStream_t s) {
  const size_t lds = attn_mfma_lds<RT, KS, FUSE, NW>(a.n_splits);
  static size_t lds_enabled = 48 * 1024;
  if (lds > lds_enabled) {
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(attn_mfma_kernel<RT, KS, FUSE, NW>),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    lds_enabled = lds;
  }
  hipLaunchKernelGGL((attn_mfma_kernel<RT, KS, FUSE, NW>), dim3(row_chunks * a.n_splits, d.Hkv, a.B), dim3(64 * NW), lds, s, d, a,
                     row_chunks);
  return hipGetLastError();
}
template <int RT, int KS, bool FUSE>
static hipError_t launch_t(const Dims& d, const AttnArgs& a, int row_chunks, hipStream_t s) {
  // 4 wavefronts: with 8 a wavefront is left with 256 registers and the step loop spills
  return launch_w<RT, KS, FUSE, 4>(d, a, row_chunks, s);
}

template <int KS, bool FUSE>
static hipError_t launch_ks(const Dims& d, const AttnArgs& a, int rt, int row_chunks, hipStream_t s) {
  switch (rt) {
    case 1: return launch_t<1, KS, FUSE>(d, a, row_chunks, s);
    case 2: return launch_t<2, KS, FUSE>(d, a, row_chunks, s);
    case 3: if (KS < 8) return launch_t<(KS < 8 ? 3 : 1), KS, FUSE>(d, a, row_chunks, s); break;
    case 4: if (KS < 8) return launch_t<(KS < 8 ? 4 : 1), KS, FUSE>(d, a, row_chunks, s); break;
  }
  return hipErrorInvalidValue;
}

// the kernel appends the new keys itself: few new positions, one row chunk, 8-dim groups that do not straddle the rotation halves
bool attention_mfma_fuses_append(const Dims& d, int T) {
  return T <= 16 && attention_mfma_row_chunks(d, T) == 1 && d.Dh % 16 == 0;
}

// rows (position x query head of a KV group) per workgroup, in tiles of 16
int attention_mfma_row_tiles(const Dims& d, int T) {
  const int rows = T * (d.Hq / d.Hkv);
  const int rt_max = d.Dh > 128 ? 2 : 4;
  const int tiles = (rows + 15) / 16;
  return tiles < rt_max ? tiles : rt_max;
}
int attention_mfma_row_chunks(const Dims& d, int T) {
  const int rows = T * (d.Hq / d.Hkv);
  const int per = 16 * attention_mfma_row_tiles(d, T);
  return (rows + per - 1) / per;
}

static constexpr int kTicketMaxBlocks = 64;          // larger launches merge in a second kernel,
static constexpr size_t kTicketMaxBytes = 64 << 10;  // and so do those with more partial data per row chunk

bool attention_mfma_accepts(const Dims& d, const AttnArgs& a) {
  return d.bf16 && d.page_tokens % 32 == 0 && d.Dh <= 256 && d.Dh % 8 == 0 && d.Dh >= 8 && a.n_splits <= 64 && a.n_splits >= 1 && a.T >= 1 &&
         a.B >= 1 && (d.page_tokens & (d.page_tokens - 1)) == 0;
}

// whether the key slices of a launch are merged by a kernel of their own
bool attention_mfma_two_kernels(const Dims& d, const AttnArgs& a) {
  const int rt = attention_mfma_row_tiles(d, a.T), row_chunks = attention_mfma_row_chunks(d, a.T);
  return a.n_splits > 1 && ((long)row_chunks * a.n_splits * d.Hkv * a.B > kTicketMaxBlocks ||
                            (size_t)a.n_splits * rt * 16 * d.Dh * sizeof(float) > kTicketMaxBytes);
}

hipError_t launch_attention_merge(const Dims& d, const AttnArgs& a, hipStream_t s) {
  hipLaunchKernelGGL(attn_merge_kernel, dim3(a.T * (d.Hq / d.Hkv), d.Hkv, a.B), dim3(256), 0, s, d, a);
  return hipGetLastError();
}

hipError_t launch_attention_mfma(const Dims& d, const AttnArgs& a_in, hipStream_t s) {
  AttnArgs a = a_in;
  if (!attention_mfma_accepts(d, a)) return hipErrorInvalidValue;
  int rt = attention_mfma_row_tiles(d, a.T), row_chunks = attention_mfma_row_chunks(d, a.T);
  if (a.n_splits == 1 && !attention_mfma_fuses_append(d, a.T) && (a.keys > 1024 || (long)row_chunks * d.Hkv * a.B <= 64)) {
    // A prefill pass of few sequences: the smallest tiles that still run side by side, one workgroup per compute unit (a
    // workgroup's key steps are a serial chain that shortens with its rows).  One sequence: 509 positions at the 0.5B shape,
    // 64 workgroups of 4 tiles or 256 of one, prefill 7.53 -> 7.40 ms; 4096 in passes of 512 through four 3B blocks, 80
    // workgroups of 4 tiles 13.10 ms, 160 of 2 tiles 12.92, 320 of one 13.14.  Up to 1024 keys only where the launch would leave
    // three quarters of the chip idle: otherwise the scan beside it is the longer branch, and loses the compute units that the
    // attention spreads over (512 positions, 4 tiles against 2: two sequences at the 0.5B shape 1505 against 1532 us, one at the
    // 3B shape 787 against 800; two sequences of 6144 positions 19.65 against 19.03 ms).
    for (int t = 1; t < rt; ++t)
      if ((long)((a.T * (d.Hq / d.Hkv) + 16 * t - 1) / (16 * t)) * d.Hkv * a.B <= 256) rt = t;
    row_chunks = (a.T * (d.Hq / d.Hkv) + 16 * rt - 1) / (16 * rt);
  }
  const int ks = (d.Dh + 31) / 32;
  const bool two_kernels = attention_mfma_two_kernels(d, a);
  if (two_kernels) a.counters = nullptr;
  hipError_t e;
  if (attention_mfma_fuses_append(d, a.T)) {
    if (ks == 1) e = launch_ks<1, true>(d, a, rt, row_chunks, s);
    else if (ks == 2) e = launch_ks<2, true>(d, a, rt, row_chunks, s);
    else if (ks <= 4) e = launch_ks<4, true>(d, a, rt, row_chunks, s);
    else e = launch_ks<8, true>(d, a, rt, row_chunks, s);
  } else {
    if (ks == 1) e = launch_ks<1, false>(d, a, rt, row_chunks, s);
    else if (ks == 2) e = launch_ks<2, false>(d, a, rt, row_chunks, s);
    else if (ks <= 4) e = launch_ks<4, false>(d, a, rt, row_chunks, s);
    else e = launch_ks<8, false>(d, a, rt, row_chunks, s);
  }
  if (e != hipSuccess || !two_kernels) return e;
  return launch_attention_merge(d, a, s);
}

}  // namespace hh
