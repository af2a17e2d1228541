// The selective scan of a few positions per pass (see ssm.hip for the layouts of state and ring).
#pragma once
#include "hh_internal.h"
#include "wave_ops.h"
#include "trace.h"

namespace hh {

__device__ __forceinline__ float softplus_f(float v) { return v > 20.0f ? v : log1pf(expf(v)); }


// ---- few positions per pass (draft steps, verification, rollback), 16-byte aligned rows.
// One wavefront per workgroup owns 64/SUBS rows p of one head, SUBS lanes share a row.  Every
// global load of the workgroup (state, conv taps and biases, the raw inputs of the T positions
// and of the 3 before them, dt, z) is issued before the first result is used, so the kernel
// costs about one memory round trip plus the recurrence.  The conv of B and C is computed
// once per workgroup, 4 channels per lane, and handed to the lanes through LDS.
// RG row groups of 64 / SUBS rows per workgroup, one after the other: the B/C convolution and the
// per-head scalars are shared by all of them, which is what a large batch needs (there a
// workgroup's fixed loads would otherwise exceed its share of the state).
// NWV wavefronts per workgroup (1 or 4), each with its own rows: with tens of thousands of
// one-wavefront workgroups the launch is bound by the workgroup dispatch rate (measured: 3
// resident wavefronts per compute unit), and four wavefronts share one B/C convolution.
// OUT = false (no outputs wanted: the commit's rebuild of the state from the ring): the read-out S C and
// the gate are not computed and positions behind the sequence's count are skipped (the count is
// uniform over the workgroup), which halves the arithmetic per position and leaves n + 1 instead of
// TMAX positions of it.
// CW (4 or 2) consecutive channels as one load or store; with 2 the upper half of the float4 is never used
template <int CW>
__device__ __forceinline__ float4 load_channels(const float* p) {
  if (CW == 4) return *reinterpret_cast<const float4*>(p);
  const float2 v = *reinterpret_cast<const float2*>(p);
  return make_float4(v.x, v.y, 0.f, 0.f);
}
template <int CW>
__device__ __forceinline__ void store_channels(float* p, const float4& v) {
  if (CW == 4) *reinterpret_cast<float4*>(p) = v;
  else *reinterpret_cast<float2*>(p) = make_float2(v.x, v.y);
}

// One workgroup: row groups bx, head h, bz = (layer, sequence); lds: TMAX * 2 N floats.
template <int NV, int SUBS, int TMAX, int RG, int NWV, bool OUT>
__device__ __forceinline__ void ssm_small_body(const Dims& d, const SsmArgs& a, const int bx, const int h, const int bz, float* lds) {
  constexpr int NTHR = 64 * NWV;
  constexpr int ROWS = 64 / SUBS, N = NV * SUBS;
  // B|C channels per thread and group: 4, or 2 where groups of 4 would leave threads of the workgroup idle (half
  // the registers for the taps and the raw rows of the convolution: one more resident wavefront per SIMD)
  constexpr int CW = 2 * N / 4 >= NTHR ? 4 : 2;
  constexpr int NGR = 2 * N / CW;                      // groups in all
  constexpr int NG = (NGR + NTHR - 1) / NTHR;          // groups per thread
  float(*BCs)[2 * N] = reinterpret_cast<float(*)[2 * N]>(lds);

  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int row = lane / SUBS, sub = lane % SUBS;
  const int p0 = (bx * NWV + wave) * ROWS * RG;
  const int lz = bz / a.B, b = bz % a.B;
  const LayerDev& ly = a.layers != nullptr ? a.layers[a.layer0 + lz] : a.one;
  TR(0);
  // Loads in the order of what they wait for.  Nothing here depends on the per-sequence
  // scalars except the ring rows (slot = position mod ring size), which come last.  (A ring holds more rows than a pass of this kernel.)
  int pr[RG], cx[RG];
  bool prow[RG];
#pragma unroll
  for (int rg = 0; rg < RG; ++rg) {
    pr[rg] = min(p0 + rg * ROWS + row, d.P - 1);
    prow[rg] = p0 + rg * ROWS + row < d.P;
    cx[rg] = h * d.P + pr[rg];
  }
  float* ring = ly.ring + (size_t)b * d.ring_slots * d.ring_w;
  const float* zx = a.zx != nullptr ? a.zx + (size_t)b * a.T * d.ldzx : nullptr;
  const int skip_v = (a.skip != nullptr ? a.skip : a.pos0)[b];   // absent arrays read pos0 instead and are ignored
  const int nacc_v = (a.n_acc != nullptr ? a.n_acc : a.pos0)[b];
  const int ntok_v = (a.n_tok != nullptr ? a.n_tok : a.pos0)[b];
  const int pos0 = a.pos0[b];
  float S[RG][NV];
  // (a macro, not a lambda: the state must stay in registers)
#define HH_LOAD_STATE()                                                                                                   \
  {                                                                                                                       \
    const float* src = a.state_in == 0 ? ly.S : (a.state_in == 1 ? ly.S_draft : nullptr);                                 \
    _Pragma("unroll") for (int rg = 0; rg < RG; ++rg) {                                                                   \
      if (src != nullptr) {                                                                                               \
        /* float4 i of a lane: elements (i/4)*4*SUBS + 4*sub .. */                                                        \
        const float* sp = src + (((size_t)b * d.Hm + h) * d.P + pr[rg]) * N + sub * 4;                                    \
        _Pragma("unroll") for (int i = 0; i < NV; i += 4) {                                                               \
          const float4 v = *reinterpret_cast<const float4*>(sp + i * SUBS);                                               \
          S[rg][i] = v.x; S[rg][i + 1] = v.y; S[rg][i + 2] = v.z; S[rg][i + 3] = v.w;                                     \
        }                                                                                                                 \
      } else {                                                                                                            \
        _Pragma("unroll") for (int i = 0; i < NV; ++i) S[rg][i] = 0.f;                                                    \
      }                                                                                                                   \
    }                                                                                                                     \
  }
  // With outputs the state is requested first (the longest wait).  The rebuild holds up to TMAX + 3 ring rows of
  // B | C per thread until the convolution is done; it requests the state behind that, which keeps it at the
  // register count of the one-position kernel (more resident wavefronts cover the wait instead).
  if (OUT) HH_LOAD_STATE();
  float4 bw[NG][CW], bb[NG], braw[NG][TMAX + 3];
  float xraw[RG][TMAX + 3], zg[RG][TMAX];
  float dtraw_l = 0.f;   // raw dt of position `lane` (lanes < T): softplus and decay are evaluated once, lane-parallel
#pragma unroll
  for (int u = 0; u < NG; ++u) {
    const int c = d.d_inner + CW * min(tid + NTHR * u, NGR - 1);
#pragma unroll
    for (int t = 0; t < CW; ++t) bw[u][t] = *reinterpret_cast<const float4*>(ly.conv_w + (size_t)(c + t) * 4);
    bb[u] = load_channels<CW>(ly.conv_b + c);
  }
  float4 xw[RG];
  float xb[RG];
#pragma unroll
  for (int rg = 0; rg < RG; ++rg) {
    xw[rg] = *reinterpret_cast<const float4*>(ly.conv_w + (size_t)cx[rg] * 4);
    xb[rg] = ly.conv_b[cx[rg]];
  }
  const float dskip = ly.d_skip[h];
  const float dtb = ly.dt_bias[h];
  const float alog = ly.a_log[h];
  if (zx != nullptr) {   // inputs of this pass: rows 0 .. T-1 of the projection buffer (rows >= nt are read but not used)
#pragma unroll
    for (int j = 0; j < TMAX; ++j) {
      const float* r = zx + (size_t)min(j, a.T - 1) * d.ldzx + d.d_inner;
#pragma unroll
      for (int u = 0; u < NG; ++u) braw[u][j + 3] = load_channels<CW>(r + d.d_inner + CW * min(tid + NTHR * u, NGR - 1));
#pragma unroll
      for (int rg = 0; rg < RG; ++rg) {
        xraw[rg][j + 3] = r[cx[rg]];
        zg[rg][j] = a.g != nullptr ? r[cx[rg] - d.d_inner] : 0.f;   // z precedes xBC in the row
      }
    }
    dtraw_l = zx[(size_t)min(lane, a.T - 1) * d.ldzx + d.d_inner + d.conv_dim + h];
  }
  if (a.skip != nullptr && skip_v) return;
  int nt = a.T;
  if (a.n_acc != nullptr) nt = nacc_v + 1;
  else if (a.n_tok != nullptr) nt = ntok_v;
  if (nt <= 0) return;
  nt = min(nt, TMAX);
  // row of raw inputs (xBC | dt) of position pos0 + j in the ring (positions before 0 read slot 0 and count as 0)
  auto ring_row = [&](int j) -> const float* { return ring + (size_t)ring_slot(d, pos0 + j) * d.ring_w; };
#pragma unroll
  for (int j = -3; j < (int)TMAX; ++j) {
    if (j >= 0 && zx != nullptr) continue;
    if (!OUT && j >= nt) continue;               // the rebuild never uses positions behind the count: no loads for them
    const float* r = ring_row(min(j, nt - 1));
#pragma unroll
    for (int u = 0; u < NG; ++u) braw[u][j + 3] = load_channels<CW>(r + d.d_inner + CW * min(tid + NTHR * u, NGR - 1));
#pragma unroll
    for (int rg = 0; rg < RG; ++rg) {
      xraw[rg][j + 3] = r[cx[rg]];
      if (j >= 0) zg[rg][j] = 0.f;
    }
  }
  if (zx == nullptr) dtraw_l = ring_row(min(lane, nt - 1))[d.conv_dim + h];
  const float negA = -expf(alog);
  TR(1);

  // ---- conv + SiLU: B and C for the whole workgroup (branch-free: clamped inputs, every
  // position computed; positions >= nt are never used)
#pragma unroll
  for (int u = 0; u < NG; ++u) {
    const int gi = tid + NTHR * u;
#pragma unroll
    for (int j = 0; j < TMAX; ++j) {
      if (!OUT && j >= nt) continue;             // (a guard per position, not a loop exit: the unrolled arrays stay in registers)
      float4 o = make_float4(0.f, 0.f, 0.f, 0.f);
      float* op = reinterpret_cast<float*>(&o);
#pragma unroll
      for (int ch = 0; ch < CW; ++ch) {
        const float r0 = pos0 + j - 3 < 0 ? 0.f : reinterpret_cast<const float*>(&braw[u][j])[ch];
        const float r1 = pos0 + j - 2 < 0 ? 0.f : reinterpret_cast<const float*>(&braw[u][j + 1])[ch];
        const float r2 = pos0 + j - 1 < 0 ? 0.f : reinterpret_cast<const float*>(&braw[u][j + 2])[ch];
        const float r3 = reinterpret_cast<const float*>(&braw[u][j + 3])[ch];
        float acc = bw[u][ch].x * r0;
        acc = fmaf(bw[u][ch].y, r1, acc); acc = fmaf(bw[u][ch].z, r2, acc); acc = fmaf(bw[u][ch].w, r3, acc);
        op[ch] = fast_silu(acc + reinterpret_cast<const float*>(&bb[u])[ch]);
      }
      if (gi < NGR) store_channels<CW>(&BCs[j][CW * gi], o);
    }
  }
  // ---- per-position scalars of the head (step and decay), all positions at once
  float dtj[TMAX], aj[TMAX];
  const float dt_l = softplus_f(dtraw_l + dtb);
  const float a_l = expf(negA * dt_l);
#pragma unroll
  for (int j = 0; j < TMAX; ++j) {
    const bool on = j < nt;
    dtj[j] = on ? __int_as_float(__builtin_amdgcn_readlane(__float_as_int(dt_l), j)) : 0.f;
    aj[j] = on ? __int_as_float(__builtin_amdgcn_readlane(__float_as_int(a_l), j)) : 1.f;   // positions >= nt leave the state as it is
  }
  // ---- keep the raw inputs of these positions for later windows and for rollback
  if (a.write_ring && zx != nullptr) {
#pragma unroll
    for (int rg = 0; rg < RG; ++rg) {
      if (sub == 0 && prow[rg]) {
#pragma unroll
        for (int j = 0; j < TMAX; ++j)
          if (j < nt) ring[(size_t)ring_slot(d, pos0 + j) * d.ring_w + cx[rg]] = xraw[rg][j + 3];
      }
    }
    if (h == 0 && bx == 0) {
#pragma unroll
      for (int u = 0; u < NG; ++u) {
        const int gi = tid + NTHR * u;
        if (gi < NGR) {
#pragma unroll
          for (int j = 0; j < TMAX; ++j)
            if (j < nt) store_channels<CW>(ring + (size_t)ring_slot(d, pos0 + j) * d.ring_w + d.d_inner + CW * gi, braw[u][j + 3]);
        }
      }
      for (int it = tid; it < nt * d.Hm; it += NTHR) {
        const int j = it / d.Hm, hh = it - j * d.Hm;
        ring[(size_t)ring_slot(d, pos0 + j) * d.ring_w + d.conv_dim + hh] = zx[(size_t)j * d.ldzx + d.d_inner + d.conv_dim + hh];
      }
    }
  }
  TR(2);
  __syncthreads();
  TR(3);
  if (!OUT) HH_LOAD_STATE();
#undef HH_LOAD_STATE

  // ---- per row group: conv + SiLU of x, recurrence, outputs
#pragma unroll
  for (int rg = 0; rg < RG; ++rg) {
    float y[TMAX];
#pragma unroll
    for (int j = 0; j < TMAX; ++j) {
      if (!OUT && j >= nt) continue;
      const float r0 = pos0 + j - 3 < 0 ? 0.f : xraw[rg][j];
      const float r1 = pos0 + j - 2 < 0 ? 0.f : xraw[rg][j + 1];
      const float r2 = pos0 + j - 1 < 0 ? 0.f : xraw[rg][j + 2];
      float acc = xw[rg].x * r0;
      acc = fmaf(xw[rg].y, r1, acc); acc = fmaf(xw[rg].z, r2, acc); acc = fmaf(xw[rg].w, xraw[rg][j + 3], acc);
      const float xv = fast_silu(acc + xb[rg]);
      const float coef = dtj[j] * xv;
      if (!OUT) {
#pragma unroll
        for (int i = 0; i < NV; i += 4) {
          const float4 Bv = *reinterpret_cast<const float4*>(&BCs[j][i * SUBS + sub * 4]);
          S[rg][i] = fmaf(aj[j], S[rg][i], coef * Bv.x);
          S[rg][i + 1] = fmaf(aj[j], S[rg][i + 1], coef * Bv.y);
          S[rg][i + 2] = fmaf(aj[j], S[rg][i + 2], coef * Bv.z);
          S[rg][i + 3] = fmaf(aj[j], S[rg][i + 3], coef * Bv.w);
        }
        continue;
      }
      const float gate = fast_silu(zg[rg][j]);
      float part = 0.f;
#pragma unroll
      for (int i = 0; i < NV; i += 4) {
        const float4 Bv = *reinterpret_cast<const float4*>(&BCs[j][i * SUBS + sub * 4]);
        const float4 Cv = *reinterpret_cast<const float4*>(&BCs[j][N + i * SUBS + sub * 4]);
        S[rg][i] = fmaf(aj[j], S[rg][i], coef * Bv.x); part = fmaf(S[rg][i], Cv.x, part);
        S[rg][i + 1] = fmaf(aj[j], S[rg][i + 1], coef * Bv.y); part = fmaf(S[rg][i + 1], Cv.y, part);
        S[rg][i + 2] = fmaf(aj[j], S[rg][i + 2], coef * Bv.z); part = fmaf(S[rg][i + 2], Cv.z, part);
        S[rg][i + 3] = fmaf(aj[j], S[rg][i + 3], coef * Bv.w); part = fmaf(S[rg][i + 3], Cv.w, part);
      }
      part += dpp_move<0xB1>(part);    // lane ^ 1
      part += dpp_move<0x4E>(part);    // lane ^ 2
      if (SUBS >= 8) part += dpp_move<0x141>(part);    // the other quad of 8 lanes
      if (SUBS == 16) part += dpp_move<0x140>(part);   // the other half of 16 lanes
      y[j] = (part + dskip * xv) * gate;
    }
    if (a.g != nullptr && sub == 0 && prow[rg]) {
#pragma unroll
      for (int j = 0; j < TMAX; ++j)
        if (j < nt) a.g[((size_t)b * a.T + j) * d.d_inner + cx[rg]] = y[j];
    }
    if (a.state_out != 0 && prow[rg]) {
      float* dst = (a.state_out == 1 ? ly.S : ly.S_draft) + (((size_t)b * d.Hm + h) * d.P + pr[rg]) * N + sub * 4;
#pragma unroll
      for (int i = 0; i < NV; i += 4)
        *reinterpret_cast<float4*>(dst + i * SUBS) = make_float4(S[rg][i], S[rg][i + 1], S[rg][i + 2], S[rg][i + 3]);
    }
  }
  TR(5);
}

}  // namespace hh
