// SSM branch of a pass with many positions per sequence (prefill chunks) in the matmul
// ("state-space dual") form, on the matrix cores in float32.
//
// The scalar-decay recurrence  S_t = a_t S_{t-1} + dt_t x_t (outer) B_t,  y_t = S_t C_t + D x_t
// over a chunk of L positions with the state S entering it is, with cum_t = sum_{i<=t} log a_i,
//     y_t = exp(cum_t) * (S C_t)  +  sum_{i<=t} [ (C_t . B_i) * exp(cum_t - cum_i) * dt_i ] x_i  +  D x_t
//     S'  = exp(cum_L) * S        +  sum_i  exp(cum_L - cum_i) * dt_i * x_i (outer) B_i
// - four small matrix products per chunk instead of L dependent state updates.  All exponents are
// <= 0, so nothing overflows whatever the decay.  Products are v_mfma_f32_16x16x4_f32 (exact
// float32 products, float32 accumulation).  cum_t reaches -70 within a chunk (32 steps of 0.3 at
// A = 8), and a decay exp(cum_t - cum_i) of neighbouring positions carries the absolute error of
// both sums: the sums and their differences are float64, the exponent is rounded once, and the
// rounding differs from the sequential kernels only in the order of the sums.  (With float32 sums
// the state behind a full chunk was 2 to 3.6 times as far from float64 as theirs, and the logits of
// its last position 1.2 to 1.6 times; now 0.9 to 1.1.  Time unchanged: prefill of 4096 tokens
// through four 3B blocks 13.38 against 13.39 ms.)
//
// What does not depend on the head - B and C behind convolution and SiLU, G = C B^T, the step sizes and their running sums - is computed
// once per chunk by ssd_shared_kernel (a workgroup per chunk and sequence), into scratch that the walking workgroups copy to LDS.  Computed
// by every pair of heads it was four fifths of their convolutions and a quarter of their time: a walk of 64 sequences x 64 positions
// at the 3B shape 323 -> 225 us, the first kernel's 15 included (a workgroup 55.6 -> 35 us: 6 for the read-out and 7 for the update of a
// chunk, of which the matrix pipe needs 3.4 each; state in and out 8); three segments' launches for 509 positions of one sequence
// at the 0.5B shape 43 -> 38; prefill of 4096 tokens through four 3B blocks 8.53 -> 7.69 ms, same bits.
//
// One workgroup of eight wavefronts per (sequence, pair of heads), head dimension P = 64: B, C and G are read once for the
// pair, and two wavefronts per SIMD hide each other's LDS latency.  Wavefront 4 hh + wq owns the 16 rows
// p = 16 wq .. 16 wq + 15 of head hh of the pair for everything - its slice of the state,
// transposed (n down, p across), lives in MFMA accumulator registers for the whole pass and is
// fed back as the A operand of the read-out product as it is: lane (g, j) holds S[p = 16 wq + j]
// [n = 16 tile + 4 g + r], which the instruction takes as A[row j][k = g] when the B operand is
// read with the same n for k = g.  Per chunk of 32 positions: the convolution + SiLU of x (a thread takes 4 channels at
// two positions) and the copies of B and C, all of it requested before the products of the chunk before, so that its latency hides
// behind the MFMAs; the masked and scaled M of each head to LDS, the read-out of the old state, the intra-chunk product M x,
// the outputs y * silu(z), and the state update.  B is kept row-major and C transposed in LDS,
// padded so that the operand reads of the two large products are free of bank conflicts; they are read a state tile (four
// positions of B) ahead of the MFMAs, explicitly: left to the compiler each read was waited for.
#include <stdlib.h>

#include <algorithm>

#include "hh_internal.h"
#include "wave_ops.h"
#include "trace.h"

namespace hh {

typedef float ssd_f32x4 __attribute__((ext_vector_type(4)));

static constexpr int kSsdL = 32;    // positions per chunk
static constexpr int kSsdP = 64;    // head dimension
static constexpr int kSsdMinT = 16; // shortest pass

__device__ __forceinline__ float ssd_softplus(float v) { return v > 20.0f ? v : log1pf(expf(v)); }

// depthwise convolution (taps tw[channel], window x0 .. x3) + SiLU of 4 channels
__device__ __forceinline__ void ssd_conv4(const float4& q0, const float4& q1, const float4& q2, const float4& q3, const float4 (&tw)[4], const float4& bias,
                                          float4& out) {
  const float x0[4] = {q0.x, q0.y, q0.z, q0.w}, x1[4] = {q1.x, q1.y, q1.z, q1.w}, x2[4] = {q2.x, q2.y, q2.z, q2.w}, x3[4] = {q3.x, q3.y, q3.z, q3.w};
  const float bq[4] = {bias.x, bias.y, bias.z, bias.w};
  float o[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    float acc = tw[q].x * x0[q];
    acc = fmaf(tw[q].y, x1[q], acc); acc = fmaf(tw[q].z, x2[q], acc); acc = fmaf(tw[q].w, x3[q], acc);
    o[q] = fast_silu(acc + bq[q]);
  }
  out = make_float4(o[0], o[1], o[2], o[3]);
}

template <int N>
struct SsdLds {
  static constexpr int LDB = N + 16, LDT = kSsdL + 4, LDX = kSsdP + 16, LDM = kSsdL + 4;
  static constexpr int kB = 0;                         // B  [L][LDB]      (position, n)
  static constexpr int kCt = kB + kSsdL * LDB;         // C^T [N][LDT]     (n, position)
  static constexpr int kX = kCt + N * LDT;             // x  [2][L][LDX]   (head of the pair, position, p)
  static constexpr int kM = kX + 2 * kSsdL * LDX;      // M  [2][L][LDM]   (head of the pair, t, i)
  static constexpr int kDt = kM + 2 * kSsdL * LDM;     // dt [2][L]
  static constexpr int kCum = kDt + 2 * kSsdL;         // cum [2][L], doubles
  static constexpr int kFloats = kCum + 4 * kSsdL;
  static_assert(kCum % 2 == 0, "the doubles are aligned");
};

// SEG_WALK: a workgroup walks the whole pass.  With few sequences that leaves most of the chip idle, so the pass is
// cut into segments of `len` positions (blockIdx.z): SEG_LOCAL computes every segment's own contribution to the state
// (as if zeros entered it) and its log-decay sum, ssd_combine_kernel chains them and leaves the state that enters each
// segment in the same place, and SEG_OUT computes the outputs of every segment from the state entering it.
enum { SEG_WALK = 0, SEG_LOCAL = 1, SEG_OUT = 2 };
struct SsdSeg {
  float* states;   // [B][n][Hm][P][N]
  float* decay;    // [B][n][Hm] log-decay sums
  int len, n;
};

// What the heads of a sequence share, once per chunk of a pass instead of once per pair of heads: B and C behind convolution and SiLU,
// G = C B^T, and every head's step sizes and log-decay sums.
//   [B: L x N][C^T: N x L][G: the tiles (0,0), (1,0), (1,1), 64 lanes x 4][log-decay sums: Hm x L doubles][dt: Hm x L]
template <int N>
struct SsdShared {
  static constexpr int kB = 0, kCt = kSsdL * N, kG = 2 * kSsdL * N, kCum = kG + 3 * 256;
  static_assert(kCum % 2 == 0, "the doubles are aligned");
  __host__ __device__ static size_t dt(int Hm) { return (size_t)kCum + 2 * kSsdL * Hm; }
  __host__ __device__ static size_t floats(int Hm) { return (size_t)kCum + 3 * kSsdL * Hm; }
};
__host__ __device__ __forceinline__ int ssd_chunks(int T) { return (T + kSsdL - 1) / kSsdL; }

// grid: x = chunks of the pass, y = sequences
template <int N>
__global__ __launch_bounds__(512) void ssd_shared_kernel(const Dims d, const SsmArgs a) {
  typedef SsdShared<N> Sh;
  constexpr int L = kSsdL, LDS = N + 4;                // rows of B and C; + 4: the operand reads are free of bank conflicts
  constexpr int NG = 2 * N / 4, PP = L * NG / 512;     // channel groups of 4, positions per thread
  __shared__ __align__(16) float rows_s[2 * L * LDS];
  const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int b = blockIdx.y, j0 = blockIdx.x * L;
  const int nt = a.n_tok != nullptr ? a.n_tok[b] : a.T;
  if (j0 >= nt) return;
  const int tc = min(L, nt - j0), pos0 = a.pos0[b], keep = ring_first(d, nt);
  const LayerDev& ly = a.one;
  float* ring = ly.ring + (size_t)b * d.ring_slots * d.ring_w;
  const float* zx = a.zx + first_row(a.row0, b, a.T) * d.ldzx;
  float* out = a.ssd_shared + ((size_t)b * ssd_chunks(a.T) + blockIdx.x) * Sh::floats(d.Hm);
  // ---- convolution + SiLU of 4 channels at PP positions
  const int sg = tid % NG, first = PP * (tid / NG), ch = d.d_inner + 4 * sg;
  float4 rows[3 + PP], tw[4];
#pragma unroll
  for (int u = 0; u < 3 + PP; ++u) {
    const int pos = pos0 + min(j0 + first - 3 + u, nt - 1);
    const float4 v = *reinterpret_cast<const float4*>(pos >= pos0 ? zx + (size_t)(pos - pos0) * d.ldzx + d.d_inner + ch
                                                                  : ring + (size_t)ring_slot(d, pos) * d.ring_w + ch);
    rows[u] = pos < 0 ? make_float4(0.f, 0.f, 0.f, 0.f) : v;
  }
#pragma unroll
  for (int q = 0; q < 4; ++q) tw[q] = *reinterpret_cast<const float4*>(ly.conv_w + (size_t)(ch + q) * 4);
  const float4 bias = *reinterpret_cast<const float4*>(ly.conv_b + ch);
  // ---- step sizes and log-decay sums: half a wavefront per head
  for (int h0 = 2 * w; h0 < d.Hm; h0 += 16) {          // (Hm is even)
    const int hd = h0 + (lane >> 5), t = lane & 31;
    const bool on = t < tc;
    const float rawdt = zx[(size_t)(j0 + min(t, tc - 1)) * d.ldzx + d.d_inner + d.conv_dim + hd];
    const float dt = on ? ssd_softplus(rawdt + ly.dt_bias[hd]) : 0.f;
    if (on && a.write_ring && j0 + t >= keep) ring[(size_t)ring_slot(d, pos0 + j0 + t) * d.ring_w + d.conv_dim + hd] = rawdt;
    float la = on ? -expf(ly.a_log[hd]) * dt : 0.f;    // log a_t, float32 as in the sequential kernels
    // a decay below exp(-200) is zero in float32, and so is every product that holds it; bounded, its sums stay finite
    // (a rate of infinity would make their differences NaN) and keep the bits of the positions around it
    la = la < -200.f ? -200.f : la;
    double c = la;                                     // summed over the positions up to t
#pragma unroll
    for (int o = 1; o < L; o <<= 1) {
      const double up = __shfl_up(c, o, 32);
      if (t >= o) c += up;
    }
    reinterpret_cast<double*>(out + Sh::kCum)[(size_t)hd * L + t] = c;
    out[Sh::dt(d.Hm) + (size_t)hd * L + t] = dt;
  }
  const bool is_c = sg >= N / 4;
#pragma unroll
  for (int u = 0; u < PP; ++u) {
    const int jj = first + u;
    const bool on = jj < tc;
    float4 o;
    ssd_conv4(rows[u], rows[u + 1], rows[u + 2], rows[u + 3], tw, bias, o);
    if (!on) o = make_float4(0.f, 0.f, 0.f, 0.f);
    *reinterpret_cast<float4*>(rows_s + (is_c ? L * LDS : 0) + jj * LDS + 4 * (sg % (N / 4))) = o;
    if (!is_c) *reinterpret_cast<float4*>(out + Sh::kB + jj * N + 4 * sg) = o;
    // the raw inputs stay in the ring for the next pass's window and for rollbacks
    if (on && a.write_ring && j0 + jj >= keep) *reinterpret_cast<float4*>(ring + (size_t)ring_slot(d, pos0 + j0 + jj) * d.ring_w + ch) = rows[u + 3];
  }
  __syncthreads();
  const float* Bs = rows_s;
  const float* Cs = rows_s + L * LDS;
  for (int i = tid; i < N * L / 4; i += 512) {         // C^T: 4 positions of one n
    const int n = i >> 3, q = i & 7;
    *reinterpret_cast<float4*>(out + Sh::kCt + 4 * i) =
        make_float4(Cs[4 * q * LDS + n], Cs[(4 * q + 1) * LDS + n], Cs[(4 * q + 2) * LDS + n], Cs[(4 * q + 3) * LDS + n]);
  }
  if (w < 3) {                                         // G on the tiles at or below the diagonal
    const int g = lane >> 4, j = lane & 15, tt = w == 0 ? 0 : 1, it = w == 2 ? 1 : 0;
    ssd_f32x4 G = {0.f, 0.f, 0.f, 0.f};
#pragma unroll 8
    for (int kk = 0; kk < N / 4; ++kk) {
      const float av = Cs[(16 * tt + j) * LDS + 4 * kk + g];   // A[row t = j][k = g] = C[t][n = 4 kk + g]
      const float bv = Bs[(16 * it + j) * LDS + 4 * kk + g];   // B[k = g][col i = j] = B[i][n = 4 kk + g]
      G = __builtin_amdgcn_mfma_f32_16x16x4f32(av, bv, G, 0, 0, 0);
    }
    *reinterpret_cast<float4*>(out + Sh::kG + w * 256 + 4 * lane) = make_float4(G[0], G[1], G[2], G[3]);   // G[t = 16 tt + 4 g + r][i = 16 it + j]
  }
}

template <int N, int MODE>
__global__ __launch_bounds__(512) void ssd_mfma_kernel(const Dims d, const SsmArgs a, const SsdSeg seg) {
  typedef SsdLds<N> Lds;
  typedef SsdShared<N> Sh;
  constexpr int L = kSsdL, P = kSsdP, NT = N / 16, NC = N / 64;   // NC: 16-byte pieces of B, and of C, per thread
  constexpr int LDB = Lds::LDB, LDT = Lds::LDT, LDX = Lds::LDX, LDM = Lds::LDM;
  extern __shared__ __align__(16) float ssd_smem[];
  float* Bs = ssd_smem + Lds::kB;
  float* Ct = ssd_smem + Lds::kCt;

  const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int hh = w >> 2, wq = w & 3;                   // head of the pair, 16-row slice of the head
  const int g = lane >> 4, j = lane & 15;
  const int h = 2 * blockIdx.x + hh, b = blockIdx.y;
  float* Xs = ssd_smem + Lds::kX + hh * L * LDX;
  float* Ms = ssd_smem + Lds::kM + hh * L * LDM;
  float* dts = ssd_smem + Lds::kDt + hh * L;
  double* cums = reinterpret_cast<double*>(ssd_smem + Lds::kCum) + hh * L;
  const LayerDev& ly = a.one;
  int nt = a.T;
  if (a.n_tok != nullptr) nt = a.n_tok[b];
  if (nt <= 0) return;
  // positions t0 .. t1 - 1 of the pass (seg.len is a multiple of the chunk length)
  const int t0 = MODE == SEG_WALK ? 0 : (int)blockIdx.z * seg.len, t1 = MODE == SEG_WALK ? nt : min(nt, t0 + seg.len);
  if (MODE != SEG_WALK && t0 >= nt) return;
  float* const seg_state = MODE == SEG_WALK ? nullptr : seg.states + (((size_t)b * seg.n + blockIdx.z) * d.Hm + h) * P * N;
  const int pos0 = a.pos0[b];
  float* ring = ly.ring + (size_t)b * d.ring_slots * d.ring_w;
  const size_t rows0 = first_row(a.row0, b, a.T);
  const float* zx = a.zx + rows0 * d.ldzx;
  const float* shared0 = a.ssd_shared + (size_t)b * ssd_chunks(a.T) * Sh::floats(d.Hm);

  // ---- staging, requested a chunk ahead: 4 channels of x (group sg, two positions) with the window before them, pieces of B
  // and C^T, the wavefront's tile of G, and one step size and log-decay sum (the first wavefront: lane / 32 = head of the pair)
  const int sg = tid & 31, sp = 2 * (tid >> 5), xch = 2 * blockIdx.x * P + 4 * sg;
  const int keep = ring_first(d, nt);
  const bool keep_raw = MODE != SEG_LOCAL && a.write_ring;
  ssd_f32x4 bc[NC], cc[NC];
  float4 xr[5], gv = make_float4(0.f, 0.f, 0.f, 0.f), tw[4];
  float dtv = 0.f;
  double cumv = 0.0;
  // (a macro, not a lambda: arrays captured by reference may end up in scratch memory, which waits for the loads)
#define HH_SSD_REQUEST(c0_)                                                                                                          \
  do {                                                                                                                               \
    const float* sh_ = shared0 + (size_t)((c0_) / L) * Sh::floats(d.Hm);                                                             \
    _Pragma("unroll") for (int u = 0; u < 5; ++u) {                                                                                  \
      const int pos_ = pos0 + min((c0_) + sp - 3 + u, nt - 1);                                                                       \
      xr[u] = *reinterpret_cast<const float4*>(pos_ >= pos0 ? zx + (size_t)(pos_ - pos0) * d.ldzx + d.d_inner + xch                  \
                                                            : ring + (size_t)ring_slot(d, pos_) * d.ring_w + xch);                    \
    }                                                                                                                                \
    _Pragma("unroll") for (int i = 0; i < NC; ++i) {                                                                                 \
      bc[i] = *reinterpret_cast<const ssd_f32x4*>(sh_ + Sh::kB + 4 * (tid + 512 * i));                                               \
      if (MODE != SEG_LOCAL) cc[i] = *reinterpret_cast<const ssd_f32x4*>(sh_ + Sh::kCt + 4 * (tid + 512 * i));                       \
    }                                                                                                                                \
    if (MODE != SEG_LOCAL) gv = *reinterpret_cast<const float4*>(sh_ + Sh::kG + min(wq, 2) * 256 + 4 * lane);                        \
    cumv = reinterpret_cast<const double*>(sh_ + Sh::kCum)[2 * blockIdx.x * L + lane];                                               \
    dtv = sh_[Sh::dt(d.Hm) + 2 * blockIdx.x * L + lane];                                                                             \
  } while (0)
  HH_SSD_REQUEST(t0);
#pragma unroll
  for (int q = 0; q < 4; ++q) tw[q] = *reinterpret_cast<const float4*>(ly.conv_w + (size_t)(xch + q) * 4);
  const float4 bias = *reinterpret_cast<const float4*>(ly.conv_b + xch);

  // ---- state slice of this wavefront, transposed: acc[tile][r] = S[16 wq + j][16 tile + 4 g + r]
  ssd_f32x4 S[NT];
  {
    const float* src = a.state_in == 0 ? ly.S : (a.state_in == 1 ? ly.S_draft : nullptr);
    if (MODE == SEG_LOCAL) src = nullptr;
    if (MODE == SEG_OUT || src != nullptr) {
      const float* sp0 = (MODE == SEG_OUT ? seg_state : src + ((size_t)b * d.Hm + h) * P * N) + (16 * wq + j) * N + 4 * g;
#pragma unroll
      for (int t = 0; t < NT; ++t) {
        const float4 v = *reinterpret_cast<const float4*>(sp0 + 16 * t);
        S[t] = ssd_f32x4{v.x, v.y, v.z, v.w};
      }
    } else {
#pragma unroll
      for (int t = 0; t < NT; ++t) S[t] = ssd_f32x4{0.f, 0.f, 0.f, 0.f};
    }
  }
  const float dskip = ly.d_skip[h];
  double total = 0.0;                                  // SEG_LOCAL: log-decay sum of the segment

  TR(0);
  for (int j0 = t0; j0 < t1; j0 += L) {
    const int tc = min(L, t1 - j0);
    if (j0 == 0) TR(1);
#pragma unroll
    for (int u = 0; u < 3; ++u)   // (nothing before the sequence; here, so that nothing waits for the loads any earlier)
      if (pos0 + j0 + sp - 3 + u < 0) xr[u] = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      float4 o;
      ssd_conv4(xr[u], xr[u + 1], xr[u + 2], xr[u + 3], tw, bias, o);
      const int jj = sp + u;
      if (jj >= tc) o = make_float4(0.f, 0.f, 0.f, 0.f);
      *reinterpret_cast<float4*>(ssd_smem + Lds::kX + (sg >> 4) * L * LDX + jj * LDX + 4 * (sg & 15)) = o;
      // the raw inputs stay in the ring for the next pass's window and for rollbacks
      if (jj < tc && keep_raw && j0 + jj >= keep) *reinterpret_cast<float4*>(ring + (size_t)ring_slot(d, pos0 + j0 + jj) * d.ring_w + xch) = xr[u + 3];
    }
#pragma unroll
    for (int i = 0; i < NC; ++i) {
      const int it = tid + 512 * i;
      *reinterpret_cast<ssd_f32x4*>(Bs + it / (N / 4) * LDB + 4 * (it % (N / 4))) = bc[i];
      if (MODE != SEG_LOCAL) *reinterpret_cast<ssd_f32x4*>(Ct + (it >> 3) * LDT + 4 * (it & 7)) = cc[i];
    }
    if (w == 0) {
      ssd_smem[Lds::kDt + lane] = dtv;
      reinterpret_cast<double*>(ssd_smem + Lds::kCum)[lane] = cumv;
    }
    const float G[4] = {gv.x, gv.y, gv.z, gv.w};
    __syncthreads();
    if (j0 == 0) TR(2);
    if (MODE == SEG_LOCAL && j0 + L < t1) HH_SSD_REQUEST(j0 + L);   // the next chunk travels while this one is multiplied

    if (MODE != SEG_LOCAL) {
    // ================= M = G * decay * dt to LDS
    {
      const int tt = wq == 0 ? 0 : 1, it = wq == 2 ? 1 : 0;        // slice 3: the tile above the diagonal is zero
      // lane (g, j) holds G[t = 16 tt' + 4 g + r][i = 16 it' + j]
      const int tt_w = wq == 3 ? 0 : tt, it_w = wq == 3 ? 1 : it;
      const int i = 16 * it_w + j;
      const double ci = cums[i];
      const float di = dts[i];
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int t = 16 * tt_w + 4 * g + r;
        const float m = (wq < 3 && i <= t) ? G[r] * di * expf((float)(cums[t] - ci)) : 0.f;
        Ms[t * LDM + i] = m;
      }
    }
    __syncthreads();
    if (j0 == 0) TR(3);
    if (j0 + L < t1) HH_SSD_REQUEST(j0 + L);   // the next chunk travels while this one is multiplied
    float4 zv[2];                       // and the gates of this one
#pragma unroll
    for (int tt = 0; tt < 2; ++tt)
      zv[tt] = *reinterpret_cast<const float4*>(zx + (size_t)(j0 + min(16 * tt + j, tc - 1)) * d.ldzx + h * P + 16 * wq + 4 * g);

    // ================= read-out of the entering state, intra-chunk product, outputs
    ssd_f32x4 Y[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};   // Y[tt][r] = y[p = 16 wq + 4 g + r][t = 16 tt + j]
    // (operands of the next state tile read while this one is multiplied; left to the compiler, every read is waited for)
    float cr[2][8];
#define HH_SSD_READ_C(t_)                                                                                            \
  _Pragma("unroll") for (int r = 0; r < 4; ++r) {                                                                    \
    const float* crow_ = Ct + (16 * (t_) + 4 * g + r) * LDT + j;   /* B[k = g][col j] = C[position][n = 16 t + 4 g + r] */ \
    cr[(t_) & 1][2 * r] = crow_[0]; cr[(t_) & 1][2 * r + 1] = crow_[16];                                             \
  }
    HH_SSD_READ_C(0);
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      if (t + 1 < NT) HH_SSD_READ_C(t + 1);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        Y[0] = __builtin_amdgcn_mfma_f32_16x16x4f32(S[t][r], cr[t & 1][2 * r], Y[0], 0, 0, 0);
        Y[1] = __builtin_amdgcn_mfma_f32_16x16x4f32(S[t][r], cr[t & 1][2 * r + 1], Y[1], 0, 0, 0);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
#undef HH_SSD_READ_C
    {
      const float e0 = expf((float)cums[j]), e1 = expf((float)cums[16 + j]);
#pragma unroll
      for (int r = 0; r < 4; ++r) { Y[0][r] *= e0; Y[1][r] *= e1; }
    }
#pragma unroll
    for (int kk = 0; kk < L / 4; ++kk) {
      const float xv = Xs[(4 * kk + g) * LDX + 16 * wq + j];       // A[row p = j][k = g] = x[i = 4 kk + g][p]
      if (kk < 4) Y[0] = __builtin_amdgcn_mfma_f32_16x16x4f32(xv, Ms[j * LDM + 4 * kk + g], Y[0], 0, 0, 0);
      Y[1] = __builtin_amdgcn_mfma_f32_16x16x4f32(xv, Ms[(16 + j) * LDM + 4 * kk + g], Y[1], 0, 0, 0);
    }
#pragma unroll
    for (int tt = 0; tt < 2; ++tt) {
      const int t = 16 * tt + j;
      if (t < tc) {
        const size_t m = rows0 + j0 + t;
        const int p = 16 * wq + 4 * g;
        const float4 xv = *reinterpret_cast<const float4*>(Xs + t * LDX + p);
        const float4 z = zv[tt];
        float4 o;
        o.x = (Y[tt][0] + dskip * xv.x) * fast_silu(z.x);
        o.y = (Y[tt][1] + dskip * xv.y) * fast_silu(z.y);
        o.z = (Y[tt][2] + dskip * xv.z) * fast_silu(z.z);
        o.w = (Y[tt][3] + dskip * xv.w) * fast_silu(z.w);
        *reinterpret_cast<float4*>(a.g + m * d.d_inner + h * P + p) = o;
      }
    }

    }
    if (j0 == 0) TR(4);
    // ================= state update: S' = exp(cum_L) S + sum_i w_i x_i (outer) B_i
    if (MODE != SEG_OUT || j0 + L < t1) {
      const double cl = cums[L - 1];
      const float el = expf((float)cl);
      total += cl;
#pragma unroll
      for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int r = 0; r < 4; ++r) S[t][r] *= el;
      float xw[L / 4];
#pragma unroll
      for (int kk = 0; kk < L / 4; ++kk) {             // B[k = g][col p = j]
        const int i = 4 * kk + g;
        xw[kk] = Xs[i * LDX + 16 * wq + j] * (dts[i] * expf((float)(cl - cums[i])));
      }
      float br[2][NT];
#define HH_SSD_READ_B(kk_)                                                                               \
  _Pragma("unroll") for (int t = 0; t < NT; ++t) br[(kk_) & 1][t] = Bs[(4 * (kk_) + g) * LDB + j + 16 * t]   // A[row n = j][k = g] = B[i][n]
      HH_SSD_READ_B(0);
#pragma unroll
      for (int kk = 0; kk < L / 4; ++kk) {
        if (kk + 1 < L / 4) HH_SSD_READ_B(kk + 1);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int t = 0; t < NT; ++t) S[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(br[kk & 1][t], xw[kk], S[t], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
      }
#undef HH_SSD_READ_B
    }
    __syncthreads();
    if (j0 == 0) TR(5);
  }
  TR(6);

  if (MODE == SEG_LOCAL && wq == 0 && lane == 0) seg.decay[((size_t)b * seg.n + blockIdx.z) * d.Hm + h] = (float)total;
  if (MODE == SEG_LOCAL || (MODE == SEG_WALK && a.state_out != 0)) {
    float* dp = (MODE == SEG_LOCAL ? seg_state : (a.state_out == 1 ? ly.S : ly.S_draft) + ((size_t)b * d.Hm + h) * P * N) + (16 * wq + j) * N + 4 * g;
#pragma unroll
    for (int t = 0; t < NT; ++t) *reinterpret_cast<float4*>(dp + 16 * t) = make_float4(S[t][0], S[t][1], S[t][2], S[t][3]);
  }
  TR(7);
#undef HH_SSD_REQUEST
}

// Chains the segments of a pass: the state entering segment q+1 is exp(decay_q) times the one entering q plus what
// segment q adds.  A thread owns 4 elements of one sequence's state; the segments' contributions are replaced by the
// states that enter them, and the state behind the last one becomes the sequence's state.
__global__ __launch_bounds__(256) void ssd_combine_kernel(const Dims d, const SsmArgs a, const SsdSeg seg) {
  const int b = blockIdx.y;
  int nt = a.T;
  if (a.n_tok != nullptr) nt = a.n_tok[b];
  if (nt <= 0) return;
  const int ns = (nt + seg.len - 1) / seg.len, per_head = d.P * d.N;
  const size_t at = ((size_t)blockIdx.x * 256 + threadIdx.x) * 4, state = (size_t)d.Hm * per_head;   // per_head % 1024 == 0
  const int h = (int)((size_t)blockIdx.x * 1024 / per_head);
  const LayerDev& ly = a.one;
  const float* src = a.state_in == 0 ? ly.S : (a.state_in == 1 ? ly.S_draft : nullptr);
  float4 s = make_float4(0.f, 0.f, 0.f, 0.f);
  if (src != nullptr) s = *reinterpret_cast<const float4*>(src + (size_t)b * state + at);
  float* p = seg.states + (size_t)b * seg.n * state + at;
  const float* dec = seg.decay + (size_t)b * seg.n * d.Hm + h;
  for (int q0 = 0; q0 < ns; q0 += 8) {
    float4 v[8];
    float e[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int q = min(q0 + u, ns - 1);
      v[u] = *reinterpret_cast<const float4*>(p + (size_t)q * state);
      e[u] = dec[(size_t)q * d.Hm];
    }
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      if (q0 + u >= ns) break;
      *reinterpret_cast<float4*>(p + (size_t)(q0 + u) * state) = s;
      const float f = expf(e[u]);
      s.x = fmaf(f, s.x, v[u].x); s.y = fmaf(f, s.y, v[u].y); s.z = fmaf(f, s.z, v[u].z); s.w = fmaf(f, s.w, v[u].w);
    }
  }
  float* dst = a.state_out == 1 ? ly.S : (a.state_out == 2 ? ly.S_draft : nullptr);
  if (dst != nullptr) *reinterpret_cast<float4*>(dst + (size_t)b * state + at) = s;
}

template <int N, int MODE>
static hipError_t ssd_launch_mode(const Dims& d, const SsmArgs& a, const SsdSeg& seg, hipStream_t s) {
  auto kern = ssd_mfma_kernel<N, MODE>;
  constexpr int lds = SsdLds<N>::kFloats * (int)sizeof(float);
  static bool enabled = false;
  if (!enabled && lds > 48 * 1024) {
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, lds);
    if (e != hipSuccess) return e;
    enabled = true;
  }
  hipLaunchKernelGGL(kern, dim3(d.Hm / 2, a.B, MODE == SEG_WALK ? 1 : seg.n), dim3(512), lds, s, d, a, seg);
  return hipGetLastError();
}
template <int N>
static hipError_t ssd_launch(const Dims& d, const SsmArgs& a, const SsdSeg& seg, hipStream_t s) {
  hipLaunchKernelGGL(ssd_shared_kernel<N>, dim3(ssd_chunks(a.T), a.B), dim3(512), 0, s, d, a);
  if (hipError_t e = hipGetLastError(); e != hipSuccess) return e;
  if (seg.n <= 1) return ssd_launch_mode<N, SEG_WALK>(d, a, seg, s);
  hipError_t e = ssd_launch_mode<N, SEG_LOCAL>(d, a, seg, s);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(ssd_combine_kernel, dim3(d.Hm * d.P * d.N / 1024, a.B), dim3(256), 0, s, d, a, seg);
  e = hipGetLastError();
  if (e != hipSuccess) return e;
  return ssd_launch_mode<N, SEG_OUT>(d, a, seg, s);
}

// When the segmented form is taken.  Fewer than 128 workgroups (sequence, pair of heads) leave half the chip idle in a
// walk, and the position-by-position kernel that served them is a serial chain of 0.36 us (0.5B shape) or 0.59 us (3B
// shape) per position.  As many segments as give kSegWorkgroups workgroups (half of them at state size 256), at least one chunk
// each.  One workgroup of 8 wavefronts is resident per compute unit at a time (108 to 248 registers; two would need 128, and at
// state size 256 the staged chunk takes 101 KB of LDS as well), so that 512 of them are up to two rounds: what was measured.  One sequence, pass of 512 positions: 0.5B shape
// 186 -> 38 us (shared inputs 9.0, segments 10.5, chaining 6.9, outputs 11.9), 3B shape 300 -> 90 us before the inputs were shared; prefill of 509 tokens at the 0.5B shape
// 13.8 -> 8.7 ms, of 4096 tokens through four 3B blocks 20.8 -> 15.0 ms, 8 sequences of 512 at 12 0.5B blocks 11.2 -> 9.7.
// The local pass repeats the staging and the state products, so at state size 256 fewer than three segments give nothing
// (6 sequences at the 3B shape: 4.22 against 4.20 ms with the position-by-position kernel).  From 96 positions on the
// three launches pay (100 positions: 5 % per prefill at either shape); below, the chain is short enough.
static constexpr int kSegWorkgroups = 512, kSegMinT = 96;

static bool ssd_shape(const Dims& d) {
  return d.P == kSsdP && d.Hm % 2 == 0 && d.d_inner % 4 == 0 && d.ldzx % 4 == 0 && d.ring_w % 4 == 0 && d.conv_dim % 4 == 0 &&
         (d.N == 64 || d.N == 128 || d.N == 256);
}
static int seg_workgroups(const Dims& d) { return d.N == 256 ? kSegWorkgroups / 2 : kSegWorkgroups; }
static SsdSeg ssd_segments(const Dims& d, int B, int T) {
  SsdSeg seg{nullptr, nullptr, 0, 1};
  const int wgs = (d.Hm / 2) * B, chunks = (T + kSsdL - 1) / kSsdL;
  const int most = seg_workgroups(d) / wgs;
  if (wgs >= 128 || T < kSegMinT || most < (d.N == 256 ? 3 : 2)) return seg;
  const int per = (chunks + most - 1) / most;      // chunks per segment
  seg.len = per * kSsdL;
  seg.n = (chunks + per - 1) / per;
  return seg;
}
// floats of scratch for the segment states of any pass of this context
size_t ssd_segment_elems(const Dims& d) {
  if (!ssd_shape(d) || d.Tmax < kSegMinT) return 0;
  size_t most = 0;
  for (int B = 1; B <= d.Bmax && (d.Hm / 2) * B < 128; ++B) {
    const size_t n = std::min((size_t)seg_workgroups(d) / ((d.Hm / 2) * B), (size_t)(d.Tmax + kSsdL - 1) / kSsdL);
    most = std::max(most, (size_t)B * n * d.Hm * ((size_t)d.P * d.N + 1));
  }
  return most;
}

// floats of scratch for what the heads of a pass share
size_t ssd_shared_elems(const Dims& d) {
  if (!ssd_shape(d) || d.Tmax < kSsdMinT) return 0;
  const size_t per = d.N == 64 ? SsdShared<64>::floats(d.Hm) : d.N == 128 ? SsdShared<128>::floats(d.Hm) : SsdShared<256>::floats(d.Hm);
  return (size_t)d.Bmax * ssd_chunks(d.Tmax) * per;
}

// true if the pass was taken by the matmul-form kernel: a single layer's pass over this call's
// projections with outputs, at least 16 positions, an even number of heads of dimension 64, state size 64, 128 or 256,
// 16-byte aligned rows
bool launch_ssd_mfma(const Dims& d, const SsmArgs& a, hipStream_t s, hipError_t* err) {
  if ((d.flags & HH_KF_SSM_SEQUENTIAL) || a.layers != nullptr || a.zx == nullptr || a.g == nullptr || a.n_acc != nullptr ||
      a.skip != nullptr || a.ssd_shared == nullptr || a.T < kSsdMinT || !ssd_shape(d) || (reinterpret_cast<uintptr_t>(a.zx) & 15) != 0 || (reinterpret_cast<uintptr_t>(a.g) & 15) != 0)
    return false;
  SsdSeg seg{nullptr, nullptr, 0, 1};
  if ((d.Hm / 2) * a.B < 128 && !(d.flags & HH_KF_SSM_MATMUL)) {
    seg = ssd_segments(d, a.B, a.T);
    if (seg.n < 2 || a.seg_scratch == nullptr) return false;
    seg.states = a.seg_scratch;
    seg.decay = a.seg_scratch + (size_t)a.B * seg.n * d.Hm * d.P * d.N;
  }
  switch (d.N) {
    case 64: *err = ssd_launch<64>(d, a, seg, s); return true;
    case 128: *err = ssd_launch<128>(d, a, seg, s); return true;
    case 256: *err = ssd_launch<256>(d, a, seg, s); return true;
  }
  return false;
}

}  // namespace hh
