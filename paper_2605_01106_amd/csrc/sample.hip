// Token choice at temperature T > 0 (Section 3.3, Eq. 6 of the paper): draws from
// softmax(logits / T) for the draft steps and for the first token, and the rejection test of
// the round with its correction token drawn from norm(max(0, P_H - P_S)).
//
// A draw from unnormalised masses p_0 .. p_{V-1} with a uniform u is the inverse CDF in index
// order: the smallest i with p_0 + .. + p_i > u * sum(p).  The uniforms are 24-bit values of a
// counter-based generator: output number c of SplitMix64 (Steele, Lea, Flood 2014) started at
// the caller's seed, c = sequence * 2^34 + stream position * 4 + purpose (0 draft draw,
// 1 acceptance test, 2 correction / bonus / first token), so any decision can be recomputed alone.
//
// The outcome of a round is written in the form the commit step already consumes: targets[i] =
// drafts[i] for the kept positions, targets[n] = the emitted token, later entries -1; the
// longest-matching-prefix rule then returns n, because the residual has no mass at a rejected draft.
#include <mutex>

#include "hh_internal.h"
#include "wave_ops.h"

namespace hh {
namespace {

constexpr int kDrawThreads = 1024;
constexpr int kDrawWaves = kDrawThreads / 64;

__device__ __forceinline__ uint64_t splitmix64_at(uint64_t seed, uint64_t counter) {
  uint64_t z = seed + (counter + 1) * 0x9E3779B97F4A7C15ull;
  z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
  z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
  return z ^ (z >> 31);
}

__device__ __forceinline__ float uniform24(uint64_t seed, int b, int idx, int purpose) {
  const uint64_t c = (static_cast<uint64_t>(b) << 34) + (static_cast<uint64_t>(idx) << 2) + static_cast<uint64_t>(purpose);
  return static_cast<float>(splitmix64_at(seed, c) >> 40) * 0x1p-24f;
}

// Over the 64 lanes, left in every lane, in the order lane ^ 32, 16, 8, 4, 2, 1, on the vector unit (a shuffle through LDS is
// a round trip of its own): the row swaps give both halves, and a rotation by 8 or 4 inside a row of 16 is lane ^ 8 or 4 once the
// lanes ^ 8 agree.
template <typename F>
__device__ __forceinline__ float wave_combine(float v, F f) {
  const uint32_t x = __float_as_uint(v);
  const auto s32 = __builtin_amdgcn_permlane32_swap(x, x, false, false);
  v = f(__uint_as_float(s32[0]), __uint_as_float(s32[1]));
  const uint32_t y = __float_as_uint(v);
  const auto s16 = __builtin_amdgcn_permlane16_swap(y, y, false, false);
  v = f(__uint_as_float(s16[0]), __uint_as_float(s16[1]));
  v = f(v, dpp_move<0x128>(v));   // row_ror:8
  v = f(v, dpp_move<0x124>(v));   // row_ror:4
  v = f(v, dpp_move<0x4E>(v));    // quad_perm [2,3,0,1]
  return f(v, dpp_move<0xB1>(v)); // quad_perm [1,0,3,2]
}
__device__ __forceinline__ float wave_max(float v) {
  return wave_combine(v, [](float p, float q) { return fmaxf(p, q); });
}
__device__ __forceinline__ float wave_sum(float v) {
  return wave_combine(v, [](float p, float q) { return p + q; });
}

// softmax(l / T) entry from the row's maximum m and 1 / sum: the one expression every kernel here uses,
// so that a probability computed in two places has the same bits.  The product is rounded on its own
// (never contracted into a following subtraction: fma(a, b, -round(a * b)) is the rounding error of
// the product, which would give the residual of two identical distributions a noise mass).
__device__ __forceinline__ float prob(float l, float m, float inv_t, float rsum) {
#pragma clang fp contract(off)
  return expf((l - m) * inv_t) * rsum;
}
// max(0, P_H - P_S) of one entry, the subtraction kept apart from the two products
__device__ __forceinline__ float residual_mass(float ph, float ps) {
#pragma clang fp contract(off)
  const float d = ph - ps;
  return fmaxf(0.f, d);
}

constexpr float kNoLogit = -3.0e38f;   // stands for an entry past the end of the row: exp((kNoLogit - m) / T) = 0

// entries jj .. jj+3 of a row (jj a multiple of 4); past `end` they read as kNoLogit.  vec: the row
// starts on a 16-byte boundary
__device__ __forceinline__ void load_group(const float* __restrict__ row, int jj, int end, bool vec, float (&l)[4]) {
  if (vec && jj + 3 < end) {
    const float4 t = *reinterpret_cast<const float4*>(row + jj);
    l[0] = t.x; l[1] = t.y; l[2] = t.z; l[3] = t.w;
  } else {
    for (int e = 0; e < 4; ++e) l[e] = jj + e < end ? row[jj + e] : kNoLogit;
  }
}
__device__ __forceinline__ bool row_is_vec(const float* row) { return (reinterpret_cast<uintptr_t>(row) & 15) == 0; }

// max over the row, by a whole workgroup; `red` holds blockDim.x / 64 floats
__device__ float row_max(const float* __restrict__ row, int V, float* red) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, nw = blockDim.x >> 6;
  const bool vec = row_is_vec(row);
  float m = kNoLogit;
#pragma unroll 4
  for (int j = threadIdx.x * 4; j < V; j += blockDim.x * 4) {
    float l[4];
    load_group(row, j, V, vec, l);
    m = fmaxf(fmaxf(m, fmaxf(l[0], l[1])), fmaxf(l[2], l[3]));
  }
  m = wave_max(m);
  if (lane == 0) red[w] = m;
  __syncthreads();
  m = red[0];
  for (int i = 1; i < nw; ++i) m = fmaxf(m, red[i]);
  __syncthreads();
  return m;
}

// max over the row and sum of exp((l - max) / T), by a whole workgroup; `red` holds blockDim.x / 64 floats
__device__ void row_stats(const float* __restrict__ row, int V, float inv_t, float* red, float& m_out, float& s_out) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, nw = blockDim.x >> 6;
  const bool vec = row_is_vec(row);
  const float m = row_max(row, V, red);
  float s = 0.f;
#pragma unroll 4
  for (int j = threadIdx.x * 4; j < V; j += blockDim.x * 4) {
    float l[4];
    load_group(row, j, V, vec, l);
    s += (expf((l[0] - m) * inv_t) + expf((l[1] - m) * inv_t)) + (expf((l[2] - m) * inv_t) + expf((l[3] - m) * inv_t));
  }
  s = wave_sum(s);
  if (lane == 0) red[w] = s;
  __syncthreads();
  s = 0.f;
  for (int i = 0; i < nw; ++i) s += red[i];
  __syncthreads();
  m_out = m; s_out = s;
}

// ---- rows held in registers.  A row of up to 65536 entries that starts on a 16-byte boundary and whose length is a
// multiple of 4 is read once, with all loads of a thread in flight together, where the loops above and below read it two
// or three times, a dependent load per pass of a loop.  Same sums in the same order, so the same bits.  Draw from 64 rows
// of 1000 entries 5.7 -> 5.0 us, of 4096 6.4 -> 5.5, of 32768 16.4 -> 10.5, of 65536 28.4 -> 15.0; acceptance of 64 sequences
// at k = 8 over 4096 entries 21 -> 14 us, over 32768 70 -> 40 (statistics of two rows on a compute unit at a time: at most 64
// registers), over 65536 130 -> 96: the statistics 74 us for 285 MB, 3.8 TB/s (a plain sum of 2 GiB reads 4.0; the next row
// requested behind the exponentials of this one takes 74 as well, with 17 registers spilled, and its scratch memory makes the
// call 7 us longer), then 22 us on one compute unit per sequence, two rows of 256 KB and 131072 exponentials each.  The draw with
// the residual keeps sums only there: 64 registers of masses spill behind the two exponentials per entry.
constexpr int kRegGroups = 16;   // groups of 4 entries per thread at most: 64 registers, one workgroup of 16 wavefronts per compute unit
__host__ __device__ constexpr int reg_vocab(int groups) { return groups * kDrawThreads * 4; }

// groups first, first + step, ... of a row (past its end: its last group, to be ignored)
template <int G>
__device__ __forceinline__ void load_groups(const float* __restrict__ row, int V, int first, int step, float4 (&l)[G]) {
#pragma unroll
  for (int i = 0; i < G; ++i) l[i] = *reinterpret_cast<const float4*>(row + min(first + i * step, V - 4));
}

// row_stats for such a row
template <int G>
__device__ void row_stats_regs(const float* __restrict__ row, int V, float inv_t, float* red, float& m_out, float& s_out) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, nw = kDrawWaves, j0 = threadIdx.x * 4;
  float4 l[G];
  load_groups(row, V, j0, kDrawThreads * 4, l);
  float m = kNoLogit;
#pragma unroll
  for (int i = 0; i < G; ++i) m = fmaxf(fmaxf(m, fmaxf(l[i].x, l[i].y)), fmaxf(l[i].z, l[i].w));
  m = wave_max(m);
  if (lane == 0) red[w] = m;
  __syncthreads();
  m = red[0];
  for (int i = 1; i < nw; ++i) m = fmaxf(m, red[i]);
  __syncthreads();
  float s = 0.f;
#pragma unroll
  for (int i = 0; i < G; ++i) {
    if (j0 + i * kDrawThreads * 4 < V)
      s += (expf((l[i].x - m) * inv_t) + expf((l[i].y - m) * inv_t)) + (expf((l[i].z - m) * inv_t) + expf((l[i].w - m) * inv_t));
  }
  s = wave_sum(s);
  if (lane == 0) red[w] = s;
  __syncthreads();
  s = 0.f;
  for (int i = 0; i < nw; ++i) s += red[i];
  m_out = m; s_out = s;
}

// A block of 256 entries in a wavefront: the lane's four masses, the running sum up to and with them, the last index with mass
// among them (-1: none).
struct WalkBlock { int jj, last; float v[4], incl; };
template <typename F>
__device__ __forceinline__ WalkBlock walk_block(int jj, int end, F val) {
  const int lane = threadIdx.x & 63;
  WalkBlock k;
  k.jj = jj; k.last = -1;
  val(jj, end, k.v);
  float t = 0.f;
  for (int e = 0; e < 4; ++e) {
    t += k.v[e];
    if (k.v[e] > 0.f) k.last = jj + e;
  }
  k.incl = t;
  for (int o = 1; o < 64; o <<= 1) {
    const float up = __shfl_up(k.incl, o);
    if (lane >= o) k.incl += up;
  }
  return k;
}
// The index drawn from a block that some lane's running sum says holds it (hit: those lanes; carry: the mass before the block;
// prev_mass: the last index with mass before it), by the whole wavefront.
__device__ __forceinline__ int pick_in_block(const WalkBlock& k, unsigned long long hit, float carry, float target, int prev_mass, int end) {
  const int lane = threadIdx.x & 63;
  float excl = __shfl_up(k.incl, 1);
  if (lane == 0) excl = 0.f;
  const int fl = __ffsll(hit) - 1;
  int r = -1;
  if (lane == fl) {
    float c2 = carry + excl;
    for (int e = 0; e < 4; ++e) {
      c2 += k.v[e];
      if (r < 0 && k.v[e] > 0.f && c2 > target) r = k.jj + e;
    }
    if (r < 0) r = k.last;
  }
  r = __shfl(r, fl);
  if (r < 0) {   // the lane's own walk fell short by rounding and it holds no mass: nearest mass before it
    int prev = lane < fl ? k.last : -1;
    for (int o = 32; o > 0; o >>= 1) prev = max(prev, __shfl_xor(prev, o));
    r = prev >= 0 ? prev : prev_mass;
    if (r < 0) r = min(k.jj, end - 1);
    r = __shfl(r, fl);
  }
  return r;
}

// Inverse-CDF draw by a workgroup of kDrawThreads threads.  val(jj, end, v) fills v[0..3] with the
// masses (>= 0) of indices jj .. jj+3, zero past `end`.
// Wavefront w owns the contiguous segment [w * seg, (w + 1) * seg); the segment sums give the
// segment that holds u * total, which is scanned in index order in blocks of 256 entries, a block per wavefront (one
// wavefront alone walked up to 16 blocks, a round trip and a scan each: draw from 64 rows of 32768 entries 12.0 -> 10.5 us,
// of 65536 20.9 -> 15.0; acceptance over 65536 entries, 8 sequences, k = 1, 42 -> 34).
// red: kDrawWaves floats, res: one int (both in LDS).  Every thread returns the drawn index, or -1
// when no entry has mass.
// draw_walk: the part behind the segment sums (acc: this thread's share of its wavefront's segment); prepare() is called
// by the wavefront that owns the segment, before the first val.
__device__ __forceinline__ int segment_size(int V) { return ((V + kDrawWaves * 256 - 1) / (kDrawWaves * 256)) * 256; }

template <typename P, typename F>
__device__ int draw_walk(float acc, P prepare, F val, int V, float u, float* red, int* res) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int seg = segment_size(V);
  acc = wave_sum(acc);
  if (lane == 0) red[w] = acc;
  __syncthreads();
  float total = 0.f;
  for (int i = 0; i < kDrawWaves; ++i) total += red[i];
  if (!(total > 0.f)) {          // uniform over the workgroup: every thread summed the same values
    __syncthreads();
    return -1;
  }
  const float target = u * total;
  int ws = -1;
  float carry = 0.f, c = 0.f;
  for (int i = 0; i < kDrawWaves; ++i) {
    const float nx = c + red[i];
    if (ws < 0 && nx > target) { ws = i; carry = c; }
    c = nx;
  }
  if (ws < 0) {   // u * total rounded up to the total: the last segment that has mass
    ws = 0;
    c = 0.f;
    for (int i = 0; i < kDrawWaves; ++i) {
      if (red[i] > 0.f) { ws = i; carry = c; }
      c += red[i];
    }
  }
  const int s0 = min(V, ws * seg), s1 = min(V, s0 + seg), n_blk = (s1 - s0 + 255) >> 8;
  int last_mass = -1;        // last index with mass before the block in hand (the answer if rounding hides the crossing)
  // Rows of up to 16384 entries: the owner alone, without the two barriers per round below (one row of 16000 entries 6.5 -> 5.7 us,
  // acceptance of one sequence at k = 2 10.8 -> 9.7; at 20000, five blocks, 7.7 -> 7.1 and 15.0 -> 14.1 with one row, but with 64
  // 8.2 -> 8.6 and 18.8 -> 19.1).
  if (n_blk <= 4) {
    if (w == ws) {
      prepare();
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
      int result = -1;
      for (int q = 0; q < n_blk && result < 0; ++q) {
        const WalkBlock k = walk_block(s0 + q * 256 + lane * 4, s1, val);
        const unsigned long long hit = __ballot(carry + k.incl > target);
        if (hit != 0ull) {
          result = pick_in_block(k, hit, carry, target, last_mass, s1);
        } else {
          carry += __shfl(k.incl, 63);
          const unsigned long long massy = __ballot(k.last >= 0);
          if (massy != 0ull) last_mass = __shfl(k.last, 63 - __clzll(massy));
        }
      }
      if (result < 0) result = last_mass >= 0 ? last_mass : max(s1 - 1, 0);
      if (lane == 0) *res = result;
    }
    __syncthreads();
    const int out = *res;
    __syncthreads();
    return out;
  }
  if (w == ws) prepare();
  __shared__ float blk_sum[kDrawWaves];      // of the blocks of a round: mass,
  __shared__ int blk_last[kDrawWaves];       // last index with mass (-1: none),
  __shared__ int blk_hit[kDrawWaves];        // whether u * total lies in the block
  __syncthreads();
  int first = -1;
  for (int b0 = 0; b0 < n_blk && first < 0; b0 += kDrawWaves) {
    WalkBlock k{};
    k.last = -1;
    if (b0 + w < n_blk) k = walk_block(s0 + (b0 + w) * 256 + lane * 4, s1, val);      // (uniform over the wavefront)
    const unsigned long long massy = __ballot(k.last >= 0);
    if (lane == 63) blk_sum[w] = k.incl;
    if (lane == (massy != 0ull ? 63 - __clzll(massy) : 0)) blk_last[w] = k.last;
    __syncthreads();
    // lane i of every wavefront holds block i's values; the sums are added in block order
    const float bs = lane < kDrawWaves ? blk_sum[lane] : 0.f;
    const int bl = lane < kDrawWaves ? blk_last[lane] : -1;
    float cw = carry;                        // mass before this wavefront's block
#pragma unroll
    for (int i = 0; i < kDrawWaves; ++i) {
      if (i == w) cw = carry;
      carry += __int_as_float(__builtin_amdgcn_readlane(__float_as_int(bs), i));   // (blocks past the segment's end hold nothing)
    }
    const unsigned long long hit = __ballot(cw + k.incl > target);
    if (lane == 0) blk_hit[w] = hit != 0ull && b0 + w < n_blk;
    __syncthreads();
    const unsigned long long hits = __ballot(lane < kDrawWaves && blk_hit[lane] != 0);
    if (hits != 0ull) first = __ffsll(hits) - 1;
    const unsigned long long with_mass = __ballot(bl >= 0), before = with_mass & ((1ull << w) - 1);
    const int prev_mass = before != 0ull ? __shfl(bl, 63 - __clzll(before)) : last_mass;
    if (with_mass != 0ull) last_mass = __shfl(bl, 63 - __clzll(with_mass));
    if (first == w) {
      const int r = pick_in_block(k, hit, cw, target, prev_mass, s1);
      if (lane == 0) *res = r;
    }
    __syncthreads();
  }
  // (every thread has read the same flags, so that they agree on the branch and on last_mass)
  return first >= 0 ? *res : last_mass >= 0 ? last_mass : max(s1 - 1, 0);
}

template <typename F>
__device__ int block_draw(F val, int V, float u, float* red, int* res) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int seg = segment_size(V);
  const int j0 = min(V, w * seg), j1 = min(V, j0 + seg);
  float acc = 0.f;
#pragma unroll 4
  for (int j = j0 + lane * 4; j < j1; j += 256) {
    float v[4];
    val(j, j1, v);
    acc += (v[0] + v[1]) + (v[2] + v[3]);
  }
  return draw_walk(acc, [] {}, val, V, u, red, res);
}

// The same for masses in registers: mass[i] holds entries j0 + 256 i + 4 lane .. + 3 of the wavefront's segment, zero past
// its end (V <= reg_vocab(G): the segment has at most G blocks of 256).  The wavefront whose segment is scanned puts
// its masses in LDS first (walk: 256 * G floats).
template <int G>
__device__ int block_draw_regs(const float4 (&mass)[G], int V, float u, float* walk, float* red, int* res) {
  const int lane = threadIdx.x & 63;
  const int seg = segment_size(V);
  float acc = 0.f;
#pragma unroll
  for (int i = 0; i < G; ++i) acc += (mass[i].x + mass[i].y) + (mass[i].z + mass[i].w);   // (adding a zero past the end keeps the bits)
  return draw_walk(
      acc,
      [&] {
#pragma unroll
        for (int i = 0; i < G; ++i) *reinterpret_cast<float4*>(walk + i * 256 + 4 * lane) = mass[i];
      },
      [&](int jj, int, float (&v)[4]) {      // (the segment starts at a multiple of its size)
        const float4 t = *reinterpret_cast<const float4*>(walk + jj % seg);
        v[0] = t.x; v[1] = t.y; v[2] = t.z; v[3] = t.w;
      },
      V, u, red, res);
}

// masses exp((l - m) / T) of the wavefront's segment from its logits, in place
template <int G>
__device__ __forceinline__ void softmax_masses(float4 (&l)[G], int V, float m, float inv_t) {
  const int seg = segment_size(V), j0 = min(V, (int)(threadIdx.x >> 6) * seg), j1 = min(V, j0 + seg), lane = threadIdx.x & 63;
#pragma unroll
  for (int i = 0; i < G; ++i) {
    const bool on = j0 + i * 256 + 4 * lane < j1;
    l[i] = on ? make_float4(expf((l[i].x - m) * inv_t), expf((l[i].y - m) * inv_t), expf((l[i].z - m) * inv_t), expf((l[i].w - m) * inv_t))
              : make_float4(0.f, 0.f, 0.f, 0.f);
  }
}

// One row per workgroup: token drawn from softmax(row / T).  G > 0: the row in registers (see above), G = 0: any row.
template <int G>
__global__ __launch_bounds__(kDrawThreads) void sample_rows_kernel(const float* __restrict__ logits, size_t row_stride, int V,
                                                                    const SamplingParams* __restrict__ prm_dev,
                                                                    const SamplingParams prm_val,
                                                                    const int* __restrict__ idx_base, int idx_off,
                                                                    int purpose, int* __restrict__ out, int out_stride,
                                                                    int out_off) {
  __shared__ float red[kDrawWaves];
  __shared__ int res;
  __shared__ __align__(16) float walk[G > 0 ? 256 * G : 4];
  const int b = blockIdx.x;
  const float* row = logits + static_cast<size_t>(b) * row_stride;
  const SamplingParams prm = prm_dev ? *prm_dev : prm_val;
  const float inv_t = prm.inv_t;
  const int idx = (idx_base ? idx_base[b] : 0) + idx_off;
  int tok;
  if constexpr (G > 0) {
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    float4 l[G];
    load_groups(row, V, min(V, w * segment_size(V)) + 4 * lane, 256, l);   // (entries past the segment belong to the row: they may count in the maximum)
    float m = kNoLogit;
#pragma unroll
    for (int i = 0; i < G; ++i) m = fmaxf(fmaxf(m, fmaxf(l[i].x, l[i].y)), fmaxf(l[i].z, l[i].w));
    m = wave_max(m);
    if (lane == 0) red[w] = m;
    __syncthreads();
    m = red[0];
    for (int i = 1; i < kDrawWaves; ++i) m = fmaxf(m, red[i]);
    __syncthreads();
    softmax_masses(l, V, m, inv_t);
    tok = block_draw_regs(l, V, uniform24(prm.seed, b, idx, purpose), walk, red, &res);
  } else {
    const bool vec = row_is_vec(row);
    const float m = row_max(row, V, red);
    const float u = uniform24(prm.seed, b, idx, purpose);
    tok = block_draw(
        [&](int jj, int end, float (&v)[4]) {
          float l[4];
          load_group(row, jj, end, vec, l);
          for (int e = 0; e < 4; ++e) v[e] = expf((l[e] - m) * inv_t);
        },
        V, u, red, &res);
  }
  if (threadIdx.x == 0) out[static_cast<size_t>(b) * out_stride + out_off] = tok;
}

// (max, sum) of the k draft rows and the k + 1 verification rows of every sequence:
// stats[b][r][2], r < kmax: draft row r; r >= kmax: verification row r - kmax.
// grid: x = rows of a sequence, y = sequences
template <int G>
__global__ __launch_bounds__(kDrawThreads) void softmax_stats_kernel(const float* __restrict__ logits_d,
                                                            const float* __restrict__ logits_v, int V, int k, int kmax,
                                                            const SamplingParams* __restrict__ prm_dev,
                                                            const SamplingParams prm_val, float* __restrict__ stats) {
  __shared__ float red[kDrawWaves];
  const int r = blockIdx.x, b = blockIdx.y;
  const float* row;
  int slot;
  if (r < k) { row = logits_d + (static_cast<size_t>(b) * kmax + r) * V; slot = r; }
  else { row = logits_v + (static_cast<size_t>(b) * (k + 1) + (r - k)) * V; slot = kmax + (r - k); }
  float m, s;
  const float inv_t = prm_dev ? prm_dev->inv_t : prm_val.inv_t;
  if constexpr (G > 0) row_stats_regs<G>(row, V, inv_t, red, m, s);
  else row_stats(row, V, inv_t, red, m, s);
  if (threadIdx.x == 0) {
    float* st = stats + (static_cast<size_t>(b) * (2 * kmax + 1) + slot) * 2;
    st[0] = m; st[1] = s;
  }
}

// The round's acceptance for one sequence per workgroup (Eq. 6) and its targets row.
template <int G>
__global__ __launch_bounds__(kDrawThreads) void spec_targets_kernel(const float* __restrict__ logits_d,
                                                                     const float* __restrict__ logits_v, int V, int k,
                                                                     int kmax, const SamplingParams* __restrict__ prm_dev,
                                                                     const SamplingParams prm_val,
                                                                     const float* __restrict__ stats,
                                                                     const int* __restrict__ drafts,
                                                                     const int* __restrict__ committed,
                                                                     int* __restrict__ targets) {
  __shared__ float red[kDrawWaves];
  __shared__ int res;
  __shared__ int n_sh;
  __shared__ __align__(16) float walk[G > 0 && G <= 8 ? 256 * G : 4];
  const int b = blockIdx.x;
  const SamplingParams prm = prm_dev ? *prm_dev : prm_val;
  const float inv_t = prm.inv_t;
  const uint64_t seed = prm.seed;
  const int base = committed[b];
  const int* d = drafts + static_cast<size_t>(b) * kmax;
  const float* st = stats + static_cast<size_t>(b) * (2 * kmax + 1) * 2;
  const float* rows_d = logits_d + static_cast<size_t>(b) * kmax * V;
  const float* rows_v = logits_v + static_cast<size_t>(b) * (k + 1) * V;
  if (threadIdx.x < 64) {   // a lane per test, 64 drafts at a time: the first that fails ends the kept prefix
    int n = k;
    for (int i0 = 0; i0 < k && n == k; i0 += 64) {
      const int i = i0 + (int)threadIdx.x;
      bool kept = true;
      if (i < k) {
        const int di = d[i];
        kept = di >= 0 && di < V;                // not a token: rejected, never used as an index
        if (kept) {
          const float ps = prob(rows_d[static_cast<size_t>(i) * V + di], st[2 * i], inv_t, 1.0f / st[2 * i + 1]);
          const float ph = prob(rows_v[static_cast<size_t>(i) * V + di], st[2 * (kmax + i)], inv_t, 1.0f / st[2 * (kmax + i) + 1]);
          kept = uniform24(seed, b, base + i, 1) < ph / ps;   // kept with probability min(1, P_H / P_S)
        }
      }
      const unsigned long long fails = __ballot(!kept);
      if (fails != 0ull) n = i0 + __ffsll(fails) - 1;
    }
    if (threadIdx.x == 0) n_sh = n;
  }
  __syncthreads();
  const int n = n_sh;
  const float u = uniform24(seed, b, base + n, 2);
  const float* lh = rows_v + static_cast<size_t>(n) * V;
  const float mh = st[2 * (kmax + n)], rsh = 1.0f / st[2 * (kmax + n) + 1];
  int tok;
  const float* ls = rows_d + static_cast<size_t>(n < k ? n : 0) * V;
  const float ms = n < k ? st[2 * n] : 0.f, rss = n < k ? 1.0f / st[2 * n + 1] : 0.f;
  auto residual = [&](const float4& a, const float4& e) {
    return make_float4(residual_mass(prob(a.x, mh, inv_t, rsh), prob(e.x, ms, inv_t, rss)), residual_mass(prob(a.y, mh, inv_t, rsh), prob(e.y, ms, inv_t, rss)),
                       residual_mass(prob(a.z, mh, inv_t, rsh), prob(e.z, ms, inv_t, rss)), residual_mass(prob(a.w, mh, inv_t, rsh), prob(e.w, ms, inv_t, rss)));
  };
  if constexpr (G > 8) {
    // Rows that would fill the registers: only the sums are kept, over chunks of 4 blocks of the segment with the next chunk
    // requested ahead of the exponentials of this one; the blocks of the segment that is scanned are read again.
    constexpr int CB = 4, NC = G / CB;
    const int lane = threadIdx.x & 63, seg = segment_size(V), j0 = min(V, (int)(threadIdx.x >> 6) * seg), j1 = min(V, j0 + seg);
    float acc = 0.f;
    auto add = [&](const float4& v, int i) {
      if (j0 + i * 256 + 4 * lane < j1) acc += (v.x + v.y) + (v.z + v.w);
    };
    auto one = [&](const float4& a) {
      return make_float4(expf((a.x - mh) * inv_t), expf((a.y - mh) * inv_t), expf((a.z - mh) * inv_t), expf((a.w - mh) * inv_t));
    };
    float4 a[2][CB], e[2][CB];
    auto sum = [&](auto load, auto mass) {
      load(0);
#pragma unroll
      for (int c = 0; c < NC; ++c) {
        if (c * CB * 256 >= seg) break;          // (the same in every thread: segments of rows just above 32768 entries end in the third chunk)
        if (c + 1 < NC && (c + 1) * CB * 256 < seg) load(c + 1);
#pragma unroll
        for (int q = 0; q < CB; ++q) add(mass(c & 1, q), c * CB + q);
        __builtin_amdgcn_sched_barrier(0);
      }
    };
    if (n < k) {
      sum([&](int c) { load_groups(lh, V, j0 + c * CB * 256 + 4 * lane, 256, a[c & 1]); load_groups(ls, V, j0 + c * CB * 256 + 4 * lane, 256, e[c & 1]); },
          [&](int h, int q) { return residual(a[h][q], e[h][q]); });
    } else {
      sum([&](int c) { load_groups(lh, V, j0 + c * CB * 256 + 4 * lane, 256, a[c & 1]); }, [&](int h, int q) { return one(a[h][q]); });
    }
    tok = draw_walk(
        acc, [] {},
        [&](int jj, int end, float(&v)[4]) {
          const int at = min(jj, V - 4);
          const float4 x = *reinterpret_cast<const float4*>(lh + at);
          float4 t;
          if (n < k) t = residual(x, *reinterpret_cast<const float4*>(ls + at));
          else t = one(x);
          const bool on = jj < end;              // (a group of 4 is inside the segment or outside)
          v[0] = on ? t.x : 0.f; v[1] = on ? t.y : 0.f; v[2] = on ? t.z : 0.f; v[3] = on ? t.w : 0.f;
        },
        V, u, red, &res);
  } else if constexpr (G > 0) {
    const int lane = threadIdx.x & 63, seg = segment_size(V), j0 = min(V, (int)(threadIdx.x >> 6) * seg), j1 = min(V, j0 + seg);
    float4 l[G];
    load_groups(lh, V, j0 + 4 * lane, 256, l);
    if (n < k) {
      constexpr int GB = G < 4 ? G : 4;          // draft groups in flight (registers: 64 hold the row)
#pragma unroll
      for (int g0 = 0; g0 < G; g0 += GB) {
        float4 c[GB];
        load_groups(ls, V, j0 + g0 * 256 + 4 * lane, 256, c);
#pragma unroll
        for (int q = 0; q < GB; ++q) {
          const float4 a = l[g0 + q], e = c[q];
          const bool on = j0 + (g0 + q) * 256 + 4 * lane < j1;
          l[g0 + q] = on ? residual(a, e)
                         : make_float4(0.f, 0.f, 0.f, 0.f);
        }
      }
    } else {
      softmax_masses(l, V, mh, inv_t);
    }
    tok = block_draw_regs(l, V, u, walk, red, &res);
  } else if (n < k) {
    const bool vec = row_is_vec(lh) && row_is_vec(ls);
    tok = block_draw(
        [&](int jj, int end, float (&v)[4]) {
          float a[4], c[4];
          load_group(lh, jj, end, vec, a);
          load_group(ls, jj, end, vec, c);
          for (int e = 0; e < 4; ++e) v[e] = residual_mass(prob(a[e], mh, inv_t, rsh), prob(c[e], ms, inv_t, rss));
        },
        V, u, red, &res);
  } else {
    const bool vec = row_is_vec(lh);
    tok = block_draw(
        [&](int jj, int end, float (&v)[4]) {
          float l[4];
          load_group(lh, jj, end, vec, l);
          for (int e = 0; e < 4; ++e) v[e] = expf((l[e] - mh) * inv_t);
        },
        V, u, red, &res);
  }
  if (n < k && tok < 0) {
    // The residual has no mass (the two distributions agree to rounding; in exact arithmetic a
    // rejection implies mass elsewhere): the token is drawn from P_H with the same uniform, and
    // should that be the rejected draft itself, its successor in index order is taken, so that
    // the targets row still encodes n.
    tok = block_draw(
        [&](int jj, int end, float (&v)[4]) {
          float l[4];
          load_group(lh, jj, end, row_is_vec(lh), l);
          for (int e = 0; e < 4; ++e) v[e] = expf((l[e] - mh) * inv_t);
        },
        V, u, red, &res);
    if (tok == d[n]) tok = tok + 1 < V ? tok + 1 : 0;
  }
  int* g = targets + static_cast<size_t>(b) * (kmax + 1);
  for (int i = threadIdx.x; i <= k; i += blockDim.x) g[i] = i < n ? d[i] : (i == n ? tok : -1);
}

}  // namespace

// register groups per thread for rows of V entries with this alignment: 0 = the kernels for any row
static int reg_groups(const void* p, const void* q, size_t stride, int V) {
  if (V % 4 != 0 || stride % 4 != 0 || ((reinterpret_cast<uintptr_t>(p) | reinterpret_cast<uintptr_t>(q)) & 15) != 0) return 0;
  for (int g = 2; g <= kRegGroups; g *= 2)
    if (V <= reg_vocab(g)) return g;
  return 0;
}
#define HH_REG_GROUPS(g_, CALL) \
  switch (g_) {                 \
    case 2: CALL(2); break;     \
    case 4: CALL(4); break;     \
    case 8: CALL(8); break;     \
    case 16: CALL(16); break;   \
    default: CALL(0); break;    \
  }

hipError_t launch_sample_rows(const float* logits, size_t row_stride, int V, int B, const SamplingParams* prm,
                              SamplingParams prm_val, const int* idx_base, int idx_off, int purpose, int* out,
                              int out_stride, int out_off, hipStream_t s) {
#define HH_CALL(G)                                                                                                             \
  hipLaunchKernelGGL((sample_rows_kernel<G>), dim3(B), dim3(kDrawThreads), 0, s, logits, row_stride, V, prm, prm_val, idx_base, \
                     idx_off, purpose, out, out_stride, out_off)
  HH_REG_GROUPS(reg_groups(logits, nullptr, row_stride, V), HH_CALL)
#undef HH_CALL
  return hipGetLastError();
}

// ---- statistics buffer of the entry point that allocates nothing (hh_accept_tokens_static):
// one array per GPU, held until the process ends.  In host code the array's name is only a
// stand-in for the symbol; the device address comes from hipGetSymbolAddress, once per device.
constexpr size_t kStaticScratchFloats = 1 << 16;
static __device__ __align__(256) float scratch[kStaticScratchFloats];

hipError_t static_accept_scratch(float** ptr, size_t* n_floats) {
  constexpr int kMaxDevices = 64;
  static std::mutex mu;
  static float* per_device[kMaxDevices] = {};
  int dev = -1;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(mu);
  if (per_device[dev] == nullptr) {
    void* p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));   // the current device's copy of the array
    if (e != hipSuccess) return e;
    if (p == nullptr) return hipErrorInvalidSymbol;
    per_device[dev] = static_cast<float*>(p);
  }
  *ptr = per_device[dev];
  *n_floats = kStaticScratchFloats;
  return hipSuccess;
}

hipError_t launch_spec_targets(const float* logits_d, const float* logits_v, int V, int B, int k, int kmax,
                               const SamplingParams* prm, SamplingParams prm_val, float* stats, const int* drafts,
                               const int* committed, int* targets, hipStream_t s) {
  const int groups = reg_groups(logits_d, logits_v, V, V);
#define HH_CALL(G)                                                                                                               \
  hipLaunchKernelGGL((softmax_stats_kernel<G>), dim3(2 * k + 1, B), dim3(kDrawThreads), 0, s, logits_d, logits_v, V, k, kmax, prm, \
                     prm_val, stats)
  HH_REG_GROUPS(groups, HH_CALL)
#undef HH_CALL
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
#define HH_CALL(G)                                                                                                          \
  hipLaunchKernelGGL((spec_targets_kernel<G>), dim3(B), dim3(kDrawThreads), 0, s, logits_d, logits_v, V, k, kmax, prm, prm_val, \
                     stats, drafts, committed, targets)
  HH_REG_GROUPS(groups, HH_CALL)
#undef HH_CALL
  return hipGetLastError();
}

}  // namespace hh
