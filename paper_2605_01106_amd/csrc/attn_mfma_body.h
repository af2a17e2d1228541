// Attention branch on the matrix cores (bf16 KV cache): causal grouped-query attention of the
// T new positions of every sequence over all keys up to each position, rotary embedding of q
// fused, keys split over the wavefronts of a workgroup and over workgroups, log-sum-exp merge
// in slice order.  The keys and values of the new positions are already in the cache.
//
// Everything is computed transposed so that no operand ever has to be transposed in LDS.
// With v_mfma_f32_16x16x32_bf16 (D[m][n] += sum_k A[m][k] B[k][n]; lane l holds A[l%16][8(l/16)..+7],
// B[8(l/16)..+7][l%16] and D[4(l/16)+r][l%16]):
//   scores   S^T[key][row] = sum_dim K[key][dim] Q[row][dim]      A = 16 keys of the cache (one
//            16-byte load per lane: a key row is contiguous), B = query rows from LDS;
//   softmax  a lane then holds 8 keys of one query row: running maximum and sum per lane,
//            combined across the 4 lane groups with two lane exchanges;
//   output   O^T[dim][row] = sum_key V^T[dim][key] P^T[key][row]   A = V pages, stored
//            transposed (16 bytes = 8 consecutive tokens of one dimension), B = the lane's own
//            8 probabilities; the accumulator of a lane belongs to one query row, so the
//            rescaling of the online softmax is a per-lane scalar.
// The A rows of the two key blocks of a step are assigned so that a lane's 8 scores are the
// 8 consecutive keys its V load covers (block 0 row m <-> key 8(m/4) + m%4, block 1: + 4).
// Queries and probabilities are float32 values split exactly into three bf16 terms, so the
// products carry float32 accuracy (with two-term probabilities, 16 mantissa bits, models with
// order-one activations lost tokens to near ties that the float32 reference path keeps); K and V
// are used as stored.  The scores
// are kept in base-2 units (log2(e) folded into the query scale) so that the exponentials are
// single v_exp_f32 instructions.
#pragma once
#include "attn_common.h"
#include "bf16_split.h"

namespace hh {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

static constexpr int kStepKeys = 32;   // keys per wavefront step
static constexpr int kMergeLd = 20;    // row stride (floats) of the in-workgroup merge buffer

union Frag {
  uint4 u;
  bf16x8 v;
};

__device__ __forceinline__ void split3(float x, uint32_t& t0, uint32_t& t1, uint32_t& t2) { split3_bf16(x, t0, t1, t2); }

// maximum over the lanes l, l^16, l^32, l^48 (the four lanes that hold one query row), through
// the row swaps of the vector unit instead of LDS permutes: v_permlane16_swap exchanges the odd
// 16-lane rows of its first operand with the even rows of its second, v_permlane32_swap the upper
// half of the first with the lower half of the second.
__device__ __forceinline__ float xor_max(float v) {
  const uint32_t x = __float_as_uint(v);
  const auto s16 = __builtin_amdgcn_permlane16_swap(x, x, false, false);
  v = fmaxf(__uint_as_float(s16[0]), __uint_as_float(s16[1]));
  const uint32_t y = __float_as_uint(v);
  const auto s32 = __builtin_amdgcn_permlane32_swap(y, y, false, false);
  return fmaxf(__uint_as_float(s32[0]), __uint_as_float(s32[1]));
}
// 2^x through the hardware instruction (scores are kept in base-2 units)
__device__ __forceinline__ float ex2(float x) { return __builtin_amdgcn_exp2f(x); }
__device__ __forceinline__ float xor_add(float v) {
  v += __shfl_xor(v, 16, 64);
  return v + __shfl_xor(v, 32, 64);
}

// One workgroup: bx of row_chunks * n_splits (key slice and row chunk), KV head kvh, sequence b.  RT = 16-row tiles per workgroup,
// KS = ceil(Dh / 32).
//
// FUSE (verification: at most 16 new positions, one row chunk): the keys and values of the new
// positions are not in the cache yet.  The cached keys (positions < pos0) are visible to every
// row; the workgroups of the last key slice take the new positions from the projection buffer (rotating
// and rounding k, rounding v), append them to the cache and score them as one more step with the
// causal mask.  Otherwise the cache already holds them (prefill).
//
// NW wavefronts per workgroup split the keys of its slice and meet in LDS.
// smem_raw: attn_mfma_lds() bytes of LDS; s_last: a word of LDS.
template <int RT, int KS, bool FUSE, int NW>
__device__ __forceinline__ void attn_mfma_body(const Dims& d, const AttnArgs& a, const int row_chunks, const int bx, const int kvh,
                                               const int b, unsigned char* smem_raw, int& s_last) {
  constexpr int NT = 64 * NW;            // threads
  constexpr int NDB = 2 * KS;            // blocks of 16 output dimensions
  constexpr int Dhp = 32 * KS;           // head dimension padded to the MFMA depth
  constexpr int QS = 3 * Dhp + 8;        // bf16 elements per staged query row (3 split terms + pad)
  constexpr int R = RT * 16;
  int* pg = reinterpret_cast<int*>(smem_raw);                                  // [NW][64] page numbers of a wavefront's steps
  uint16_t* qT = reinterpret_cast<uint16_t*>(smem_raw + NT * 4);               // [R][QS]
  // FUSE: the new keys [16][KNS] and, transposed, the new values [Dhp][VNS] (rows of 16-byte groups, padded against bank conflicts)
  constexpr int KNS = Dhp + 8, VNS = 24, NEWS = FUSE ? 16 * KNS + Dhp * VNS : 0;
  uint16_t* kN = qT + R * QS;
  uint16_t* vN = kN + 16 * KNS;
  float* mrg = reinterpret_cast<float*>(smem_raw + NT * 4 + (size_t)(R * QS + NEWS) * 2);   // merge scratch
  float* mrg_o = mrg;                                                          // [NW-1][Dhp][kMergeLd]
  float* mrg_ml = mrg + (NW - 1) * Dhp * kMergeLd;                             // [NW-1][16][2]

  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int g = lane >> 4, n = lane & 15;
  const int chunk = bx % row_chunks, sp = bx / row_chunks;
  TR(0);
  const int nt = a.n_tok != nullptr ? a.n_tok[b] : a.T;
  const int pos0 = a.pos0[b];
  const int Dh = d.Dh, G = d.Hq / d.Hkv, half = Dh >> 1, S = a.n_splits;
  const int n_rows = a.T * G;
  const int row_lim = min(n_rows, nt * G);     // row = position j * G + query head of the group; valid while j < nt
  const int row0 = chunk * R;
  if (a.row0 != nullptr && row0 >= row_lim) return;   // packed rows: no row of this chunk exists (the whole workgroup leaves)
  const int jmax = row0 < row_lim ? (min(row_lim, row0 + R) - 1) / G : -1;
  const int nk_all = jmax < 0 ? 0 : pos0 + jmax + 1;      // keys 0 .. nk_all-1 are visible to some row of this chunk
  const int nk = FUSE ? min(nk_all, pos0) : nk_all;       // ... of which the cache holds 0 .. nk-1
  const int* pt_row = a.page_table + (size_t)b * d.pages_per_seq;
  const int pshift = 31 - __clz(d.page_tokens), pmask = d.page_tokens - 1;
  const uint16_t* kp = static_cast<const uint16_t*>(a.kpool);
  const uint16_t* vp = static_cast<const uint16_t*>(a.vpool);
  const size_t rows0 = first_row(a.row0, b, a.T);
  const float* xrow = a.qkv + rows0 * d.ldzx;
  const bool al4 = (d.ldzx & 3) == 0 && (reinterpret_cast<uintptr_t>(xrow) & 15) == 0;   // 16-byte aligned rows (dq, Dh are multiples of 8)

  // key steps of this workgroup and of this wavefront
  const int steps = (nk + kStepKeys - 1) / kStepKeys;
  const int sps = (steps + S - 1) / S;
  const int sb = sp * sps, se = min(steps, sb + sps);
  // (the last wavefront of the last slice scores the new positions: one step less for it)
  const int extra = FUSE && sp == S - 1 ? 1 : 0;
  const int per = (max(se - sb, 0) + extra + NW - 1) / NW;
  const int ws = sb + wave * per, we = min(se, ws + per);

  // Operand loads of one step.  A step's 32 keys lie in one page (the page size is a multiple of
  // 32 on this path), so the page number is a scalar load and the lane offsets within the page
  // are computed once.
  Frag kA[KS], kB[KS], vT[NDB];
  const size_t head_elems = (size_t)d.page_tokens * Dh;              // elements per (page, head)
  const int kofsA = 8 * (n >> 2) + (n & 3);                          // key of block A row n within the step
  int voff[NDB];                                                     // dimension (clamped) * page_tokens
#pragma unroll
  for (int db = 0; db < NDB; ++db) voff[db] = min(db * 16 + n, Dh - 1) * d.page_tokens;
  const bool dh32 = (Dh & 31) == 0;
  // The page numbers of 64 steps at a time go through LDS (one per lane, read back by the whole
  // wavefront): a page-table load in the step loop would expose its memory latency every step.
  int* pgw = pg + wave * 64;
  auto stage_pages = [&](int step0) { pgw[lane] = pt_row[(max(min(step0 + lane, steps - 1), 0) * kStepKeys) >> pshift]; };
  stage_pages(ws);
  auto load_step = [&](int step, Frag(&ka)[KS], Frag(&kb)[KS], Frag(&vt)[NDB]) {
    const int key0 = step * kStepKeys;
    if (step != ws && ((step - ws) & 63) == 0) stage_pages(step);
    const int page = __builtin_amdgcn_readfirstlane(pgw[(step - ws) & 63]);
    const size_t base = ((size_t)page * d.Hkv + kvh) * head_elems;
    const int in0 = key0 & pmask, last = nk - 1 - (key0 - in0);      // in-page index of the step's first key / of the last cached key
    // past the end: a valid key, masked later
    const uint16_t* pa = kp + base + (size_t)(min(in0 + kofsA, last) * Dh + 8 * g);
    const uint16_t* pb = kp + base + (size_t)(min(in0 + kofsA + 4, last) * Dh + 8 * g);
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      // unconditional loads (a branch around them would make the wait for the previous step's
      // operands wait for these as well); lanes past the head dimension re-read dimension 0
      const int off = (dh32 || ks * 32 + 8 * g < Dh) ? ks * 32 : -8 * g;
      ka[ks].u = *reinterpret_cast<const uint4*>(pa + off);
      kb[ks].u = *reinterpret_cast<const uint4*>(pb + off);
    }
    if (!dh32) {
#pragma unroll
      for (int ks = 0; ks < KS; ++ks)
        if (ks * 32 + 8 * g >= Dh) { ka[ks].u = make_uint4(0, 0, 0, 0); kb[ks].u = make_uint4(0, 0, 0, 0); }
    }
    // 8 consecutive tokens of one dimension (tokens >= nk are zeroed when the step is scored)
    const int tok = in0 + 8 * g;
    const int cnt = min(max(last + 1 - tok, 0), 8);
    const uint16_t* pv = vp + base + (cnt > 0 ? tok : (last & ~7));
#pragma unroll
    for (int db = 0; db < NDB; ++db) vt[db].u = *reinterpret_cast<const uint4*>(pv + voff[db]);
  };
  if (ws < we) load_step(ws, kA, kB, vT);
  TR(1);

  // ---- the new positions (FUSE), in the workgroups of the last slice: all threads rotate and round the new keys and
  // values, append them to the cache and leave them in LDS, from where the last wavefront takes them as the operands of
  // one more step.  (Built by that wavefront alone, from 64 and more loads of its own, they were the longest chain of a
  // short launch.  Launch after a pass over 600 MB, before and after: 24 sequences x 1 position over 777 keys of head
  // dimension 128 23.4 -> 20.9 us, 64 x 9 over 400 keys 29.7 -> 25.0; one sequence x 3 over 512 keys of dimension 64
  // 11.9 -> 9.1, 16 x 5 over 2048 keys in 8 slices 12.6 -> 10.6.)
  // Items of 4 dimensions: nt * half / 4 pairs of key dimensions, then nt * Dh / 4 groups of a value.
  const bool has_new = FUSE && sp == S - 1 && nk_all > pos0;
  const bool new_wave = has_new && wave == NW - 1;
  const int k_items = has_new ? nt * (half >> 2) : 0, kv_items = has_new ? k_items + nt * (Dh >> 2) : 0;
  auto load4 = [&](const float* src) -> float4 {
    return al4 ? *reinterpret_cast<const float4*>(src) : make_float4(src[0], src[1], src[2], src[3]);
  };
  struct NewItem { float4 x0, x1, c0, c1; int page; };
  auto new_load = [&](int it) -> NewItem {
    NewItem v;
    v.x0 = v.x1 = v.c0 = v.c1 = make_float4(0.f, 0.f, 0.f, 0.f);
    v.page = 0;
    if (it >= kv_items) return v;
    const bool key = it < k_items;
    const int per = key ? half >> 2 : Dh >> 2, i0 = key ? it : it - k_items, j = i0 / per, i = 4 * (i0 - j * per);
    v.page = pt_row[(pos0 + j) >> pshift];
    const float* src = xrow + (size_t)j * d.ldzx + d.dq + (key ? 0 : d.dkv) + (size_t)kvh * Dh + i;
    v.x0 = load4(src);
    if (key) {
      v.x1 = load4(src + half);
      const float4* c = reinterpret_cast<const float4*>(a.rope + ((size_t)(pos0 + j) * half + i) * 2);
      v.c0 = c[0]; v.c1 = c[1];
    }
    return v;
  };
  auto new_store = [&](int it, const NewItem& v) {
    if (it >= kv_items) return;
    const bool key = it < k_items;
    const int per = key ? half >> 2 : Dh >> 2, i0 = key ? it : it - k_items, j = i0 / per, i = 4 * (i0 - j * per);
    const int in = (pos0 + j) & pmask;
    auto pack = [](float p, float q) { return (uint32_t)f32_to_bf16_rne(p) | ((uint32_t)f32_to_bf16_rne(q) << 16); };
    if (key) {
      const uint2 lo = make_uint2(pack(v.x0.x * v.c0.x - v.x1.x * v.c0.y, v.x0.y * v.c0.z - v.x1.y * v.c0.w),
                                  pack(v.x0.z * v.c1.x - v.x1.z * v.c1.y, v.x0.w * v.c1.z - v.x1.w * v.c1.w));
      const uint2 hi = make_uint2(pack(v.x1.x * v.c0.x + v.x0.x * v.c0.y, v.x1.y * v.c0.z + v.x0.y * v.c0.w),
                                  pack(v.x1.z * v.c1.x + v.x0.z * v.c1.y, v.x1.w * v.c1.z + v.x0.w * v.c1.w));
      uint16_t* dst = static_cast<uint16_t*>(a.kpool) + (((size_t)v.page * d.Hkv + kvh) * d.page_tokens + in) * Dh + i;
      *reinterpret_cast<uint2*>(dst) = lo;
      *reinterpret_cast<uint2*>(dst + half) = hi;
      *reinterpret_cast<uint2*>(kN + j * KNS + i) = lo;
      *reinterpret_cast<uint2*>(kN + j * KNS + half + i) = hi;
    } else {
      const float x[4] = {v.x0.x, v.x0.y, v.x0.z, v.x0.w};
      uint16_t* dst = static_cast<uint16_t*>(a.vpool) + (((size_t)v.page * d.Hkv + kvh) * Dh + i) * d.page_tokens + in;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const uint16_t h = f32_to_bf16_rne(x[q]);
        dst[(size_t)q * d.page_tokens] = h;
        vN[(i + q) * VNS + j] = h;
      }
    }
  };
  // the first items of a thread travel while the queries are staged: two, or one where 16 positions have no more (head
  // dimensions up to 32: 192 items; a second one is 17 registers and a division for nothing)
  constexpr bool two_items = KS > 1;
  NewItem new0, new1;
  if (FUSE && has_new) {
    new0 = new_load(tid);
    if (two_items) new1 = new_load(tid + NT);
  }

  // ---- query rows: rotate to their positions, scale, split into 3 bf16 terms, stage in LDS
  {
    const float scale = 1.4426950408889634f / sqrtf((float)Dh);   // scores in base-2 units: softmax through 2^x
    const float2* rope = reinterpret_cast<const float2*>(a.rope);
    // (up to head dimension 32 the single elements below keep more threads busy, in one round trip as well: with these two
    // rules the launch is back at its time before the items of 4, e.g. 64 sequences x 1 position over 1000 keys of head
    // dimension 32 12.5 -> 11.3 us, 16 x 3 over 300 keys of head dimension 16 8.8 -> 7.8; runs differ by up to 5 %)
    if (KS > 1 && al4 && (half & 3) == 0) {
      // items of 4 dimension pairs, four per thread and pass, their loads issued together: up to 4 NT items (1024 with four
      // wavefronts; 32 rows of head dimension 128 are 512) take one round trip to memory
      const int h4 = half >> 2, items = R * h4;
      for (int it0 = tid; it0 < items; it0 += 4 * NT) {
        float4 x0[4], x1[4], c0[4], c1[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const int it = it0 + u * NT, r = it / h4, i = 4 * (it - r * h4), rr = row0 + r;
          x0[u] = x1[u] = c0[u] = c1[u] = make_float4(0.f, 0.f, 0.f, 0.f);
          if (it < items && rr < row_lim) {
            const int j = rr / G;
            const float* q = xrow + (size_t)j * d.ldzx + (size_t)(kvh * G + rr % G) * Dh + i;
            const float4* c = reinterpret_cast<const float4*>(rope + (size_t)(pos0 + j) * half + i);
            c0[u] = c[0]; c1[u] = c[1];
            x0[u] = *reinterpret_cast<const float4*>(q); x1[u] = *reinterpret_cast<const float4*>(q + half);
          }
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const int it = it0 + u * NT, r = it / h4, i = 4 * (it - r * h4);
          if (it >= items) break;
          const float lo[4] = {(x0[u].x * c0[u].x - x1[u].x * c0[u].y) * scale, (x0[u].y * c0[u].z - x1[u].y * c0[u].w) * scale,
                               (x0[u].z * c1[u].x - x1[u].z * c1[u].y) * scale, (x0[u].w * c1[u].z - x1[u].w * c1[u].w) * scale};
          const float hi[4] = {(x1[u].x * c0[u].x + x0[u].x * c0[u].y) * scale, (x1[u].y * c0[u].z + x0[u].y * c0[u].w) * scale,
                               (x1[u].z * c1[u].x + x0[u].z * c1[u].y) * scale, (x1[u].w * c1[u].z + x0[u].w * c1[u].w) * scale};
          uint16_t* row = qT + (size_t)r * QS + i;
          uint2 t[3];
          split3_bf16_pair(lo[0], lo[1], t[0].x, t[1].x, t[2].x);
          split3_bf16_pair(lo[2], lo[3], t[0].y, t[1].y, t[2].y);
#pragma unroll
          for (int k = 0; k < 3; ++k) *reinterpret_cast<uint2*>(row + k * Dhp) = t[k];
          split3_bf16_pair(hi[0], hi[1], t[0].x, t[1].x, t[2].x);
          split3_bf16_pair(hi[2], hi[3], t[0].y, t[1].y, t[2].y);
#pragma unroll
          for (int k = 0; k < 3; ++k) *reinterpret_cast<uint2*>(row + k * Dhp + half) = t[k];
        }
      }
    } else {
      // four items per thread and pass, their loads issued together
      for (int it0 = tid; it0 < R * half; it0 += 4 * NT) {
        float x0[4], x1[4];
        float2 c[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const int it = it0 + u * NT, r = it / half, i = it - r * half, rr = row0 + r;
          x0[u] = 0.f; x1[u] = 0.f; c[u] = make_float2(0.f, 0.f);
          if (it < R * half && rr < row_lim) {
            const int j = rr / G;
            const float* q = xrow + (size_t)j * d.ldzx + (size_t)(kvh * G + rr % G) * Dh;
            c[u] = rope[(size_t)(pos0 + j) * half + i];
            x0[u] = q[i]; x1[u] = q[i + half];
          }
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const int it = it0 + u * NT, r = it / half, i = it - r * half;
          if (it >= R * half) break;
          const float lo = (x0[u] * c[u].x - x1[u] * c[u].y) * scale, hi = (x1[u] * c[u].x + x0[u] * c[u].y) * scale;
          uint32_t l0, l1, l2, h0, h1, h2;
          split3(lo, l0, l1, l2);
          split3(hi, h0, h1, h2);
          uint16_t* row = qT + (size_t)r * QS;
          row[i] = (uint16_t)l0; row[Dhp + i] = (uint16_t)l1; row[2 * Dhp + i] = (uint16_t)l2;
          row[i + half] = (uint16_t)h0; row[Dhp + i + half] = (uint16_t)h1; row[2 * Dhp + i + half] = (uint16_t)h2;
        }
      }
    }
    if (Dh < Dhp) {
      const int padw = Dhp - Dh;
      for (int it = tid; it < R * padw * 3; it += NT) {
        const int r = it / (padw * 3), rem = it - r * padw * 3, term = rem / padw, i = rem - term * padw;
        qT[(size_t)r * QS + term * Dhp + Dh + i] = 0;
      }
    }
  }
  if (FUSE && has_new) {
    new_store(tid, new0);
    if (two_items) {
      new_store(tid + NT, new1);
      for (int it = tid + 2 * NT; it < kv_items; it += NT) new_store(it, new_load(it));
    }
    // values of positions that do not exist meet zero probabilities: they must not be NaN
    for (int it = tid; it < Dh * (16 - nt); it += NT) vN[(it / (16 - nt)) * VNS + nt + it % (16 - nt)] = 0;
  }
  __syncthreads();
  TR(2);

  // the key limit of this lane's query row in each tile (row n of tile rt)
  int lim[RT];
#pragma unroll
  for (int rt = 0; rt < RT; ++rt) {
    const int rr = row0 + rt * 16 + n;
    lim[rt] = rr < row_lim ? (FUSE ? pos0 - 1 : pos0 + rr / G) : 0x7fffffff;   // rows past the end: never stored
  }
  const int lim_min = FUSE ? pos0 - 1 : pos0 + row0 / G;     // the smallest limit of the chunk's rows
  float mrun[RT], lrun[RT];
  f32x4 acc[RT][NDB];
#pragma unroll
  for (int rt = 0; rt < RT; ++rt) {
    mrun[rt] = -INFINITY; lrun[rt] = 0.f;
#pragma unroll
    for (int db = 0; db < NDB; ++db) acc[rt][db] = f32x4{0.f, 0.f, 0.f, 0.f};
  }

  // one step of 32 keys: scores, online softmax, output.  The lane's 8 keys are kbase .. kbase+7,
  // visible to the lane's row of tile rt while <= limit[rt].
  // `masked` (wavefront-uniform): some key of the step may be invisible to some row; otherwise
  // all 32 keys are visible to every row and the comparisons are skipped.
  // `nvalid`: keys >= nvalid of a cached step are not in the cache: their value operands are
  // zeroed here (0 * stale bits must not be a NaN).
  auto score_step = [&](const Frag(&ka)[KS], const Frag(&kb)[KS], Frag(&vt)[NDB], const int kbase, const int(&limit)[RT],
                        const bool masked, const int nvalid) {
    if (kbase - 8 * g + kStepKeys > nvalid) {             // wavefront-uniform: the last step of the sequence
      const int cnt = min(max(nvalid - kbase, 0), 8);
      uint32_t mw[4];
#pragma unroll
      for (int w = 0; w < 4; ++w) mw[w] = (2 * w < cnt ? 0x0000FFFFu : 0u) | (2 * w + 1 < cnt ? 0xFFFF0000u : 0u);
#pragma unroll
      for (int db = 0; db < NDB; ++db) { vt[db].u.x &= mw[0]; vt[db].u.y &= mw[1]; vt[db].u.z &= mw[2]; vt[db].u.w &= mw[3]; }
    }
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) {
      // large tiles: re-read the query fragments from LDS every step instead of keeping all
      // of them in registers across the loop
      if (RT * KS > 4) asm volatile("" ::: "memory");
      f32x4 sA = f32x4{0.f, 0.f, 0.f, 0.f}, sB = f32x4{0.f, 0.f, 0.f, 0.f};
      const uint16_t* qrow = qT + (size_t)(rt * 16 + n) * QS + 8 * g;
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) {
#pragma unroll
        for (int term = 0; term < 3; ++term) {
          Frag q;
          q.u = *reinterpret_cast<const uint4*>(qrow + term * Dhp + ks * 32);
          sA = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ka[ks].v, q.v, sA, 0, 0, 0);
          sB = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kb[ks].v, q.v, sB, 0, 0, 0);
        }
      }
      float sc[8] = {sA[0], sA[1], sA[2], sA[3], sB[0], sB[1], sB[2], sB[3]};
      if (masked) {
#pragma unroll
        for (int i = 0; i < 8; ++i) sc[i] = kbase + i <= limit[rt] ? sc[i] : -INFINITY;
      }
      const float mx = fmaxf(fmaxf(fmaxf(sc[0], sc[1]), fmaxf(sc[2], sc[3])), fmaxf(fmaxf(sc[4], sc[5]), fmaxf(sc[6], sc[7])));
      const float mold = mrun[rt];
      const float mnew = fmaxf(mold, xor_max(mx));
      // every key masked so far: keep the state (2^(-inf - -inf) is not a number)
      const float msub = masked && mnew == -INFINITY ? 0.f : mnew;
      float pr[8];
#pragma unroll
      for (int i = 0; i < 8; ++i) pr[i] = ex2(sc[i] - msub);       // 2^-inf = 0 for masked keys
      const float psum = ((pr[0] + pr[1]) + (pr[2] + pr[3])) + ((pr[4] + pr[5]) + (pr[6] + pr[7]));
      const float corr = ex2(mold - msub);                         // 0 while nothing was accumulated
      lrun[rt] = lrun[rt] * corr + psum;
      mrun[rt] = mnew;
      // the probabilities go into the value product split exactly into three bf16 terms
      Frag p0, p1, p2;
      split3_bf16_pair(pr[0], pr[1], p0.u.x, p1.u.x, p2.u.x);
      split3_bf16_pair(pr[2], pr[3], p0.u.y, p1.u.y, p2.u.y);
      split3_bf16_pair(pr[4], pr[5], p0.u.z, p1.u.z, p2.u.z);
      split3_bf16_pair(pr[6], pr[7], p0.u.w, p1.u.w, p2.u.w);
      // the accumulators are rescaled only when some row's maximum rose (and it holds something)
      if (__builtin_amdgcn_ballot_w64(corr != 1.f && mold != -INFINITY) != 0) {
#pragma unroll
        for (int db = 0; db < NDB; ++db) {
          acc[rt][db][0] *= corr; acc[rt][db][1] *= corr; acc[rt][db][2] *= corr; acc[rt][db][3] *= corr;
        }
      }
#pragma unroll
      for (int db = 0; db < NDB; ++db) {
        f32x4 c = acc[rt][db];
        c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vt[db].v, p0.v, c, 0, 0, 0);
        c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vt[db].v, p1.v, c, 0, 0, 0);
        c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vt[db].v, p2.v, c, 0, 0, 0);
        acc[rt][db] = c;
      }
    }
  };

  // ---- the new positions (FUSE): scored as one more step by the last wavefront
  if (FUSE && new_wave) {
    Frag nA[KS], nB[KS], nV[NDB];
    const uint4 zero = make_uint4(0, 0, 0, 0);
    const int j0 = 8 * (n >> 2) + (n & 3);                       // new positions of this lane's key rows: j0 and j0 + 4
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      const int d0 = ks * 32 + 8 * g;
      nA[ks].u = d0 < Dh && j0 < nt ? *reinterpret_cast<const uint4*>(kN + j0 * KNS + d0) : zero;
      nB[ks].u = d0 < Dh && j0 + 4 < nt ? *reinterpret_cast<const uint4*>(kN + (j0 + 4) * KNS + d0) : zero;
    }
#pragma unroll
    for (int db = 0; db < NDB; ++db)
      nV[db].u = db * 16 + n < Dh && g < 2 ? *reinterpret_cast<const uint4*>(vN + (db * 16 + n) * VNS + 8 * g) : zero;
    int limn[RT];
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) {
      const int rr = row0 + rt * 16 + n;
      limn[rt] = rr < row_lim ? rr / G : -1;                     // new position j is visible to position rr / G >= j
    }
    score_step(nA, nB, nV, 8 * g, limn, true, 0x7fffffff);
  }

  // Two operand sets in turn: the loads of a step are issued before the previous step is scored.
  // The loop body is branch-free (two steps, loads unconditional: past the last step they repeat
  // it) so that each wait counts exactly the loads issued after the operands it needs; an odd
  // last step follows the loop.
  {
    Frag kA2[KS], kB2[KS], vT2[NDB];
    const int n_steps = max(we - ws, 0);
    for (int step = ws; step + 1 < we; step += 2) {
      load_step(step + 1, kA2, kB2, vT2);
      score_step(kA, kB, vT, step * kStepKeys + 8 * g, lim, (step + 1) * kStepKeys - 1 > lim_min, nk);
      load_step(min(step + 2, we - 1), kA, kB, vT);
      score_step(kA2, kB2, vT2, (step + 1) * kStepKeys + 8 * g, lim, (step + 2) * kStepKeys - 1 > lim_min, nk);
    }
    if (n_steps & 1) score_step(kA, kB, vT, (we - 1) * kStepKeys + 8 * g, lim, we * kStepKeys - 1 > lim_min, nk);
  }
  TR(3);
#pragma unroll
  for (int rt = 0; rt < RT; ++rt) lrun[rt] = xor_add(lrun[rt]);

  // ---- merge the wavefronts (key slices in order) into wavefront 0, one row tile at a time
#pragma unroll
  for (int rt = 0; rt < RT; ++rt) {
    if (wave > 0) {
      if (g == 0) { mrg_ml[((wave - 1) * 16 + n) * 2] = mrun[rt]; mrg_ml[((wave - 1) * 16 + n) * 2 + 1] = lrun[rt]; }
#pragma unroll
      for (int db = 0; db < NDB; ++db)
#pragma unroll
        for (int r = 0; r < 4; ++r) mrg_o[((wave - 1) * Dhp + db * 16 + 4 * g + r) * kMergeLd + n] = acc[rt][db][r];
    }
    __syncthreads();
    if (wave == 0) {
      float mw[NW - 1], lw[NW - 1], M = mrun[rt];
#pragma unroll
      for (int w = 0; w < NW - 1; ++w) { mw[w] = mrg_ml[(w * 16 + n) * 2]; lw[w] = mrg_ml[(w * 16 + n) * 2 + 1]; M = fmaxf(M, mw[w]); }
      const float f0 = mrun[rt] == -INFINITY ? 0.f : ex2(mrun[rt] - M);
      float fw[NW - 1];
      float lsum = f0 * lrun[rt];
#pragma unroll
      for (int w = 0; w < NW - 1; ++w) { fw[w] = mw[w] == -INFINITY ? 0.f : ex2(mw[w] - M); lsum = fmaf(fw[w], lw[w], lsum); }
      lrun[rt] = lsum;
      mrun[rt] = M;
#pragma unroll
      for (int db = 0; db < NDB; ++db)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          float v = f0 * acc[rt][db][r];
#pragma unroll
          for (int w = 0; w < NW - 1; ++w) v = fmaf(fw[w], mrg_o[(w * Dhp + db * 16 + 4 * g + r) * kMergeLd + n], v);
          acc[rt][db][r] = v;
        }
    }
    __syncthreads();
  }
  TR(4);

  // ---- results of the workgroup (held by wavefront 0): final, or the partial of its key slice
  if (wave == 0) {
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) {
      const int rr = row0 + rt * 16 + n;
      if (rr >= (a.row0 != nullptr ? row_lim : n_rows)) continue;   // (packed rows: what follows is the next sequence's)
      const int j = rr / G, hq = kvh * G + rr % G;
      if (S == 1) {
        const float inv = (rr < row_lim && lrun[rt] > 0.f) ? 1.0f / lrun[rt] : 0.f;
        float* orow = a.o + (rows0 + j) * d.dq + (size_t)hq * Dh;
#pragma unroll
        for (int db = 0; db < NDB; ++db) {
          const int dim = db * 16 + 4 * g;
          if (dim < Dh)
            *reinterpret_cast<float4*>(orow + dim) =
                make_float4(acc[rt][db][0] * inv, acc[rt][db][1] * inv, acc[rt][db][2] * inv, acc[rt][db][3] * inv);
        }
      } else {
        const size_t rid = (((size_t)b * a.T + j) * d.Hq + hq) * S + sp;
#pragma unroll
        for (int db = 0; db < NDB; ++db) {
          const int dim = db * 16 + 4 * g;
          if (dim < Dh)
            *reinterpret_cast<float4*>(a.part_o + rid * Dh + dim) =
                make_float4(acc[rt][db][0], acc[rt][db][1], acc[rt][db][2], acc[rt][db][3]);
        }
        if (g == 0) { a.part_ml[rid * 2] = mrun[rt]; a.part_ml[rid * 2 + 1] = lrun[rt]; }
      }
    }
  }
  if (S == 1 || a.counters == nullptr) return;   // no counters: a merge kernel follows

  // Make the partials visible device-wide (release), then take a ticket; the workgroup that
  // draws the last ticket sees all of them after its acquire fence and merges the slices.
  TR(5);
  __threadfence();
  __syncthreads();
  int* counter = a.counters + ((size_t)b * d.Hkv + kvh) * row_chunks + chunk;
  if (tid == 0) {
    const int ticket = atomicAdd(counter, 1);
    s_last = ticket == S - 1;
    if (s_last) *counter = 0;   // ready for the next launch (launches on a context are ordered)
  }
  __syncthreads();
  TR(6);
  if (!s_last) return;
  __threadfence();
  float2* gm = reinterpret_cast<float2*>(mrg);   // [R][S] (maximum, sum) of every slice
  const int d4n = Dh >> 2;
  // the first 8 slices of this thread's first output item are requested together with the
  // slice statistics (they do not depend on them)
  float4 pv0[8];
  {
    const int it = min(tid, R * d4n - 1), r = it / d4n, c4 = it - r * d4n, rr = min(row0 + r, n_rows - 1);
    const size_t rid = ((size_t)b * a.T + rr / G) * d.Hq + kvh * G + rr % G;
#pragma unroll
    for (int u = 0; u < 8; ++u) pv0[u] = *reinterpret_cast<const float4*>(a.part_o + (rid * S + min(u, S - 1)) * Dh + 4 * c4);
  }
  for (int it = tid; it < R * S; it += NT) {
    const int r = it / S, s = it - r * S, rr = row0 + r;
    float2 v = make_float2(-INFINITY, 0.f);
    if (rr < n_rows) {
      const size_t rid = ((size_t)b * a.T + rr / G) * d.Hq + kvh * G + rr % G;
      v = reinterpret_cast<const float2*>(a.part_ml)[rid * S + s];
    }
    gm[it] = v;
  }
  __syncthreads();
  TR(7);
  for (int it = tid; it < R * d4n; it += NT) {
    const int r = it / d4n, c4 = it - r * d4n, rr = row0 + r;
    if (rr >= n_rows) continue;
    const int j = rr / G, hq = kvh * G + rr % G;
    const size_t rid = ((size_t)b * a.T + j) * d.Hq + hq;
    float M = -INFINITY;
    for (int s = 0; s < S; ++s) M = fmaxf(M, gm[r * S + s].x);
    float4 out = make_float4(0.f, 0.f, 0.f, 0.f);
    float L = 0.f;
    for (int s0 = 0; s0 < S; s0 += 16) {                // slice order: deterministic; 16 loads in flight
      float4 pv[16];
      if (it == tid && s0 == 0) {   // (copied by value: a choice between the two places would keep the array in scratch memory)
#pragma unroll
        for (int u = 0; u < 8; ++u) pv[u] = pv0[u];
      } else {
#pragma unroll
        for (int u = 0; u < 8; ++u) pv[u] = *reinterpret_cast<const float4*>(a.part_o + (rid * S + min(s0 + u, S - 1)) * Dh + 4 * c4);
      }
      if (s0 + 8 < S) {
#pragma unroll
        for (int u = 8; u < 16; ++u) pv[u] = *reinterpret_cast<const float4*>(a.part_o + (rid * S + min(s0 + u, S - 1)) * Dh + 4 * c4);
      }
#pragma unroll
      for (int u = 0; u < 16; ++u) {
        if (s0 + u < S) {
          const float2 ml = gm[r * S + s0 + u];
          const float w = ml.x == -INFINITY ? 0.f : ex2(ml.x - M);
          L = fmaf(w, ml.y, L);
          out.x = fmaf(w, pv[u].x, out.x); out.y = fmaf(w, pv[u].y, out.y);
          out.z = fmaf(w, pv[u].z, out.z); out.w = fmaf(w, pv[u].w, out.w);
        }
      }
    }
    const float inv = (rr < row_lim && L > 0.f) ? 1.0f / L : 0.f;
    *reinterpret_cast<float4*>(a.o + ((size_t)b * a.T + j) * d.dq + (size_t)hq * Dh + 4 * c4) =
        make_float4(out.x * inv, out.y * inv, out.z * inv, out.w * inv);
  }
  TR(8);
}

// bytes of LDS of a workgroup
template <int RT, int KS, bool FUSE, int NW>
size_t attn_mfma_lds(int n_splits) {
  constexpr int Dhp = 32 * KS, QS = 3 * Dhp + 8;
  size_t scratch = (size_t)((NW - 1) * Dhp * kMergeLd + (NW - 1) * 16 * 2) * sizeof(float);
  const size_t gm = (size_t)RT * 16 * n_splits * sizeof(float2);
  if (gm > scratch) scratch = gm;
  constexpr int news = FUSE ? 16 * (Dhp + 8) + Dhp * 24 : 0;
  return (size_t)NW * 64 * 4 + (size_t)(RT * 16 * QS + news) * 2 + scratch;
}

}  // namespace hh
