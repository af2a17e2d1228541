// Attention branch of the hybrid block for multi-position passes (verification, prefill):
// the float32-FMA kernel (float32 KV cache; any head dimension that is a multiple of 8), the
// append of new keys and values to the paged cache, and the dispatch between this kernel and
// the matrix-core kernel used for a bf16 cache with pages of 32 tokens and more (with pages of 16 it takes this one as well).
//
// One kernel per layer: rotary embedding of q and k, append of k and v to the paged KV cache
// (rounded to the storage type), causal grouped-query attention of the T new positions over
// all keys up to each position, split along the keys, and the log-sum-exp merge of the key
// slices in slice order.
//
// A workgroup owns 16 query rows (row = position j x query head of one KV group) and one
// slice of the keys.  K and V tiles of 64 keys are staged through LDS in float32: cached keys
// come from the pages; the keys of the new positions are rotated from the projection buffer,
// rounded, written to the cache by the one workgroup that owns them, and used as rounded.
// Lane t scores key t for the wavefront's 4 rows, the softmax is kept online per row, lane d
// accumulates output dimension d.  With several key slices every workgroup stores its partial
// result; the last one to finish (a counter per row chunk) merges them, so no second launch.
#include <stdlib.h>
#include "wave_ops.h"

#include "attn_common.h"

namespace hh {

static constexpr int kKeys = 64;      // keys per LDS tile
static constexpr int kRowsPerWave = 4;
static constexpr int kRowsPerBlock = 16;
static constexpr int kMaxDh = 256;

// Reductions over the 64 lanes without LDS traffic: DPP butterflies inside each row of 16
// lanes, then the four row results are read out and combined.  All lanes must be active.
__device__ __forceinline__ float wave_max(float v) {
  v = fmaxf(v, dpp_move<0xB1>(v));
  v = fmaxf(v, dpp_move<0x4E>(v));
  v = fmaxf(v, dpp_move<0x141>(v));
  v = fmaxf(v, dpp_move<0x140>(v));
  const int iv = __float_as_int(v);
  return fmaxf(fmaxf(__int_as_float(__builtin_amdgcn_readlane(iv, 0)), __int_as_float(__builtin_amdgcn_readlane(iv, 16))),
               fmaxf(__int_as_float(__builtin_amdgcn_readlane(iv, 32)), __int_as_float(__builtin_amdgcn_readlane(iv, 48))));
}
__device__ __forceinline__ float wave_add(float v) {
  v += dpp_move<0xB1>(v);
  v += dpp_move<0x4E>(v);
  v += dpp_move<0x141>(v);
  v += dpp_move<0x140>(v);
  const int iv = __float_as_int(v);
  return (__int_as_float(__builtin_amdgcn_readlane(iv, 0)) + __int_as_float(__builtin_amdgcn_readlane(iv, 16))) +
         (__int_as_float(__builtin_amdgcn_readlane(iv, 32)) + __int_as_float(__builtin_amdgcn_readlane(iv, 48)));
}


__device__ __forceinline__ float round_store(float v, int bf16) {
  return bf16 ? __uint_as_float((uint32_t)f32_to_bf16_rne(v) << 16) : v;
}

// grid: x = row_chunks * n_splits, y = Hkv, z = B.  E = ceil(Dh / 64); FULL: Dh = 64 * E, so that every index division is one
// by a constant and the operand reads of the products are 16 bytes wide.
//
// Bound by its chain of memory round trips, one workgroup having few keys.  Order of the global loads (each later group needs
// the one before): position of the sequence | page numbers -> rotation table, query rows, new keys | cached keys of the first
// tile.  Whole tiles are requested whatever their number of cached keys, page numbers first: loads under a condition per
// item make the compiler wait for each item's page number before it asks for the next.  The first key slice does not even
// need the position for its first tile.  The cached keys of tile t + 1 are requested before tile t is scored.
template <int BF16, int E, bool FULL, bool WALK>
__global__ __launch_bounds__(256) void attention_kernel(const Dims d, const AttnArgs a, const int row_chunks) {
  constexpr int EPI = BF16 ? 8 : 4;          // elements per 16-byte item
  constexpr int NI = BF16 ? 2 * E : 4 * E;   // items of a K (or V) tile per thread
  constexpr int NQ = 2 * E;                  // rotation pairs of the query rows per thread
  extern __shared__ __align__(16) float smem[];
  __shared__ int s_last;
  const int Dh = FULL ? 64 * E : d.Dh, G = d.Hq / d.Hkv, half = Dh >> 1;
  const int ldk = Dh + 1;
  float* Ks = smem;                         // [kKeys][Dh+1]
  float* Vs = Ks + kKeys * ldk;             // [kKeys][Dh]
  float* qs = Vs + kKeys * Dh;              // [kRowsPerBlock][Dh]
  float* ps = qs + kRowsPerBlock * Dh;      // [4 waves][kRowsPerWave][kKeys]

  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int chunk = blockIdx.x % row_chunks, sp = blockIdx.x / row_chunks;
  const int kvh = blockIdx.y, b = blockIdx.z;
  TR(0);
  const int n_rows = a.T * G;
  const int* pt_row = a.page_table + (size_t)b * d.pages_per_seq;
  const float scale = 1.0f / sqrtf((float)Dh);
  const float2* rope = reinterpret_cast<const float2*>(a.rope);
  const size_t rows0 = first_row(a.row0, b, a.T);
  const float* xrow = a.qkv + rows0 * d.ldzx;   // q | k | v of this sequence's positions
  const size_t esz = BF16 ? 2 : 4;
  const char* kbytes = static_cast<const char*>(a.kpool);
  const char* vbytes = static_cast<const char*>(a.vpool);

  // ---- cached keys of a tile: pages -> registers -> LDS as float32.  A K item is 16 bytes of one key row; a V item is 16 bytes
  // of one dimension (consecutive tokens of a page).  Items without a cached key read their place in the page all the same (a
  // page number of the table's end where the tile goes past it) and are not used.
  const int cpk = Dh / EPI;                 // items per key
  const int n_items = kKeys * cpk;
  uint4 kreg[NI], vreg[NI];
  constexpr int TPI = EPI;                   // tokens per V item
  const int pshift = 31 - __clz(d.page_tokens), pmask = d.page_tokens - 1;   // page sizes are powers of two
  // Item i of a thread, number tid + 256 i, as (key, group of its row) and (group of tokens, dimension).  WALK: from the item before
  // it, and anew for every tile; otherwise by divisions, which the compiler keeps from tile to tile in up to 50 registers.
  struct Place { int kq, c, grp, dd; };
  const Place origin{tid / cpk, tid % cpk, tid / Dh, tid % Dh};
  auto place = [&](int i, Place& p) {
    if (!WALK) {
      const int it = tid + 256 * i;
      p.kq = it / cpk; p.c = it - p.kq * cpk; p.grp = it / Dh; p.dd = it - p.grp * Dh;
    } else if (i == 0) {
      p = origin;
      asm volatile("" : "+v"(p.kq), "+v"(p.c), "+v"(p.grp), "+v"(p.dd));
    } else {
      p.c += 256 % cpk; p.kq += 256 / cpk;
      if (p.c >= cpk) { p.c -= cpk; ++p.kq; }
      p.dd += 256 % Dh; p.grp += 256 / Dh;
      if (p.dd >= Dh) { p.dd -= Dh; ++p.grp; }
    }
  };
  auto load_tile = [&](int t) {
    const int key0 = t * kKeys;
    int kpg[NI], vpg[NI];
    Place p;
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      place(i, p);
      kpg[i] = pt_row[min((key0 + min(p.kq, kKeys - 1)) >> pshift, d.pages_per_seq - 1)];
      vpg[i] = pt_row[min((key0 + min(p.grp, kKeys / TPI - 1) * TPI) >> pshift, d.pages_per_seq - 1)];
    }
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      place(i, p);
      const int kpos = key0 + min(p.kq, kKeys - 1), vpos = key0 + min(p.grp, kKeys / TPI - 1) * TPI;
      kreg[i] = *reinterpret_cast<const uint4*>(kbytes + ((((size_t)kpg[i] * d.Hkv + kvh) * d.page_tokens + (kpos & pmask)) * Dh + p.c * EPI) * esz);
      vreg[i] = *reinterpret_cast<const uint4*>(vbytes + ((((size_t)vpg[i] * d.Hkv + kvh) * Dh + p.dd) * d.page_tokens + (vpos & pmask)) * esz);
    }
  };
  // (Longer passes ask for it below, once the position says that something is cached: of a prompt's first pass nothing is.)
  if (sp == 0 && a.T <= 16) load_tile(0);

  // rows of this workgroup: row = position j * G + query head of the group; valid while j < nt
  const int nt = a.n_tok != nullptr ? a.n_tok[b] : a.T;
  const int pos0 = a.pos0[b];
  const int row_lim = min(n_rows, nt * G);
  const int row0 = chunk * kRowsPerBlock;
  const int jmax = row0 < row_lim ? (min(row_lim, row0 + kRowsPerBlock) - 1) / G : -1;
  int rj[kRowsPerWave], rq[kRowsPerWave];
  bool rok[kRowsPerWave];
#pragma unroll
  for (int r = 0; r < kRowsPerWave; ++r) {
    const int rg = row0 + wave * kRowsPerWave + r;
    rj[r] = rg / G; rq[r] = kvh * G + rg % G;
    rok[r] = rg < row_lim;
  }

  // key slice of this workgroup (whole tiles)
  const int nk = jmax < 0 ? 0 : pos0 + jmax + 1;
  const int tiles = (nk + kKeys - 1) / kKeys;
  const int tps = (tiles + a.n_splits - 1) / a.n_splits;
  const int t_begin = sp * tps, t_end = min(tiles, (sp + 1) * tps);
  auto store_tile = [&](int t) {
    const int key0 = t * kKeys;
    const int n_old = min(max(pos0 - key0, 0), kKeys);
    Place p;
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      place(i, p);
      if (tid + 256 * i >= n_items) continue;
      float* kd = Ks + p.kq * ldk + p.c * EPI;
      if (p.kq < n_old) {
        const uint32_t kw[4] = {kreg[i].x, kreg[i].y, kreg[i].z, kreg[i].w};
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          if (BF16) { kd[2 * e] = __uint_as_float(kw[e] << 16); kd[2 * e + 1] = __uint_as_float(kw[e] & 0xffff0000u); }
          else kd[e] = __uint_as_float(kw[e]);
        }
      } else if (key0 + p.kq >= nk) {         // past the last key: zeros (the new keys are staged separately)
#pragma unroll
        for (int e = 0; e < EPI; ++e) kd[e] = 0.f;
      }
      const uint32_t vw[4] = {vreg[i].x, vreg[i].y, vreg[i].z, vreg[i].w};
#pragma unroll
      for (int e = 0; e < TPI; ++e) {
        const int vk = p.grp * TPI + e;
        float val = 0.f;
        if (vk < n_old) val = BF16 ? ((e & 1) ? __uint_as_float(vw[e >> 1] & 0xffff0000u) : __uint_as_float(vw[e >> 1] << 16))
                                   : __uint_as_float(vw[e & 3]);
        if (vk < n_old || key0 + vk >= nk) Vs[vk * Dh + p.dd] = val;
      }
    }
  };
  // ---- keys of the new positions in a tile: rotate, round, append to the cache, use as rounded
  struct NewKey { float k0, k1, v0, v1; float2 c; };
  auto new_count = [&](int t) {
    const int key0 = t * kKeys;
    return min(nk - key0, kKeys) - min(max(pos0 - key0, 0), kKeys);
  };
  auto load_new = [&](int t, int it, NewKey& nw) {
    const int key0 = t * kKeys;
    const int n_old = min(max(pos0 - key0, 0), kKeys);
    const int kk = n_old + it / half, i = it % half;
    const int j = key0 + kk - pos0;
    const float* kr = xrow + (size_t)j * d.ldzx + d.dq + (size_t)kvh * Dh;
    const float* vr = kr + d.dkv;
    nw.c = rope[(size_t)(pos0 + j) * half + i];
    nw.k0 = kr[i]; nw.k1 = kr[i + half]; nw.v0 = vr[i]; nw.v1 = vr[i + half];
  };
  auto store_new = [&](int t, int it, const NewKey& nw) {
    const int key0 = t * kKeys;
    const int n_old = min(max(pos0 - key0, 0), kKeys);
    const int kk = n_old + it / half, i = it % half;
    const int j = key0 + kk - pos0;
    const float klo = round_store(nw.k0 * nw.c.x - nw.k1 * nw.c.y, BF16), khi = round_store(nw.k1 * nw.c.x + nw.k0 * nw.c.y, BF16);
    const float vlo = round_store(nw.v0, BF16), vhi = round_store(nw.v1, BF16);
    Ks[kk * ldk + i] = klo; Ks[kk * ldk + i + half] = khi;
    Vs[kk * Dh + i] = vlo; Vs[kk * Dh + i + half] = vhi;
    if (chunk == (j * G) / kRowsPerBlock) {   // the one row chunk that owns position j writes it
      const size_t at = k_index(d, pt_row, kvh, pos0 + j);
      const size_t v0 = v_index(d, pt_row, kvh, pos0 + j, i), v1 = v_index(d, pt_row, kvh, pos0 + j, i + half);
      if (BF16) {
        uint16_t* kp = static_cast<uint16_t*>(a.kpool) + at;
        uint16_t* vp = static_cast<uint16_t*>(a.vpool);
        kp[i] = (uint16_t)(__float_as_uint(klo) >> 16); kp[i + half] = (uint16_t)(__float_as_uint(khi) >> 16);
        vp[v0] = (uint16_t)(__float_as_uint(vlo) >> 16); vp[v1] = (uint16_t)(__float_as_uint(vhi) >> 16);
      } else {
        float* kp = static_cast<float*>(a.kpool) + at;
        float* vp = static_cast<float*>(a.vpool);
        kp[i] = klo; kp[i + half] = khi; vp[v0] = vlo; vp[v1] = vhi;
      }
    }
  };

  // ---- loads of the prologue, all in flight together
  float qx0[NQ], qx1[NQ];
  float2 qc[NQ];
#pragma unroll
  for (int i = 0; i < NQ; ++i) {
    const int it = tid + 256 * i;
    const int r = it / half, ii = it - r * half, rg = row0 + r;
    qx0[i] = 0.f; qx1[i] = 0.f; qc[i] = make_float2(0.f, 0.f);
    if (r < kRowsPerBlock && rg < row_lim) {
      const int j = rg / G;
      const float* q = xrow + (size_t)j * d.ldzx + (size_t)(kvh * G + rg % G) * Dh;
      qc[i] = rope[(size_t)(pos0 + j) * half + ii];
      qx0[i] = q[ii]; qx1[i] = q[ii + half];
    }
  }
  NewKey nw0;
  const int n_new0 = t_begin < t_end ? new_count(t_begin) * half : 0;   // rotation pairs of new keys in the first tile
  if (tid < n_new0) load_new(t_begin, tid, nw0);
  if (t_begin < t_end && t_begin * kKeys < pos0 && (sp != 0 || a.T > 16)) load_tile(t_begin);
  TR(1);
  // query rows, rotated to their positions and scaled
#pragma unroll
  for (int i = 0; i < NQ; ++i) {
    const int it = tid + 256 * i;
    const int r = it / half, ii = it - r * half;
    if (r < kRowsPerBlock) {
      qs[r * Dh + ii] = (qx0[i] * qc[i].x - qx1[i] * qc[i].y) * scale;
      qs[r * Dh + ii + half] = (qx1[i] * qc[i].x + qx0[i] * qc[i].y) * scale;
    }
  }

  const bool rows_here = row0 + wave * kRowsPerWave < row_lim;
  float mrun[kRowsPerWave], lrun[kRowsPerWave], acc[kRowsPerWave][E];
#pragma unroll
  for (int r = 0; r < kRowsPerWave; ++r) {
    mrun[r] = -INFINITY; lrun[r] = 0.f;
#pragma unroll
    for (int e = 0; e < E; ++e) acc[r][e] = 0.f;
  }

  for (int t = t_begin; t < t_end; ++t) {
    const int key0 = t * kKeys;
    if (t != t_begin) __syncthreads();      // the previous tile has been consumed
    const int n_new = new_count(t) * half;
    if (t == t_begin) {
      if (tid < n_new) store_new(t, tid, nw0);
      for (int it = tid + 256; it < n_new; it += 256) { NewKey nw; load_new(t, it, nw); store_new(t, it, nw); }
    } else {
      for (int it = tid; it < n_new; it += 256) { NewKey nw; load_new(t, it, nw); store_new(t, it, nw); }
    }
    TR(2);
    store_tile(t);
    __syncthreads();
    TR(3);
    if (t + 1 < t_end && (t + 1) * kKeys < pos0) load_tile(t + 1);
    if (!rows_here) continue;               // none of this wavefront's rows exists
    // scores: lane = key
    float sc[kRowsPerWave];
#pragma unroll
    for (int r = 0; r < kRowsPerWave; ++r) sc[r] = 0.f;
#pragma unroll 4
    for (int dd = 0; dd < Dh; dd += 4) {    // (Dh is a multiple of 8)
      float kvv[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) kvv[u] = Ks[lane * ldk + dd + u];
#pragma unroll
      for (int r = 0; r < kRowsPerWave; ++r) {
        const float4 q = *reinterpret_cast<const float4*>(qs + (wave * kRowsPerWave + r) * Dh + dd);
        sc[r] = fmaf(q.x, kvv[0], sc[r]); sc[r] = fmaf(q.y, kvv[1], sc[r]); sc[r] = fmaf(q.z, kvv[2], sc[r]); sc[r] = fmaf(q.w, kvv[3], sc[r]);
      }
    }
    TR(4);
    const int key = key0 + lane;
#pragma unroll
    for (int r = 0; r < kRowsPerWave; ++r) {
      const bool vis = rok[r] && key <= pos0 + rj[r];
      const float sv = vis ? sc[r] : -INFINITY;
      const float mnew = fmaxf(mrun[r], wave_max(sv));
      float pr = 0.f, corr = 1.f;
      if (mnew != -INFINITY) {
        pr = vis ? expf(sv - mnew) : 0.f;
        corr = mrun[r] == -INFINITY ? 0.f : expf(mrun[r] - mnew);
      }
      lrun[r] = lrun[r] * corr + wave_add(pr);
      mrun[r] = mnew;
#pragma unroll
      for (int e = 0; e < E; ++e) acc[r][e] *= corr;
      ps[(wave * kRowsPerWave + r) * kKeys + lane] = pr;
    }
    // (ps is written and read by the same wavefront only)
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    TR(5);
    // output: lane = dimension
#pragma unroll 4
    for (int kk = 0; kk < kKeys; kk += 4) {
      float4 p[kRowsPerWave];
#pragma unroll
      for (int r = 0; r < kRowsPerWave; ++r) p[r] = *reinterpret_cast<const float4*>(ps + (wave * kRowsPerWave + r) * kKeys + kk);
#pragma unroll
      for (int e = 0; e < E; ++e) {
        const int dd = lane + 64 * e;
        if (FULL || dd < Dh) {
          float vv[4];
#pragma unroll
          for (int u = 0; u < 4; ++u) vv[u] = Vs[(kk + u) * Dh + dd];
#pragma unroll
          for (int r = 0; r < kRowsPerWave; ++r) {
            acc[r][e] = fmaf(p[r].x, vv[0], acc[r][e]); acc[r][e] = fmaf(p[r].y, vv[1], acc[r][e]);
            acc[r][e] = fmaf(p[r].z, vv[2], acc[r][e]); acc[r][e] = fmaf(p[r].w, vv[3], acc[r][e]);
          }
        }
      }
    }
  }

  TR(6);
  // ---- results: final when there is one key slice, else partial + merge by the last workgroup
  if (a.n_splits == 1) {
#pragma unroll
    for (int r = 0; r < kRowsPerWave; ++r) {
      const int rg = row0 + wave * kRowsPerWave + r;
      if (rg >= (a.row0 != nullptr ? row_lim : n_rows)) continue;   // (packed rows: what follows is the next sequence's)
      const size_t mrow = rows0 + rj[r];
      const float inv = (rok[r] && lrun[r] > 0.f) ? 1.0f / lrun[r] : 0.f;
#pragma unroll
      for (int e = 0; e < E; ++e) {
        const int dd = lane + 64 * e;
        if (dd < Dh) a.o[mrow * d.dq + (size_t)rq[r] * Dh + dd] = acc[r][e] * inv;
      }
    }
    return;
  }
  const int S = a.n_splits;
#pragma unroll
  for (int r = 0; r < kRowsPerWave; ++r) {
    const int rg = row0 + wave * kRowsPerWave + r;
    if (rg >= n_rows) continue;
    const size_t rid = (((size_t)b * a.T + rj[r]) * d.Hq + rq[r]) * S + sp;
#pragma unroll
    for (int e = 0; e < E; ++e) {
      const int dd = lane + 64 * e;
      if (dd < Dh) a.part_o[rid * Dh + dd] = acc[r][e];
    }
    if (lane == 0) { a.part_ml[rid * 2] = mrun[r]; a.part_ml[rid * 2 + 1] = lrun[r]; }
  }
  // Make the partials visible device-wide (release), then take a ticket; the workgroup that
  // draws the last ticket sees all of them after its acquire fence and merges.
  TR(7);
  __threadfence();
  __syncthreads();
  TR(8);
  int* counter = a.counters + ((size_t)b * d.Hkv + kvh) * row_chunks + chunk;
  if (tid == 0) {
    const int ticket = atomicAdd(counter, 1);
    s_last = ticket == S - 1;
    if (s_last) *counter = 0;   // ready for the next launch (launches on a context are ordered)
  }
  __syncthreads();
  TR(9);
  if (!s_last) return;
  __threadfence();
  TR(10);
  // lane s holds slice s of each of the wavefront's rows (S <= 64); all loads are issued
  // before the first of them is used
  constexpr int kAhead = 4;
  float ms[kRowsPerWave], ls[kRowsPerWave], po[kRowsPerWave][E][kAhead];
  size_t rid0[kRowsPerWave];
#pragma unroll
  for (int r = 0; r < kRowsPerWave; ++r) {
    const int rg = min(row0 + wave * kRowsPerWave + r, n_rows - 1);
    rid0[r] = (((size_t)b * a.T + rg / G) * d.Hq + kvh * G + rg % G) * S;
    const float2 ml = reinterpret_cast<const float2*>(a.part_ml)[rid0[r] + min(lane, S - 1)];
    ms[r] = lane < S ? ml.x : -INFINITY; ls[r] = lane < S ? ml.y : 0.f;
  }
#pragma unroll
  for (int r = 0; r < kRowsPerWave; ++r)
#pragma unroll
    for (int e = 0; e < E; ++e)
#pragma unroll
      for (int u = 0; u < kAhead; ++u)
        po[r][e][u] = a.part_o[(rid0[r] + min(u, S - 1)) * Dh + min(lane + 64 * e, Dh - 1)];
  TR(11);
#pragma unroll
  for (int r = 0; r < kRowsPerWave; ++r) {
    const int rg = row0 + wave * kRowsPerWave + r;
    if (rg >= n_rows) continue;                     // uniform per wavefront
    const float M = wave_max(ms[r]);
    const float ws = ms[r] != -INFINITY ? expf(ms[r] - M) : 0.f;
    const float L = wave_add(ws * ls[r]);
    const int wbits = __float_as_int(ws);
    float out[E];
#pragma unroll
    for (int e = 0; e < E; ++e) out[e] = 0.f;
#pragma unroll
    for (int u = 0; u < kAhead; ++u) {              // slice order: deterministic
      if (u < S) {
        const float w = __int_as_float(__builtin_amdgcn_readlane(wbits, u));
#pragma unroll
        for (int e = 0; e < E; ++e) out[e] = fmaf(w, po[r][e][u], out[e]);
      }
    }
    for (int s0 = kAhead; s0 < S; s0 += kAhead) {
      float pn[E][kAhead];
#pragma unroll
      for (int e = 0; e < E; ++e)
#pragma unroll
        for (int u = 0; u < kAhead; ++u)
          pn[e][u] = a.part_o[(rid0[r] + min(s0 + u, S - 1)) * Dh + min(lane + 64 * e, Dh - 1)];
#pragma unroll
      for (int u = 0; u < kAhead; ++u) {
        if (s0 + u < S) {
          const float w = __int_as_float(__builtin_amdgcn_readlane(wbits, s0 + u));
#pragma unroll
          for (int e = 0; e < E; ++e) out[e] = fmaf(w, pn[e][u], out[e]);
        }
      }
    }
    const size_t mrow = (size_t)b * a.T + rj[r];
    const float inv = (rok[r] && L > 0.f) ? 1.0f / L : 0.f;
#pragma unroll
    for (int e = 0; e < E; ++e) {
      const int dd = lane + 64 * e;
      if (dd < Dh) a.o[mrow * d.dq + (size_t)rq[r] * Dh + dd] = out[e] * inv;
    }
  }
  TR(12);
}

template <int BF16, int E, bool FULL, bool WALK>
static hipError_t launch_attention_f(const Dims& d, const AttnArgs& a, int row_chunks, size_t lds, hipStream_t s) {
  static size_t lds_enabled = 48 * 1024;
  if (lds > lds_enabled) {
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(attention_kernel<BF16, E, FULL, WALK>),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    lds_enabled = lds;
  }
  hipLaunchKernelGGL((attention_kernel<BF16, E, FULL, WALK>), dim3(row_chunks * a.n_splits, d.Hkv, a.B), dim3(256), lds, s, d, a,
                     row_chunks);
  return hipGetLastError();
}
template <int BF16, int E>
static hipError_t launch_attention_t(const Dims& d, const AttnArgs& a, int row_chunks, size_t lds, hipStream_t s) {
  // (a bf16 cache comes here with pages of 16 tokens, and for cross-checks)
  // The registers of whole tiles (float32, 64: 211 against 155, two workgroups per compute unit instead of three) pay in large launches as
  // well.  Item loads under a condition each, and now: 64 sequences x 3 positions over 300 keys, head dimension 64 73 -> 46 us, 128
  // 104 -> 72; x 9 over 1000 keys 190 -> 93 and 374 -> 196; a prefill pass of 64 positions each over up to 300 keys 115 -> 83 and 270 -> 160;
  // bf16 with 16-token pages, 128: 90 -> 65, 298 -> 167 and 228 -> 153.
  if (!BF16 && d.Dh == 64 * E) return launch_attention_f<BF16, E, !BF16, false>(d, a, row_chunks, lds, s);
  // Places of the items walked where the registers they take cost a workgroup per compute unit in launches of many.  Float32,
  // head dimensions 72 to 120 (256 + 41 registers against 213: one against two), head dimension 96: prefill of 64 x 300 positions
  // 2570 -> 1480 us, of 256 x 100 1850 -> 996, verification of 64 x 9 positions over 1000 keys 300 -> 189, of one sequence the
  // same, of 64 x 3 over 300 keys 65.9 -> 67.5.  Head dimensions below 64, bf16 64 as well (203 to 233 registers against 147 to
  // 159: two against three), prefill: float32, 40, 256 x 100 positions 605 -> 452 us, bf16, 64, 694 -> 530; not verification (64 x 9
  // positions over 1000 keys, float32 96 against 104 us walked, bf16 104 against 109), nor where no workgroup is gained (bf16,
  // 128: prefill of 64 x 300 positions 1510 against 1554 us walked; float32, 200: 2503 against 2610).
  if constexpr (!BF16 && E == 2) return launch_attention_f<BF16, E, false, true>(d, a, row_chunks, lds, s);
  else if (E == 1 && a.T > 16) return launch_attention_f<BF16, E, false, E == 1>(d, a, row_chunks, lds, s);
  else return launch_attention_f<BF16, E, false, false>(d, a, row_chunks, lds, s);
}

// Keys and values of the new positions: rotate k, round to the storage type, write to the pages.
// grid: one workgroup per (sequence, new position).
__global__ __launch_bounds__(256) void kv_append_kernel(const Dims d, const AttnArgs a) {
  const int m = blockIdx.x, b = m / a.T, j = m - b * a.T;
  const int nt = a.n_tok != nullptr ? a.n_tok[b] : a.T;
  if (j >= nt) return;
  const int pos = a.pos0[b] + j;
  const int Dh = d.Dh, half = Dh >> 1;
  const float* krow = a.qkv + (first_row(a.row0, b, a.T) + j) * d.ldzx + d.dq;
  const float* vrow = krow + d.dkv;
  const int* pt_row = a.page_table + (size_t)b * d.pages_per_seq;
  const float2* cs = reinterpret_cast<const float2*>(a.rope) + (size_t)pos * half;
  for (int it = threadIdx.x; it < d.Hkv * half; it += 256) {
    const int kvh = it / half, i = it - kvh * half;
    const float2 c = cs[i];
    const float x0 = krow[kvh * Dh + i], x1 = krow[kvh * Dh + i + half];
    const float lo = x0 * c.x - x1 * c.y, hi = x1 * c.x + x0 * c.y;
    const size_t at = k_index(d, pt_row, kvh, pos);
    if (d.bf16) {
      uint16_t* kp = static_cast<uint16_t*>(a.kpool) + at;
      kp[i] = f32_to_bf16_rne(lo); kp[i + half] = f32_to_bf16_rne(hi);
    } else {
      float* kp = static_cast<float*>(a.kpool) + at;
      kp[i] = lo; kp[i + half] = hi;
    }
  }
  for (int it = threadIdx.x; it < d.Hkv * Dh; it += 256) {
    const int kvh = it / Dh, dd = it - kvh * Dh;
    const size_t at = v_index(d, pt_row, kvh, pos, dd);
    if (d.bf16) static_cast<uint16_t*>(a.vpool)[at] = f32_to_bf16_rne(vrow[it]);
    else static_cast<float*>(a.vpool)[at] = vrow[it];
  }
}

// The same for a bf16 cache whose pages hold a multiple of 8 tokens, in groups of 8 consecutive positions
// (aligned to 8, so a group lies in one page): the values of one dimension for the 8 tokens are 16 contiguous
// bytes of the transposed V page and are written as one store (the kernel above writes them as 8 separate
// 2-byte stores from 8 workgroups).  Same arithmetic and rounding.  grid: x = sequence x groups_per_seq, y = the items
// of a group (values of a dimension, then rotation pairs of keys), one per thread: each is a chain of memory round trips,
// so that loops over them cost a launch of one sequence 9 us (now 5).
__global__ __launch_bounds__(256) void kv_append8_kernel(const Dims d, const AttnArgs a, int groups_per_seq) {
  const int b = blockIdx.x / groups_per_seq, gl = blockIdx.x - b * groups_per_seq;
  const int nt = min(a.n_tok != nullptr ? a.n_tok[b] : a.T, a.T);
  const int pos0 = a.pos0[b];
  const int p_first = ((pos0 >> 3) + gl) << 3;               // first position of this group
  if (nt <= 0 || p_first >= pos0 + nt) return;
  const int Dh = d.Dh, half = Dh >> 1;
  const int* pt_row = a.page_table + (size_t)b * d.pages_per_seq;
  const float* rows = a.qkv + first_row(a.row0, b, a.T) * d.ldzx + d.dq;   // row j: k | v of position pos0 + j
  const bool whole = p_first >= pos0 && p_first + 8 <= pos0 + nt;
  uint16_t* vpool = static_cast<uint16_t*>(a.vpool);
  uint16_t* kpool = static_cast<uint16_t*>(a.kpool);
  const int per = d.Hkv * half, n_v = d.Hkv * Dh;
  const int item = blockIdx.y * 256 + threadIdx.x;
  if (item >= n_v + 8 * per) return;
  if (item < n_v) {
    const int it = item, kvh = it / Dh, dd = it - kvh * Dh;
    const size_t at = v_index(d, pt_row, kvh, p_first, dd);
    if (whole) {
      uint32_t h[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) h[u] = f32_to_bf16_rne(rows[(size_t)(p_first - pos0 + u) * d.ldzx + d.dkv + it]);
      *reinterpret_cast<uint4*>(vpool + at) = make_uint4(h[0] | (h[1] << 16), h[2] | (h[3] << 16), h[4] | (h[5] << 16), h[6] | (h[7] << 16));
    } else {
      for (int u = 0; u < 8; ++u) {
        const int j = p_first + u - pos0;
        if (j >= 0 && j < nt) vpool[at + u] = f32_to_bf16_rne(rows[(size_t)j * d.ldzx + d.dkv + it]);
      }
    }
    return;
  }
  const int it = item - n_v, u = it / per, rem = it - u * per, kvh = rem / half, i = rem - kvh * half;
  const int pos = p_first + u, j = pos - pos0;
  if (j < 0 || j >= nt) return;
  const float2 c = reinterpret_cast<const float2*>(a.rope)[(size_t)pos * half + i];
  const float* krow = rows + (size_t)j * d.ldzx;
  const float x0 = krow[kvh * Dh + i], x1 = krow[kvh * Dh + i + half];
  const float lo = x0 * c.x - x1 * c.y, hi = x1 * c.x + x0 * c.y;
  uint16_t* kp = kpool + k_index(d, pt_row, kvh, pos);
  kp[i] = f32_to_bf16_rne(lo); kp[i + half] = f32_to_bf16_rne(hi);
}

// bf16 cache: matrix-core kernel (HH_KF_ATTN_SCALAR selects the float32-FMA kernel instead, for cross-checks)
bool attention_uses_mfma(const Dims& d) {
  return d.bf16 && !(d.flags & HH_KF_ATTN_SCALAR) && d.page_tokens % 32 == 0;   // a 32-key step of that kernel lies in one page
}

hipError_t launch_attention(const Dims& d, const AttnArgs& a, hipStream_t s) {
  if (d.Dh > kMaxDh || d.Dh % 8 != 0 || a.n_splits > 64 || a.n_splits < 1 || a.T < 1 || a.B < 1 || (a.row0 != nullptr && a.n_splits != 1)) return hipErrorInvalidValue;
  if (attention_uses_mfma(d)) {
    if (!attention_mfma_fuses_append(d, a.T)) {
      if (a.T >= 16 && d.page_tokens % 8 == 0) {
        const int groups = (a.T + 7) / 8 + 1;      // 8-aligned groups that T consecutive positions can touch
        // an item per thread: each is a chain of page number, inputs and store
        const int parts = (d.Hkv * d.Dh * 5 + 255) / 256;
        hipLaunchKernelGGL(kv_append8_kernel, dim3(a.B * groups, parts), dim3(256), 0, s, d, a, groups);
      } else {
        hipLaunchKernelGGL(kv_append_kernel, dim3(a.B * a.T), dim3(256), 0, s, d, a);
      }
      hipError_t e = hipGetLastError();
      if (e != hipSuccess) return e;
    }
    return launch_attention_mfma(d, a, s);
  }
  const int G = d.Hq / d.Hkv;
  const int row_chunks = (a.T * G + kRowsPerBlock - 1) / kRowsPerBlock;
  const size_t lds = ((size_t)kKeys * (d.Dh + 1) + (size_t)kKeys * d.Dh + (size_t)kRowsPerBlock * d.Dh +
                      4 * kRowsPerWave * kKeys) * sizeof(float);
  const int E = (d.Dh + 63) / 64;
  if (d.bf16) {
    if (E == 1) return launch_attention_t<1, 1>(d, a, row_chunks, lds, s);
    if (E == 2) return launch_attention_t<1, 2>(d, a, row_chunks, lds, s);
    return launch_attention_t<1, 4>(d, a, row_chunks, lds, s);
  }
  if (E == 1) return launch_attention_t<0, 1>(d, a, row_chunks, lds, s);
  if (E == 2) return launch_attention_t<0, 2>(d, a, row_chunks, lds, s);
  return launch_attention_t<0, 4>(d, a, row_chunks, lds, s);
}

// upper bound on the row chunks of either kernel (sizes the ticket counters)
int attention_row_chunks(const Dims& d, int T) { return (T * (d.Hq / d.Hkv) + kRowsPerBlock - 1) / kRowsPerBlock; }

__global__ void export_kv_kernel(const Dims d, const LayerDev* layer, const int* page_table, int seq, int tok0,
                                 int n_tokens, float* k, float* v) {
  const int* pt_row = page_table + (size_t)seq * d.pages_per_seq;
  const size_t total = (size_t)n_tokens * d.Hkv * d.Dh;
  for (size_t it = blockIdx.x * (size_t)blockDim.x + threadIdx.x; it < total; it += (size_t)gridDim.x * blockDim.x) {
    const int dd = it % d.Dh, kvh = (it / d.Dh) % d.Hkv, pos = tok0 + (int)(it / ((size_t)d.Dh * d.Hkv));
    const size_t at = k_index(d, pt_row, kvh, pos) + dd, vat = v_index(d, pt_row, kvh, pos, dd);
    if (d.bf16) {
      k[it] = __uint_as_float((uint32_t) static_cast<const uint16_t*>(layer->kpool)[at] << 16);
      v[it] = __uint_as_float((uint32_t) static_cast<const uint16_t*>(layer->vpool)[vat] << 16);
    } else {
      k[it] = static_cast<const float*>(layer->kpool)[at];
      v[it] = static_cast<const float*>(layer->vpool)[vat];
    }
  }
}

hipError_t launch_export_kv(const Dims& d, const LayerDev* layer, const int* page_table, int seq, int tok0,
                            int n_tokens, float* k, float* v, hipStream_t s) {
  if (n_tokens <= 0) return hipSuccess;
  hipLaunchKernelGGL(export_kv_kernel, dim3(64), dim3(256), 0, s, d, layer, page_table, seq, tok0, n_tokens, k, v);
  return hipGetLastError();
}

}  // namespace hh
