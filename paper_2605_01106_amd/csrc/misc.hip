// Small kernels of the round protocol: token gathering and embedding lookup, the final
// step of the LM-head argmax, greedy acceptance with its bookkeeping, and helpers for
// prefill.  All token ids, lengths and counts stay on the device between the calls of a
// round; nothing here is read back by the host.
#include "hh_internal.h"

namespace hh {

// A row of the embedding as float32, by a whole workgroup (D % 8 == 0; an id that is no token reads a valid row, never
// out of bounds).
__device__ __forceinline__ void embed_row(const void* embed, int bf16, int tok, int D, int V, float* h) {
  const size_t src = (size_t)min(max(tok, 0), V - 1) * D;
  if ((reinterpret_cast<uintptr_t>(embed) & 15) != 0) {   // (the caller's matrix: no alignment is asked of it)
    for (int k = threadIdx.x; k < D; k += blockDim.x)
      h[k] = bf16 ? __uint_as_float((uint32_t) static_cast<const uint16_t*>(embed)[src + k] << 16) : static_cast<const float*>(embed)[src + k];
    return;
  }
  for (int k = threadIdx.x * 4; k < D; k += blockDim.x * 4) {
    float4 v;
    if (bf16) {
      const uint2 u = *reinterpret_cast<const uint2*>(static_cast<const uint16_t*>(embed) + src + k);
      v = make_float4(__uint_as_float(u.x << 16), __uint_as_float(u.x & 0xffff0000u), __uint_as_float(u.y << 16),
                      __uint_as_float(u.y & 0xffff0000u));
    } else {
      v = *reinterpret_cast<const float4*>(static_cast<const float*>(embed) + src + k);
    }
    *reinterpret_cast<float4*>(h + k) = v;
  }
}

// Start of a pass, one workgroup per row m = b*T + j: the row's token, its embedding into h[m], the position of the
// sequence's first row, and a cleared argmax key of the row (the many-row LM heads raise them with atomic maxima).
//   PASS_DRAFT   draft step `step`: pending[b] at step 0, else drafts[b][step-1]; position kv_len[b] + step
//   PASS_VERIFY  pending[b], drafts[b][j-1]; position kv_len[b]
//   PASS_PROMPT  prompt[b][off + j] for j < n_tok[b] (token 0 beyond, or no row at all: row0); position kv_len[b]
__global__ __launch_bounds__(256) void begin_pass_kernel(const PassArgs a) {
  const int m = blockIdx.x, b = m / a.T, j = m - b * a.T;
  int tok;
  if (a.mode == PASS_DRAFT) tok = a.step == 0 ? a.pending[b] : a.drafts[b * a.kmax + a.step - 1];
  else if (a.mode == PASS_VERIFY) tok = j == 0 ? a.pending[b] : a.drafts[b * a.kmax + j - 1];
  else tok = j < a.n_tok[b] ? a.prompt[(size_t)b * a.row_stride + a.off + j] : 0;
  if (threadIdx.x == 0) {
    if (j == 0) a.pos0[b] = a.kv_len[b] + (a.mode == PASS_DRAFT ? a.step : 0);
    if (a.clear != nullptr) a.clear[m] = 0ull;
  }
  if (a.row0 != nullptr && j >= a.n_tok[b]) return;
  embed_row(a.embed, a.bf16, tok, a.D, a.V, a.h + (first_row(a.row0, b, a.T) + j) * a.D);
}

hipError_t launch_begin_pass(const PassArgs& a, int B, hipStream_t s) {
  if (B * a.T <= 0) return hipSuccess;
  hipLaunchKernelGGL(begin_pass_kernel, dim3(B * a.T), dim3(256), 0, s, a);
  return hipGetLastError();
}

// Reduce the per-workgroup argmax partials of the LM head: row m = b*T + j -> out[b*out_stride + out_off + j].
// next.h != nullptr (draft steps, T = 1): the workgroup also begins the next step of its sequence with the token it has
// just found (position kv_len[b] + next.step, embedding, cleared key), which saves that step's first launch.
__global__ __launch_bounds__(256) void argmax_finish_kernel(const unsigned long long* best, int n_part, int M, int* out, int out_stride,
                                                            int out_off, int T, const PassArgs next) {
  const int m = blockIdx.x;
  unsigned long long v = 0ull;
  for (int i = threadIdx.x; i < n_part; i += blockDim.x) v = max(v, best[(size_t)m * n_part + i]);
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v = max(v, (unsigned long long)__shfl_xor((long long)v, o, 64));
  __shared__ unsigned long long w[4];
  if ((threadIdx.x & 63) == 0) w[threadIdx.x >> 6] = v;
  __syncthreads();
  v = max(max(w[0], w[1]), max(w[2], w[3]));
  const int tok = (int)(0xFFFFFFFFu - (uint32_t)(v & 0xFFFFFFFFull));
  if (threadIdx.x == 0) {
    const int b = m / T, j = m % T;
    out[(size_t)b * out_stride + out_off + j] = tok;
  }
  if (next.h == nullptr) return;
  if (threadIdx.x == 0) {
    next.pos0[m] = next.kv_len[m] + next.step;
    if (next.clear != nullptr) next.clear[m] = 0ull;      // (n_part = 1 then: the key this workgroup alone has read)
  }
  embed_row(next.embed, next.bf16, tok, next.D, next.V, next.h + (size_t)m * next.D);
}

hipError_t launch_argmax_finish(const unsigned long long* best, int n_part, int M, int* out, int out_stride,
                                int out_off, int T, const PassArgs* next, hipStream_t s) {
  hipLaunchKernelGGL(argmax_finish_kernel, dim3(M), dim3(256), 0, s, best, n_part, M, out, out_stride, out_off, T,
                     next != nullptr ? *next : PassArgs{});
  return hipGetLastError();
}

// Greedy acceptance (longest prefix with drafts[i] == targets[i]) or a forced count, then the
// bookkeeping of the commit: emitted tokens, pending token, committed count.  The cache length
// is advanced later (after the state rebuild has used it) by adding adv[b].
__global__ void accept_kernel(const CommitArgs a) {
  const int b = blockIdx.x * blockDim.x + threadIdx.x;
  if (b >= a.B) return;
  const int done = a.committed[b] >= a.G;
  a.skip[b] = done;
  if (done) { a.n_acc[b] = 0; a.adv[b] = 0; return; }
  const int* d = a.drafts + (size_t)b * a.kmax;
  const int* g = a.targets + (size_t)b * (a.kmax + 1);
  int n = 0;
  if (a.forced != nullptr) {
    n = min(max(a.forced[b], 0), a.k);
  } else {
    while (n < a.k && d[n] == g[n]) ++n;
  }
  int c = a.committed[b];
  int* row = a.out_tok + (size_t)b * a.out_stride;    // the committed count, then the tokens
  int* out = row + 1;
  for (int i = 0; i < n && c < a.G; ++i) out[c++] = d[i];
  if (c < a.G) out[c++] = g[n];
  a.committed[b] = c;
  row[0] = c;
  a.pending[b] = g[n];
  a.last_n[b] = n;
  a.n_acc[b] = n;
  a.adv[b] = n + 1;
  // acceptance statistics: drafts 1..n passed their test, draft n+1 (if there is one) failed it
  if (a.acc_stats != nullptr && a.k > 0) {
    atomicAdd(a.acc_stats, (unsigned long long)n);
    atomicAdd(a.acc_stats + 1, (unsigned long long)min(n + 1, a.k));
  }
}

hipError_t launch_accept(const CommitArgs& a, hipStream_t s) {
  hipLaunchKernelGGL(accept_kernel, dim3((a.B + 63) / 64), dim3(64), 0, s, a);
  return hipGetLastError();
}

__global__ void advance_kernel(int* kv_len, const int* n, int B) {
  const int b = blockIdx.x * blockDim.x + threadIdx.x;
  if (b < B) kv_len[b] += n[b];
}

hipError_t launch_advance(int* kv_len, const int* n, int B, hipStream_t s) {
  hipLaunchKernelGGL(advance_kernel, dim3((B + 63) / 64), dim3(64), 0, s, kv_len, n, B);
  return hipGetLastError();
}

// After a prefill pass: keep the stream of each sequence's last prompt position (input of the
// LM head) and advance the cache length by the positions consumed.
__global__ void prefill_tail_kernel(const float* h, int T, int D, const int* n_tok, const int* row0, const int* is_last, float* lasth,
                                    int* kv_len) {
  const int b = blockIdx.x;
  const int nt = n_tok[b];
  if (nt > 0 && is_last[b]) {
    const float* src = h + (first_row(row0, b, T) + nt - 1) * D;
    for (int k = threadIdx.x; k < D; k += blockDim.x) lasth[(size_t)b * D + k] = src[k];
  }
  if (threadIdx.x == 0) kv_len[b] += nt;
}

hipError_t launch_prefill_tail(const float* h, int T, int D, const int* n_tok, const int* row0, const int* is_last, float* lasth,
                               int* kv_len, int B, hipStream_t s) {
  hipLaunchKernelGGL(prefill_tail_kernel, dim3(B), dim3(256), 0, s, h, T, D, n_tok, row0, is_last, lasth, kv_len);
  return hipGetLastError();
}

// First generated token: pending, first entry of the output (behind its count), committed = 1
__global__ void prefill_finish_kernel(const int* first_tok, int* pending, int* out_tok, int out_stride, int* committed,
                                      int* last_n, int B) {
  const int b = blockIdx.x * blockDim.x + threadIdx.x;
  if (b >= B) return;
  pending[b] = first_tok[b];
  out_tok[(size_t)b * out_stride] = 1;
  out_tok[(size_t)b * out_stride + 1] = first_tok[b];
  committed[b] = 1;
  last_n[b] = 0;
}

hipError_t launch_prefill_finish(const int* first_tok, int* pending, int* out_tok, int out_stride, int* committed,
                                 int* last_n, int B, hipStream_t s) {
  hipLaunchKernelGGL(prefill_finish_kernel, dim3((B + 63) / 64), dim3(64), 0, s, first_tok, pending, out_tok, out_stride,
                     committed, last_n, B);
  return hipGetLastError();
}

__global__ void fill_i32_kernel(int* p, int v, size_t n) {
  for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x) p[i] = v;
}
__global__ void fill_f32_kernel(float* p, float v, size_t n) {
  for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x) p[i] = v;
}

hipError_t launch_fill_i32(int* p, int v, size_t n, hipStream_t s) {
  if (n == 0) return hipSuccess;
  const int blocks = (int)((n + 255) / 256 < 4096 ? (n + 255) / 256 : 4096);
  hipLaunchKernelGGL(fill_i32_kernel, dim3(blocks), dim3(256), 0, s, p, v, n);
  return hipGetLastError();
}
hipError_t launch_fill_f32(float* p, float v, size_t n, hipStream_t s) {
  if (n == 0) return hipSuccess;
  const int blocks = (int)((n + 255) / 256 < 4096 ? (n + 255) / 256 : 4096);
  hipLaunchKernelGGL(fill_f32_kernel, dim3(blocks), dim3(256), 0, s, p, v, n);
  return hipGetLastError();
}

}  // namespace hh
