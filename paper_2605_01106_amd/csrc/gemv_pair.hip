// Two skinny products of the same rows in one launch (see gemv.hip for the kernel).
#include "gemv_kernel.h"

namespace hh {

template <int BF16, int MT, int R, int NCW, int KS>
static hipError_t launch_one(const GemvArgs& a, const GemvArgs& b, const GemvPlan& pa, const GemvPlan& pb, hipStream_t s) {
  auto kern = gemv_pair_kernel<BF16, MT, R, NCW, KS>;
  const size_t lds = pa.lds > pb.lds ? pa.lds : pb.lds;
  static size_t lds_enabled = 48 * 1024;
  if (lds > lds_enabled) {
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    lds_enabled = lds;
  }
  hipLaunchKernelGGL(kern, dim3(pa.blocks + pb.blocks), dim3(kGemvThreads), lds, s, a, b, pa.iters, pb.iters, pa.blocks);
  return hipGetLastError();
}
template <int BF16, int MT, int R>
static hipError_t launch_ks(const GemvArgs& a, const GemvArgs& b, const GemvPlan& pa, const GemvPlan& pb, hipStream_t s) {
  if (pa.NCW == 2 && pa.KS == 1) return launch_one<BF16, MT, R, 2, 1>(a, b, pa, pb, s);
  if (pa.NCW == 2 && pa.KS == 2) return launch_one<BF16, MT, R, 2, 2>(a, b, pa, pb, s);
  if (pa.NCW == 2 && pa.KS == 4) return launch_one<BF16, MT, R, 2, 4>(a, b, pa, pb, s);
  if (pa.NCW == 4 && pa.KS == 4) return launch_one<BF16, MT, R, 4, 4>(a, b, pa, pb, s);
  return hipErrorInvalidValue;
}

// bf16 weights: up to 3 rows (more take the matrix cores); float32: up to 8
bool gemv_pair_fits(const GemvArgs& a, const GemvArgs& b) {
  GemvPlan pa, pb;
  return (!a.bf16 || a.M <= 3) && gemv_pair_plan(a, b, pa, pb);
}

hipError_t launch_gemv_pair(const GemvArgs& a, const GemvArgs& b, hipStream_t s) {
  GemvPlan pa, pb;
  if (!gemv_pair_fits(a, b) || !gemv_pair_plan(a, b, pa, pb)) return hipErrorInvalidValue;
  switch (a.bf16 * 256 + pa.MT * 16 + pa.R) {
    case 0x111: return launch_ks<1, 1, 1>(a, b, pa, pb, s);
    case 0x112: return launch_ks<1, 1, 2>(a, b, pa, pb, s);
    case 0x114: return launch_ks<1, 1, 4>(a, b, pa, pb, s);
    case 0x131: return launch_ks<1, 3, 1>(a, b, pa, pb, s);
    case 0x132: return launch_ks<1, 3, 2>(a, b, pa, pb, s);
    case 0x134: return launch_ks<1, 3, 4>(a, b, pa, pb, s);
    case 0x011: return launch_ks<0, 1, 1>(a, b, pa, pb, s);
    case 0x031: return launch_ks<0, 3, 1>(a, b, pa, pb, s);
    case 0x051: return launch_ks<0, 5, 1>(a, b, pa, pb, s);
    case 0x081: return launch_ks<0, 8, 1>(a, b, pa, pb, s);
  }
  return hipErrorInvalidValue;
}

}  // namespace hh
