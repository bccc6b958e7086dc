// Launch of split-K units by themselves: one workgroup per (unit, block of kv heads).
#include "splitk_unit.h"

namespace tl {

namespace {

template <int VREAD>
__global__ __launch_bounds__(unit::kThreads) void splitk_unit_attn_kernel(const AttnArgs a) {
  extern __shared__ __attribute__((aligned(16))) uint16_t lds[];
  unit::splitk_unit<VREAD, false>(a, a.work[blockIdx.x], blockIdx.y, lds);
}

}  // namespace

tl_status launch_splitk_units(const AttnArgs& a, int n_work, hipStream_t st) {
  if (n_work == 0) return TL_OK;
  if (!unit::can_deal(a))
    TL_FAIL(TL_EINVAL, "launch_splitk_units: %d kv heads cannot be dealt %d to a workgroup", a.kv_heads, 1 << a.unit_heads_log2);
  const dim3 grid((unsigned)n_work, (unsigned)unit_head_blocks(a.kv_heads, a.unit_heads_log2)), block(unit::kThreads);
  static std::atomic<uint64_t> allowed[2];
  const bool scalar_v = get_option_vread() != 0;
  auto kern = scalar_v ? splitk_unit_attn_kernel<1> : splitk_unit_attn_kernel<0>;
  const tl_status rc = allow_lds((const void*)kern, unit::kLdsBytes, allowed[scalar_v]);
  if (rc != TL_OK) return rc;
  hipLaunchKernelGGL(kern, grid, block, unit::kLdsBytes, st, a);
  TL_HIP(hipGetLastError());
  return TL_OK;
}

}  // namespace tl
