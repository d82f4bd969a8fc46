// attn_agpr.hip -- the attention instances that run faster with their
// accumulators in AGPRs (the compiler's default) than in VGPRs, as attn.hip is
// compiled.  One wave per SIMD has the whole register file either way, but in
// VGPRs these need more than 256 and spill to AGPRs inside the tile loop.  All
// are bf16 verifies, d = 128, MFMA results in VGPRs -> AGPRs:
//   balanced, two row tiles: 5 tokens of 64 x 16384-32768, paged 1033 -> 1011 us
//   three row tiles, contiguous: 5 tokens, G = 8, of 16 x 131072
//       1256 -> 1231 us; balanced, 64 x 16384-32768, 1056 -> 1032
// (paged, whose page addresses cost the AGPR form more, three row tiles stay in
// VGPRs: 16 x 32768 328 us against 354).
#include "attn_kernel.h"

namespace md {

const void* attn_agpr_kernel() {
  return reinterpret_cast<const void*>(
      &attn_partial_kernel<128, true, 2, true, false, 1, 1, true, kWaves, true>);
}

hipError_t launch_attn_agpr(const AttnParams& p, int NT, bool paged, int64_t n_blocks,
                            hipStream_t s) {
  const dim3 grid(static_cast<uint32_t>(n_blocks)), block(kWaves * 64);
  if (NT == 2 && p.bal && paged)
    hipLaunchKernelGGL((attn_partial_kernel<128, true, 2, true, false, 1, 1, true, kWaves, true>),
                       grid, block, 0, s, p);
  else if (NT == 2 && p.bal)
    hipLaunchKernelGGL((attn_partial_kernel<128, true, 2, false, false, 1, 1, true, kWaves, true>),
                       grid, block, 0, s, p);
  else if (NT == 3 && !paged && p.bal)
    hipLaunchKernelGGL((attn_partial_kernel<128, true, 3, false, false, 1, 1, true, kWaves, true>),
                       grid, block, 0, s, p);
  else if (NT == 3 && !paged)
    hipLaunchKernelGGL((attn_partial_kernel<128, true, 3, false, false, 1, 1, false, kWaves,
                                            true>),
                       grid, block, 0, s, p);
  else
    return hipErrorInvalidValue;
  return hipGetLastError();
}

}  // namespace md
