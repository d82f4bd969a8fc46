// attn.hip -- the attention instances and their host-side dispatch (kernel in
// attn_kernel.h).  Compiled with MFMA results in VGPRs: with accumulators in
// AGPRs the instances of three and four row tiles, and fp32 from two, need more
// than the 512 registers of a lane or copy every score out of an AGPR.
// Measured, accumulators in AGPRs -> VGPRs: 8-token verify of 32 x 4096, G = 8
// (four row tiles) 119 -> 107 us, 5-token 64 x 16384-32768, G = 8 (three)
// 1122 -> 1009, fp32 8-token 64 x 2048, G = 8 739 -> 330; two row tiles then
// fit 256 registers, so two workgroups share a compute unit (48 x 2000: 90 ->
// 77).  The exceptions are in attn_agpr.hip.
#include <atomic>

#include "attn_kernel.h"

namespace md {

// ---------------------------------------------------------------------------
// Host-side dispatch over the compiled instances.

template <int D, bool BF16, int NT, bool IDX, int P, int OCC, bool BAL = false, int W = kWaves,
          bool CONTIGUOUS = true>
static hipError_t launch_p(const AttnParams& p, bool paged, int64_t n_blocks, hipStream_t s) {
  dim3 grid(static_cast<uint32_t>(n_blocks)), block(W * 64);
  if (paged)
    hipLaunchKernelGGL((attn_partial_kernel<D, BF16, NT, true, IDX, P, OCC, BAL, W>), grid, block,
                       0, s, p);
  else if constexpr (CONTIGUOUS)
    hipLaunchKernelGGL((attn_partial_kernel<D, BF16, NT, false, IDX, P, OCC, BAL, W>), grid, block,
                       0, s, p);
  else
    return hipErrorInvalidValue;
  return hipGetLastError();
}

// Instances: tiles in flight per wave (depth) x waves per SIMD (occupancy).
// Two waves per SIMD fit the register file with one tile in flight and up to
// two row tiles; a second tile in flight is built for the bf16 range modes
// with up to three row tiles (MD_PREFETCH_DEPTH); everything else runs one
// tile, one wave per SIMD.
template <int D, bool BF16, int NT, bool IDX>
static hipError_t launch_nt(const AttnParams& p, bool paged, int depth, int occ,
                            int64_t n_blocks, hipStream_t s) {
  // Verifies that run faster with their accumulators in AGPRs.
  constexpr bool kAgpr = D == 128 && BF16 && !IDX;
  if constexpr (kAgpr && NT == 2)
    if (p.bal) return launch_attn_agpr(p, NT, paged, n_blocks, s);
  if constexpr (kAgpr && NT == 3)
    if (!paged && p.mode == MD_MODE_VERIFY && (p.bal || (depth < 2 && p.waves == kWaves)))
      return launch_attn_agpr(p, NT, paged, n_blocks, s);
  // The balanced verify: one tile in flight, the verify's default waves per
  // SIMD (two for one row tile of bf16, else one).  Compiled only where its
  // piece loop fits the registers without spilling (bf16 up to three row
  // tiles, fp32 up to two); the planner never chooses it elsewhere.
  if constexpr (!IDX && NT <= kBalMaxNT(BF16) && !(kAgpr && NT == 2)) {
    if (p.bal) {
      (void)depth;
      (void)occ;
      return launch_p<D, BF16, NT, IDX, 1, (BF16 && NT == 1) ? 2 : 1, true, kWaves,
                      !(kAgpr && NT == 3)>(p, paged, n_blocks, s);
    }
  } else {
    if (p.bal) return hipErrorInvalidValue;
  }
  if constexpr (BF16 && NT <= 2 && !IDX) {
    // Eight waves in one workgroup, two per SIMD (the registers of up to two
    // row tiles allow it, 248 at two): each takes half as many of the unit's
    // tiles.  Their merge buffers fill 140 KB of LDS at two row tiles.
    if (p.waves == kWavesWide)
      return launch_p<D, BF16, NT, IDX, 1, 2, false, kWavesWide>(p, paged, n_blocks, s);
  }
  if (p.waves != kWaves) return hipErrorInvalidValue;
  if constexpr (BF16) {
    if constexpr (!IDX && NT <= 3)
      if (depth >= 2) return launch_p<D, BF16, NT, IDX, 2, 1>(p, paged, n_blocks, s);
    if constexpr (NT <= 2)
      if (occ >= 2) return launch_p<D, BF16, NT, IDX, 1, 2>(p, paged, n_blocks, s);
    return launch_p<D, BF16, NT, IDX, 1, 1>(p, paged, n_blocks, s);
  } else {
    (void)depth;  // fp32 serves small problems: one tile in flight
    (void)occ;
    return launch_p<D, BF16, NT, IDX, 1, 1>(p, paged, n_blocks, s);
  }
}

template <int D, bool BF16, bool IDX>
static hipError_t launch_d(const AttnParams& p, int NT, bool paged, int depth, int occ,
                           int64_t n_blocks, hipStream_t s) {
  switch (NT) {
    case 1: return launch_nt<D, BF16, 1, IDX>(p, paged, depth, occ, n_blocks, s);
    case 2: return launch_nt<D, BF16, 2, IDX>(p, paged, depth, occ, n_blocks, s);
    case 3: return launch_nt<D, BF16, 3, IDX>(p, paged, depth, occ, n_blocks, s);
    case 4: return launch_nt<D, BF16, 4, IDX>(p, paged, depth, occ, n_blocks, s);
  }
  return hipErrorInvalidValue;
}

template <bool IDX>
static hipError_t launch_i(const AttnParams& p, int head_dim, bool bf16, int NT, bool paged,
                           int depth, int occ, int64_t n_blocks, hipStream_t s) {
  if (head_dim == 128)
    return bf16 ? launch_d<128, true, IDX>(p, NT, paged, depth, occ, n_blocks, s)
                : launch_d<128, false, IDX>(p, NT, paged, depth, occ, n_blocks, s);
  return bf16 ? launch_d<64, true, IDX>(p, NT, paged, depth, occ, n_blocks, s)
              : launch_d<64, false, IDX>(p, NT, paged, depth, occ, n_blocks, s);
}

// The instances live in two code objects, this file's and attn_agpr.hip's, and the
// runtime loads one at its first launch: a verify would load the one and the
// first draft after it the other, a stall of 6 ms in the middle of a run, with
// slower clocks for ten steps behind it (1400 -> 1250 us a verify).  So the first
// attention call on a device loads both (asking for a kernel's attributes does).
static void load_instances(hipStream_t s) {
  static std::atomic<uint64_t> loaded{0};
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return;
  const uint64_t bit = uint64_t{1} << dev;
  if (loaded.load(std::memory_order_relaxed) & bit) return;
  hipStreamCaptureStatus capture = hipStreamCaptureStatusNone;
  hipError_t e = hipStreamIsCapturing(s, &capture);
  if (e == hipSuccess && capture == hipStreamCaptureStatusNone) {
    hipFuncAttributes attr;
    e = hipFuncGetAttributes(
        &attr, reinterpret_cast<const void*>(
                   &attn_partial_kernel<128, true, 1, false, false, 1, 2, false, kWaves>));
    if (e == hipSuccess) e = hipFuncGetAttributes(&attr, attn_agpr_kernel());
    loaded.fetch_or(bit, std::memory_order_relaxed);
  }
  // A launch reports its own errors; one that was pending before is the caller's.
  if (e != hipSuccess) (void)hipGetLastError();
}

hipError_t launch_attn_partial(const AttnParams& p, int head_dim, bool bf16, int NT, bool paged,
                               int depth, int occ, int64_t n_blocks, hipStream_t s) {
  if (n_blocks <= 0) return hipSuccess;
  load_instances(s);
  if (p.mode == MD_MODE_DRAFT_INDEXED)
    return launch_i<true>(p, head_dim, bf16, NT, paged, depth, occ, n_blocks, s);
  return launch_i<false>(p, head_dim, bf16, NT, paged, depth, occ, n_blocks, s);
}

}  // namespace md
