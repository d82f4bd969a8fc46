// merge.hip -- log-sum-exp merge of attention partials computed over
// disjoint key sets: the second phase of the split-KV decomposition (the
// Flash-Decoding identity the paper cites in Sec. 2), and the public
// md_merge_lse.
//
// One wave per row.  The part count is small (tens), so each lane first
// scans the lse values for the row maximum and the normaliser, then the wave
// walks the parts in order, each lane owning d/64 channels of the row.  Parts
// with lse = -inf are skipped without reading their O.  When every part's O is
// readable (the library's own split plans, which write every part) and there
// are at most kRegParts parts, each lane instead issues the loads of all lse
// values and of its channels of every part at once and combines them from
// registers: one memory round trip instead of two dependent ones.
#include <hip/hip_runtime.h>

#include "kernels.h"

namespace md {

typedef float f32x2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ uint32_t merge_f32_to_bf16(float f) {
  uint32_t u = __float_as_uint(f);
  if ((u & 0x7fffffffu) > 0x7f800000u) return (u >> 16) | 0x40u;
  u += 0x7fffu + ((u >> 16) & 1u);
  return u >> 16;
}

constexpr int kRegParts = 8;

template <int D, bool OUT_BF16, bool REG>
__global__ void __launch_bounds__(256)
merge_lse_kernel(int n_parts, int64_t n_rows, const float* __restrict__ o_parts,
                 const float* __restrict__ lse_parts, void* __restrict__ o,
                 float* __restrict__ lse) {
  constexpr float kLog2e = 1.44269504088896340736f;
  constexpr float kLn2 = 0.69314718055994530942f;
  constexpr int CPL = D / 64;  // channels per lane
  const int lane = threadIdx.x & 63;
  const int64_t row = static_cast<int64_t>(blockIdx.x) * 4 + (threadIdx.x >> 6);
  if (row >= n_rows) return;

  if constexpr (REG) {
    // n_parts <= kRegParts, every part's O readable: all loads first.
    float lv[kRegParts];
    float xo[kRegParts][CPL];
    for (int k = 0; k < kRegParts; ++k) {
      if (k < n_parts) {
        lv[k] = lse_parts[k * n_rows + row];
        const float* src = o_parts + (k * n_rows + row) * D + lane * CPL;
        if constexpr (CPL == 2) {
          const f32x2 x = *reinterpret_cast<const f32x2*>(src);
          xo[k][0] = x.x;
          xo[k][1] = x.y;
        } else {
          xo[k][0] = src[0];
        }
      }
    }
    float mx = -INFINITY;
    for (int k = 0; k < kRegParts; ++k)
      if (k < n_parts && (lv[k] > mx || lv[k] != lv[k])) mx = lv[k];  // a NaN part's row is NaN
    float acc[CPL];
    for (int j = 0; j < CPL; ++j) acc[j] = 0.f;
    float lse_r = -INFINITY;
    if (mx != -INFINITY) {
      float tot = 0.f;
      for (int k = 0; k < kRegParts; ++k)
        if (k < n_parts && lv[k] != -INFINITY) tot += __builtin_amdgcn_exp2f((lv[k] - mx) * kLog2e);
      lse_r = mx + __builtin_amdgcn_logf(tot) * kLn2;
      for (int k = 0; k < kRegParts; ++k) {
        // An empty part's O is ignored (never multiplied: it may hold NaN).
        if (k >= n_parts || lv[k] == -INFINITY) continue;
        const float w = __builtin_amdgcn_exp2f((lv[k] - lse_r) * kLog2e);
        for (int j = 0; j < CPL; ++j) acc[j] += w * xo[k][j];
      }
    }
    if constexpr (OUT_BF16) {
      uint16_t* dst = static_cast<uint16_t*>(o) + row * D + lane * CPL;
      if constexpr (CPL == 2)
        *reinterpret_cast<uint32_t*>(dst) =
            merge_f32_to_bf16(acc[0]) | (merge_f32_to_bf16(acc[1]) << 16);
      else
        dst[0] = static_cast<uint16_t>(merge_f32_to_bf16(acc[0]));
    } else {
      float* dst = static_cast<float*>(o) + row * D + lane * CPL;
      for (int j = 0; j < CPL; ++j) dst[j] = acc[j];
    }
    if (lse && lane == 0) lse[row] = lse_r == lse_r ? lse_r : -INFINITY;  // as an unsplit row
    return;
  }

  float mx = -INFINITY;
  for (int k = lane; k < n_parts; k += 64) mx = fmaxf(mx, lse_parts[k * n_rows + row]);
  for (int off = 32; off > 0; off >>= 1) mx = fmaxf(mx, __shfl_xor(mx, off));

  float acc[CPL];
  for (int j = 0; j < CPL; ++j) acc[j] = 0.f;
  float lse_r = -INFINITY;
  if (mx != -INFINITY) {
    float tot = 0.f;
    for (int k = lane; k < n_parts; k += 64) {
      float l = lse_parts[k * n_rows + row];
      if (l != -INFINITY) tot += __builtin_amdgcn_exp2f((l - mx) * kLog2e);
    }
    for (int off = 32; off > 0; off >>= 1) tot += __shfl_xor(tot, off);
    lse_r = mx + __builtin_amdgcn_logf(tot) * kLn2;
    for (int k = 0; k < n_parts; ++k) {
      const float l = lse_parts[k * n_rows + row];
      if (l == -INFINITY) continue;
      const float w = __builtin_amdgcn_exp2f((l - lse_r) * kLog2e);
      const float* src = o_parts + (k * n_rows + row) * D + lane * CPL;
      if constexpr (CPL == 2) {
        f32x2 x = *reinterpret_cast<const f32x2*>(src);
        acc[0] += w * x.x;
        acc[1] += w * x.y;
      } else {
        acc[0] += w * src[0];
      }
    }
  }
  if constexpr (OUT_BF16) {
    uint16_t* dst = static_cast<uint16_t*>(o) + row * D + lane * CPL;
    if constexpr (CPL == 2)
      *reinterpret_cast<uint32_t*>(dst) = merge_f32_to_bf16(acc[0]) | (merge_f32_to_bf16(acc[1]) << 16);
    else
      dst[0] = static_cast<uint16_t>(merge_f32_to_bf16(acc[0]));
  } else {
    float* dst = static_cast<float*>(o) + row * D + lane * CPL;
    for (int j = 0; j < CPL; ++j) dst[j] = acc[j];
  }
  if (lse && lane == 0) lse[row] = lse_r;
}

// The library's own split plans with more than kRegParts parts (a few long
// sequences cut into up to a chunk per compute unit): one workgroup per row,
// whose waves take kRegParts parts each per round with all their loads in
// flight, and sum through LDS.  Every part's O is readable.  Bounded by
// latency (32 parts of 160 rows are 2.6 MB): one wave walking a row's parts is
// a chain of loads (5-token verify of one 32768-token sequence, 32 parts: the
// whole call 41 us with it, 34 us with this).
constexpr int kManyWaves = 4;

template <int D, bool OUT_BF16>
__global__ void __launch_bounds__(64 * kManyWaves)
merge_many_kernel(int n_parts, int64_t n_rows, const float* __restrict__ o_parts,
                  const float* __restrict__ lse_parts, void* __restrict__ o,
                  float* __restrict__ lse) {
  constexpr float kLog2e = 1.44269504088896340736f;
  constexpr float kLn2 = 0.69314718055994530942f;
  constexpr int CPL = D / 64;  // channels per lane
  __shared__ float s_m[kManyWaves], s_l[kManyWaves];
  __shared__ float s_o[kManyWaves][D];
  const int lane = threadIdx.x & 63;
  const int w = threadIdx.x >> 6;
  const int64_t row = blockIdx.x;

  // This wave's parts: running max, sum of 2^(lse - max), weighted O.
  float m = -INFINITY, l = 0.f, acc[CPL];
  for (int j = 0; j < CPL; ++j) acc[j] = 0.f;
  for (int k0 = w * kRegParts; k0 < n_parts; k0 += kManyWaves * kRegParts) {
    float lv[kRegParts];
    float xo[kRegParts][CPL];
#pragma unroll
    for (int t = 0; t < kRegParts; ++t) {
      const int k = min(k0 + t, n_parts - 1);  // a repeated last part is dropped below
      lv[t] = lse_parts[k * n_rows + row];
      const float* src = o_parts + (k * n_rows + row) * D + lane * CPL;
      if constexpr (CPL == 2) {
        const f32x2 x = *reinterpret_cast<const f32x2*>(src);
        xo[t][0] = x.x;
        xo[t][1] = x.y;
      } else {
        xo[t][0] = src[0];
      }
    }
    float mx = m;
#pragma unroll
    for (int t = 0; t < kRegParts; ++t) {
      if (k0 + t >= n_parts) lv[t] = -INFINITY;
      mx = fmaxf(mx, lv[t]);
    }
    if (mx == -INFINITY) {  // uniform over the wave: empty parts, or NaN ones
#pragma unroll
      for (int t = 0; t < kRegParts; ++t) {
        if (lv[t] == lv[t]) continue;
        l = lv[t];
        for (int j = 0; j < CPL; ++j) acc[j] = lv[t];
      }
      continue;
    }
    const float f = __builtin_amdgcn_exp2f((m - mx) * kLog2e);
    l *= f;
    for (int j = 0; j < CPL; ++j) acc[j] *= f;
#pragma unroll
    for (int t = 0; t < kRegParts; ++t) {
      // An empty part's O is ignored (never multiplied: it may hold NaN).
      if (lv[t] == -INFINITY) continue;
      const float wt = __builtin_amdgcn_exp2f((lv[t] - mx) * kLog2e);
      l += wt;
      for (int j = 0; j < CPL; ++j) acc[j] += wt * xo[t][j];
    }
    m = mx;
  }
  if (lane == 0) {
    s_m[w] = m;
    s_l[w] = l;
  }
  for (int j = 0; j < CPL; ++j) s_o[w][lane * CPL + j] = acc[j];
  __syncthreads();
  float M = -INFINITY;
  for (int x = 0; x < kManyWaves; ++x) M = fmaxf(M, s_m[x]);
  float L = 0.f, fx[kManyWaves];
  for (int x = 0; x < kManyWaves; ++x) {
    fx[x] = s_m[x] == -INFINITY ? 0.f : __builtin_amdgcn_exp2f((s_m[x] - M) * kLog2e);
    L += s_l[x] * fx[x];
  }
  const float inv = L > 0.f ? 1.f / L : 0.f;
  const int c = threadIdx.x;
  if (c < D) {
    float v = 0.f;
    for (int x = 0; x < kManyWaves; ++x) v += s_o[x][c] * fx[x];
    v *= inv;
    if constexpr (OUT_BF16)
      static_cast<uint16_t*>(o)[row * D + c] = static_cast<uint16_t>(merge_f32_to_bf16(v));
    else
      static_cast<float*>(o)[row * D + c] = v;
  }
  if (lse && c == 0) lse[row] = L > 0.f ? M + __builtin_amdgcn_logf(L) * kLn2 : -INFINITY;
}

template <int D, bool OUT_BF16>
static void launch_d(bool reg, dim3 grid, dim3 block, hipStream_t s, int n_parts, int64_t n_rows,
                     const float* o_parts, const float* lse_parts, void* o, float* lse) {
  if (reg)
    hipLaunchKernelGGL((merge_lse_kernel<D, OUT_BF16, true>), grid, block, 0, s, n_parts, n_rows,
                       o_parts, lse_parts, o, lse);
  else
    hipLaunchKernelGGL((merge_lse_kernel<D, OUT_BF16, false>), grid, block, 0, s, n_parts,
                       n_rows, o_parts, lse_parts, o, lse);
}

hipError_t launch_merge_lse(int n_parts, int64_t n_rows, int head_dim, bool out_bf16,
                            const float* o_parts, const float* lse_parts, void* o, float* lse,
                            hipStream_t s, bool parts_readable) {
  if (n_rows <= 0) return hipSuccess;
  dim3 grid(static_cast<uint32_t>((n_rows + 3) / 4)), block(256);
  const bool reg = parts_readable && n_parts <= kRegParts;
  if (parts_readable && !reg) {
    const dim3 g(static_cast<uint32_t>(n_rows)), blk(64 * kManyWaves);
#define MD_MERGE_MANY(D, BF)                                                                 \
  hipLaunchKernelGGL((merge_many_kernel<D, BF>), g, blk, 0, s, n_parts, n_rows, o_parts,     \
                     lse_parts, o, lse)
    if (head_dim == 128) {
      if (out_bf16) MD_MERGE_MANY(128, true); else MD_MERGE_MANY(128, false);
    } else {
      if (out_bf16) MD_MERGE_MANY(64, true); else MD_MERGE_MANY(64, false);
    }
#undef MD_MERGE_MANY
    return hipGetLastError();
  }
  if (head_dim == 128) {
    if (out_bf16)
      launch_d<128, true>(reg, grid, block, s, n_parts, n_rows, o_parts, lse_parts, o, lse);
    else
      launch_d<128, false>(reg, grid, block, s, n_parts, n_rows, o_parts, lse_parts, o, lse);
  } else {
    if (out_bf16)
      launch_d<64, true>(reg, grid, block, s, n_parts, n_rows, o_parts, lse_parts, o, lse);
    else
      launch_d<64, false>(reg, grid, block, s, n_parts, n_rows, o_parts, lse_parts, o, lse);
  }
  return hipGetLastError();
}

}  // namespace md
