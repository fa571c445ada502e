// AKVQ-style token retention (HeadGuard §4, Quantization setup): in every KV
// head the keys and values of a nominal 2 % of the image tokens, those whose
// keys have the largest norms, stay in BF16, with or without head protection.
//
// The quantize kernel, and the one-pass simulated quantization out of place,
// write the squared key norm of every image token in the pass that reads the
// keys; key_norm_kernel computes them on their own for an in-place one-pass
// call, whose outputs would otherwise overwrite the rows to keep.  Then, per
// (l, b, h):
//  - retain_select_kernel (norms staged in LDS) finds the k-th largest norm by
//    a most-significant-digit-first radix select over the fp32 bit patterns
//    (non-negative, so they order as unsigned integers), starting below the
//    bits every norm of the head shares and stopping once the chosen digit's
//    candidates are all taken; lists the retained tokens in ascending order
//    (all larger norms, then the lowest-index ties); and, in the same
//    workgroup, gathers their K and V rows for each tensor the head does not
//    keep in BF16 (an out-of-place one-pass call, which computes the norms in
//    its own pass, copies them from the input straight to the output); in a
//    quantize call the same code runs in the launch of the values where its
//    LDS fits (quantize.hip);
//  - retain_rows_kernel writes the gathered rows back over the
//    reconstruction (dequantize calls of one launch with short lists store them
//    in the dequantize kernel).

#include "hg_device.h"
#include "hg_kernels.h"
#include "hg_retain.h"

namespace hg {

// ------------------------------------------------------------ key norms

// One workgroup per kBlockTokens tokens of one key slice; a token row is held
// by D/8 lanes, 8 channels each.
template <int D>
__global__ __launch_bounds__(kThreads) void key_norm_kernel(const Params p) {
  constexpr int R = D / 8;                // lanes per token row
  constexpr int RPL = 64 / R;             // token rows per load
  constexpr int NL = kWaveTokens / RPL;   // loads per lane
  const uint32_t s = blockIdx.x / (uint32_t)p.tiles;
  const int tile = (int)(blockIdx.x % (uint32_t)p.tiles);
  const int lane = threadIdx.x & 63;
  const int t_first = tile * kBlockTokens + (threadIdx.x >> 6) * kWaveTokens;
  if (t_first >= p.n) return;
  const int c = lane % R, r = lane / R;
  const uint16_t* rows = p.cache[0] + ((size_t)s * p.T + p.s0) * D;
  float* norm = p.norm + (size_t)s * p.n;
  u32x4 v[NL];
#pragma unroll
  for (int k = 0; k < NL; ++k) {
    const int t = min(t_first + r + RPL * k, p.n - 1);  // rows past the end: not stored
    v[k] = *(const u32x4*)(rows + (size_t)t * D + 8 * c);
  }
#pragma unroll
  for (int k = 0; k < NL; ++k) {
    const float sq = row_sqnorm<D>(v[k]);
    const int t = t_first + r + RPL * k;
    if (c == 0 && t < p.n) norm[t] = sq;
  }
}

// ------------------------------------------------------------ selection

// One workgroup per (l, b, h); requires 1 <= k <= n.  Writes ret_idx, then
// copies the retained rows (kGather or kCacheToOut).
template <bool RESIDENT, int D, RowCopy MODE>
__global__ __launch_bounds__(kThreads) void retain_select_kernel(const Params p) {
  extern __shared__ uint32_t lds_keys[];  // n keys when RESIDENT
  retain_select<RESIDENT, D, MODE>(p, blockIdx.x, lds_keys);
}

// ------------------------------------------------------------ retained rows

// Grid l*B*H: the retained rows of one (l, b, h) per workgroup, listed in
// p.ret_idx (the dequantize direction, and an in-place one-pass call).
template <int D, RowCopy MODE>
__global__ __launch_bounds__(kThreads) void retain_rows_kernel(const Params p) {
  copy_retained_rows<D, MODE>(p, blockIdx.x, p.ret_idx + (size_t)blockIdx.x * (uint32_t)p.k);
}

// ------------------------------------------------------------ launchers

hipError_t launch_key_norms(const Params& p, int D, hipStream_t stream) {
  const uint32_t blocks = (uint32_t)p.L * p.B * p.H * (uint32_t)p.tiles;
  if (D == 64)
    hipLaunchKernelGGL((key_norm_kernel<64>), dim3(blocks), dim3(kThreads), 0, stream, p);
  else if (D == 128)
    hipLaunchKernelGGL((key_norm_kernel<128>), dim3(blocks), dim3(kThreads), 0, stream, p);
  else if (D == 256)
    hipLaunchKernelGGL((key_norm_kernel<256>), dim3(blocks), dim3(kThreads), 0, stream, p);
  else
    return hipErrorInvalidValue;
  return hipGetLastError();
}

template <int D>
static hipError_t launch_rows_d(const Params& p, RowCopy mode, hipStream_t stream) {
  const dim3 grid((uint32_t)p.L * p.B * p.H);
  switch (mode) {
    case RowCopy::kGather:
      hipLaunchKernelGGL((retain_rows_kernel<D, RowCopy::kGather>), grid, dim3(kThreads), 0, stream, p);
      break;
    case RowCopy::kScatter:
      hipLaunchKernelGGL((retain_rows_kernel<D, RowCopy::kScatter>), grid, dim3(kThreads), 0, stream, p);
      break;
    default:
      hipLaunchKernelGGL((retain_rows_kernel<D, RowCopy::kCacheToOut>), grid, dim3(kThreads), 0, stream, p);
      break;
  }
  return hipGetLastError();
}

hipError_t launch_retain_rows(const Params& p, int D, RowCopy mode, hipStream_t stream) {
  if (D == 64) return launch_rows_d<64>(p, mode, stream);
  if (D == 128) return launch_rows_d<128>(p, mode, stream);
  if (D == 256) return launch_rows_d<256>(p, mode, stream);
  return hipErrorInvalidValue;
}

template <bool RESIDENT, int D>
static void launch_select_r(const Params& p, RowCopy mode, dim3 grid, size_t lds, hipStream_t stream) {
  if (mode == RowCopy::kGather)
    hipLaunchKernelGGL((retain_select_kernel<RESIDENT, D, RowCopy::kGather>), grid, dim3(kThreads), lds, stream, p);
  else
    hipLaunchKernelGGL((retain_select_kernel<RESIDENT, D, RowCopy::kCacheToOut>), grid, dim3(kThreads), lds,
                       stream, p);
}

template <int D>
static void launch_select_d(const Params& p, RowCopy mode, hipStream_t stream) {
  const dim3 grid((uint32_t)p.L * p.B * p.H);
  if (p.n <= kResidentKeys)
    launch_select_r<true, D>(p, mode, grid, (size_t)p.n * sizeof(uint32_t), stream);
  else
    launch_select_r<false, D>(p, mode, grid, 0, stream);
}

hipError_t launch_retain_select(const Params& p, int D, RowCopy mode, hipStream_t stream) {
  if (mode == RowCopy::kScatter) return hipErrorInvalidValue;
  if (D == 64)
    launch_select_d<64>(p, mode, stream);
  else if (D == 128)
    launch_select_d<128>(p, mode, stream);
  else if (D == 256)
    launch_select_d<256>(p, mode, stream);
  else
    return hipErrorInvalidValue;
  return hipGetLastError();
}

}  // namespace hg
