// Instantiations of the verification kernels.
#include <algorithm>

#include "launch.hpp"
#include "verify_fused.hpp"

namespace ts {

int verify_argmax_chunks(int V, int nrows, bool bf16, int most) {
  // a sweep of a workgroup: one 16-byte group per thread.  Pieces of four
  // sweeps (all of a thread's loads in flight at once) unless that leaves
  // the launch under two workgroups per CU; then down to one sweep.
  const int sweep = kVerifyThreads * (bf16 ? 8 : 4);
  const int sweeps = (V + sweep - 1) / sweep;
  int c = (sweeps + 3) / 4;
  while (c < sweeps && (long long)c * nrows < 512) ++c;
  c = std::min(c, std::max(1, (1 << 22) / std::max(nrows, 1)));  // a launch's grid stays within its limits
  return std::max(1, std::min(c, most));
}

void launch_verify_argmax(const void* target, bool bf16, int V, const int* rows, int nrows, int nchunks,
                          ArgmaxPart* part, hipStream_t s) {
  const dim3 grid((unsigned)nrows * nchunks), block(kVerifyThreads);
  if (bf16)
    hipLaunchKernelGGL((verify_argmax_kernel<uint16_t>), grid, block, 0, s, static_cast<const uint16_t*>(target), V,
                       rows, nchunks, part);
  else
    hipLaunchKernelGGL((verify_argmax_kernel<float>), grid, block, 0, s, static_cast<const float*>(target), V, rows,
                       nchunks, part);
}

template <typename TT>
static void verify_level_t(const VerifyPass& vp, int mmax, hipStream_t s) {
  const dim3 grid(vp.nitems * vp.nchunks), block(kVerifyThreads);
  const int J = mmax > 1 ? mmax : 1;
  hipLaunchKernelGGL((verify_pass_a_kernel<TT>), grid, block, 0, s, vp);
  for (int j = 1; j <= J; ++j) hipLaunchKernelGGL((verify_stage_kernel<TT>), grid, block, 0, s, vp, j);
  hipLaunchKernelGGL((verify_resolve_kernel<TT>), dim3(vp.nitems), dim3(64), 0, s, vp, J);
}

void launch_verify_level(const VerifyPass& vp, bool bf16, int mmax, hipStream_t s) {
  if (bf16)
    verify_level_t<uint16_t>(vp, mmax, s);
  else
    verify_level_t<float>(vp, mmax, s);
}

int verify_fused_quads(bool bf16) { return bf16 ? kFusedQuadsBf16 : kFusedQuadsF32; }

int verify_fused_blocks_per_cu(bool bf16) {
  static int cached[2] = {-1, -1};
  int& n = cached[bf16 ? 1 : 0];
  if (n < 0) {
    int b = 0;
    const hipError_t e =
        bf16 ? hipOccupancyMaxActiveBlocksPerMultiprocessor(
                   &b, verify_fused_kernel<uint16_t, kFusedQuadsBf16>, kVerifyThreads, 0)
             : hipOccupancyMaxActiveBlocksPerMultiprocessor(
                   &b, verify_fused_kernel<float, kFusedQuadsF32>, kVerifyThreads, 0);
    n = (e == hipSuccess && b > 0) ? b : 0;
  }
  return n;
}

void launch_verify_fused(const VerifyPass& vp, const VFused& f, bool bf16, hipStream_t s) {
  const dim3 grid(vp.nitems * f.cpi), block(kVerifyThreads);
  if (bf16)
    hipLaunchKernelGGL((verify_fused_kernel<uint16_t, kFusedQuadsBf16>), grid, block, 0, s, VFusedArgs{vp, f});
  else
    hipLaunchKernelGGL((verify_fused_kernel<float, kFusedQuadsF32>), grid, block, 0, s, VFusedArgs{vp, f});
}

// Copies n16 16-byte pieces (a round's rows, from the host's pinned buffer) and
// n16b more (a small round's items), and clears nclear of them (the level slots).
__global__ void verify_stage_in_kernel(const u32x4* src, u32x4* dst, int n16, const u32x4* src2, u32x4* dst2, int n16b,
                                       u32x4* clear, int nclear) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  u32x4 a = {}, b = {};
  if (i < n16) a = src[i];
  if (i < n16b) b = src2[i];
  if (i < n16) dst[i] = a;
  if (i < n16b) dst2[i] = b;
  if (i < nclear) clear[i] = u32x4{0u, 0u, 0u, 0u};
}

void launch_verify_stage_in(const void* src, void* dst, size_t bytes, void* clear, size_t clear_bytes, hipStream_t s,
                            const void* src2, void* dst2, size_t bytes2) {
  const int n16 = (int)((bytes + 15) / 16), n16b = (int)((bytes2 + 15) / 16), nc = (int)((clear_bytes + 15) / 16);
  const int n = std::max(std::max(n16, n16b), nc);
  if (n > 0)
    hipLaunchKernelGGL(verify_stage_in_kernel, dim3((n + 255) / 256), dim3(256), 0, s, static_cast<const u32x4*>(src),
                       static_cast<u32x4*>(dst), n16, static_cast<const u32x4*>(src2), static_cast<u32x4*>(dst2), n16b,
                       static_cast<u32x4*>(clear), nc);
}

}  // namespace ts
