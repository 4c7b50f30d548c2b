// The kernel of two wavefronts (128 queries = two query blocks of 64 per workgroup), for masks whose neighbouring rows differ;
// two workgroups share a CU.  A wavefront fetches half of every tile (16 loads a chunk instead of 8, in slots 56 .. 71)
// and steps only through the merged list of two rows.  gfx950 (CDNA4) only.
#include "attn_pair_body.h"

namespace dr {
namespace {

__global__ __launch_bounds__(128) __attribute__((amdgpu_waves_per_eu(1, 1))) void k_attn_mfma_duo(AttnArgs) { attn_pair_body<64, 2>(); }

}  // namespace

hipError_t launch_attn_mfma_duo(const AttnArgs& a, int grid, hipStream_t s) {
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(k_attn_mfma_duo), hipFuncAttributeMaxDynamicSharedMemorySize, kLdsBytes);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_attn_mfma_duo, dim3(grid), dim3(128), kLdsBytes, s, a);
    return hipGetLastError();
}

}  // namespace dr
