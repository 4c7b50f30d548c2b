// The kernels of four wavefronts (256 queries per workgroup) for the three block sizes, and the launch of all kernels that
// walk merged rows with 64 queries per wavefront.  gfx950 (CDNA4) only.
#include "attn_pair_body.h"

#include <algorithm>

namespace dr {
namespace {

constexpr int kWaves = 4, kThreads = kWaves * 64;

// Block size 128: two query blocks per workgroup, an entry of the merged list is two chunks.  Block size 64: four
// query blocks, one per wavefront, an entry is one chunk; the same 256 queries and the same code otherwise.
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(1, 1))) void k_attn_mfma_pair(AttnArgs) { attn_pair_body<128, 4>(); }
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(1, 1))) void k_attn_mfma_quad(AttnArgs) { attn_pair_body<64, 4>(); }
// Block size 32: eight query blocks, two per wavefront (one per query half); a chunk is two entries of the merged list,
// its two key halves come from two 32-row windows, and a 32 x 32 tile whose query block does not list the key block of
// its key half contributes probabilities of 0 (they are masked where they are packed to bf16).
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(1, 1))) void k_attn_mfma_oct(AttnArgs) { attn_pair_body<32, 4>(); }

}  // namespace

bool attn_mfma_pair_supported(const AttnArgs& a) {
    // every chunk is a full 64-row window: the sequence must hold one; the 32-bit per-lane offsets must cover it
    return a.bf16 && a.td.d == kD && (a.Bs == 128 || a.Bs == 64 || a.Bs == 32) && a.td.N >= kChunkKeys &&
           a.Sb < (a.Bs == 32 ? (1 << 24) : (1 << 28)) &&
           a.td.stride_n * 2 * kChunkKeys < (1ll << 31) && a.gcol && a.gcount && a.flags && a.queue;
}

hipError_t launch_attn_mfma_pair(const AttnArgs& a, hipStream_t s) {
    if (!attn_mfma_pair_supported(a)) return hipErrorNotSupported;
    // Masks of one head each: the selections of neighbouring query blocks differ, so at block size 64 the merged list of four
    // rows is long (1.38 times the kept blocks at 17 frames of 31 x 45 tokens, 1.14 for two) and every wavefront steps through
    // all of it.  There two workgroups of two wavefronts share a CU instead: 1.86 -> 1.77 ms, 1 to 19 % less up to one
    // round of the larger workgroup, 0 to 2 % less beyond two.  Between one and two rounds the smaller one measured 0 to 10 %
    // longer (288 to 512 items: its last, short round starts as late), and the larger one stays.  Masks shared by the heads follow the field they were pooled from (1.06 for four rows at 75 600
    // tokens), and a tile fetched once for four wavefronts costs half the traffic.  At block size 32 two wavefronts save
    // nothing (1.34 against 1.39).
    const int64_t items256 = ((int64_t)a.td.N + 255) / 256 * a.td.H * a.td.B;
    const bool duo = a.Bs == 64 && a.mask_heads > 1 && (items256 <= a.cus || items256 > 2 * (int64_t)a.cus);
    const int L = (duo ? 128 : 256) / a.Bs;
    // workgroups that fit the device at once, or one per item if there are fewer; a multiple of the queues
    const int64_t items = (int64_t)((a.Sb + L - 1) / L) * a.td.H * a.td.B, fit = (int64_t)a.cus * (duo ? 2 : 1);
    const int grid = (int)((std::min(items, fit) + kXcds - 1) / kXcds) * kXcds;
    hipError_t e = launch_group_union(L, a, s, grid / kXcds);
    if (e != hipSuccess) return e;
    if (duo) return launch_attn_mfma_duo(a, grid, s);
    auto kern = a.Bs == 128 ? k_attn_mfma_pair : a.Bs == 64 ? k_attn_mfma_quad : k_attn_mfma_oct;
    e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, kLdsBytes);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(kern, dim3(grid), dim3(kThreads), kLdsBytes, s, a);
    return hipGetLastError();
}

}  // namespace dr
