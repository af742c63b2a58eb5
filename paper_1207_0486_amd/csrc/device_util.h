// Device helpers shared by the kernel files: wavefront sums, workgroup
// numbering, Dirichlet bits.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace hns {
namespace {

// One DPP move of a double (both 32-bit halves): lanes whose source lies
// outside the pattern (bound_ctrl) or whose row is masked off read 0.
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ double dpp_move(double v)
{
    const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), CTRL, ROW_MASK, 0xf, true);
    const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), CTRL, ROW_MASK, 0xf, true);
    return __hiloint2double(hi, lo);
}

// Wavefront sum through the DPP network instead of LDS permutes (all 64
// lanes active): row_shr 1, 2, 4, 8 leave each 16-lane row's sum in its
// lane 15, row_bcast 15 adds row 0's into row 1 and row 2's into row 3, and
// row_bcast 31 adds lane 31's into rows 2 and 3, so lane 63 holds the total,
// which every lane then reads.  A fixed order, the same in every wavefront.
__device__ __forceinline__ double wave_sum_dpp(double v)
{
    v += dpp_move<0x111, 0xf>(v);   // row_shr:1
    v += dpp_move<0x112, 0xf>(v);   // row_shr:2
    v += dpp_move<0x114, 0xf>(v);   // row_shr:4
    v += dpp_move<0x118, 0xf>(v);   // row_shr:8
    v += dpp_move<0x142, 0xa>(v);   // row_bcast:15
    v += dpp_move<0x143, 0xc>(v);   // row_bcast:31
    const int lo = __builtin_amdgcn_readlane(__double2loint(v), 63);
    const int hi = __builtin_amdgcn_readlane(__double2hiint(v), 63);
    return __hiloint2double(hi, lo);
}

// Every block reduction of the path calls this with all 64 lanes active.
__device__ __forceinline__ double wave_sum(double v) { return wave_sum_dpp(v); }

// Workgroups are dealt to the 8 XCDs round-robin; renumber them so that each
// XCD works on one contiguous eighth of the rows (neighbour gathers of the
// SpMV then hit that XCD's own L2).
__device__ __forceinline__ int xcd_block(int b, int G)
{
    return (G >= 8 && (G & 7) == 0) ? (b & 7) * (G >> 3) + (b >> 3) : b;
}

__device__ __forceinline__ bool is_dirichlet(const uint8_t *bc, int bit, int64_t i)
{
    return bc != nullptr && ((bc[i] >> bit) & 1u);
}

// Fused multiply-add in the vector type (the direction and x updates of the
// scaled recurrence are written with it wherever they are evaluated, so that
// every evaluation of p' = r + beta p gives the same bits)
__device__ __forceinline__ double fma_t(double a, double b, double c) { return __builtin_fma(a, b, c); }
__device__ __forceinline__ float fma_t(float a, float b, float c) { return __builtin_fmaf(a, b, c); }

// Keeps the compiler from carrying what derives from v (the LDS addresses
// of its neighbours, say) across iterations in registers, which the matrix needs.
__device__ __forceinline__ int fresh(int v)
{
    asm volatile("" : "+v"(v));
    return v;
}

}  // namespace
}  // namespace hns
