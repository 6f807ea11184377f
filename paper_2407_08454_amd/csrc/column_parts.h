// The column sums that the single score pass (attn_single.hip) leaves behind, one row of them per workgroup, and their sum.
#pragma once

#include "kvm_common.h"

namespace kvm {

constexpr int COLUMN_BLOCK = 256;                            // threads of a workgroup that adds 64 columns up

struct ColumnParts {
    const float *part;                                       // (slices, P, n_pad)
    float *mass;                                             // (slices, n)
    int G, n, n_pad, P, rows, blocks_per_slice;
};

// mass[j] = sum over the workgroups p, in order, of their column sums; workgroup p holds the keys up to the last row of its first unit
__device__ __forceinline__ void add_column_parts(const ColumnParts &a, int block, float (*sums)[64])
{
    const int slice = block / a.blocks_per_slice, j0 = (block % a.blocks_per_slice) * 64;
    const int lane = threadIdx.x & 63, q = threadIdx.x >> 6, j = j0 + lane;
    // key j is in the first unit of workgroup p, row group (n - 1) / rows - p / G, or above it
    const int count = min(a.P, ((a.n - 1) / a.rows - j / a.rows + 1) * a.G);
    const float *src = a.part + (size_t)slice * a.P * a.n_pad + j;
    float s = 0.f;
    if (j < a.n)
        for (int p = q; p < count; p += 4) s += src[(size_t)p * a.n_pad];
    sums[q][lane] = s;
    __syncthreads();
    if (q == 0 && j < a.n) a.mass[(size_t)slice * a.n + j] = (sums[0][lane] + sums[1][lane]) + (sums[2][lane] + sums[3][lane]);
}

// The cosine scan (identify.hip), and in the same launch, by workgroups after its own, those sums.
kvm_status launch_cosine_scan_and_sums(const kvm_shape &sh, const void *K, float *sim, const ColumnParts &sums, hipStream_t st);

}  // namespace kvm
