// Partial sums of a GEMM whose contraction is cut evenly over the CUs (pf_part_kernel in ee_prefill.hip), as the kernels
// that add them up see them.
#pragma once
#include <hip/hip_runtime.h>

#include "ee_internal.h"

namespace ee {

typedef float part_f32x4 __attribute__((ext_vector_type(4)));

// Sums of N neighbouring weight tiles T0.. (of one panel of 16) and row tile mt, in the order of K: lane (li, rg) receives
// features rg * 4 .. + 3 of row li.  All the loads of up to eight parts go out before the first is used.
template <int N>
__device__ __forceinline__ void sum_parts(const PartGeom& g, const part_f32x4* __restrict__ part, int mt, int T0, int lane, part_f32x4 (&v)[N]) {
    const int p = (T0 / 16) * g.n_wgM + mt / g.mtl;
    const int w0 = p * g.KT / g.unit, n = ((p + 1) * g.KT - 1) / g.unit - w0 + 1;
    const size_t slot = (size_t)16 * g.mtl * 64;
    const part_f32x4* q = part + (size_t)(w0 + p) * slot + ((T0 % 16) * g.mtl + mt % g.mtl) * 64 + lane;
#pragma unroll
    for (int i = 0; i < N; ++i) v[i] = part_f32x4{0.f, 0.f, 0.f, 0.f};
    for (int s = 0; s < n; s += 8) {
        part_f32x4 u[8][N];
#pragma unroll
        for (int h = 0; h < 8; h += 4)
            if (s + h < n) {  // (uniform)
#pragma unroll
                for (int k = h; k < h + 4; ++k)
#pragma unroll
                    for (int i = 0; i < N; ++i) u[k][i] = q[(size_t)(s + k < n ? s + k : s) * slot + i * g.mtl * 64];
            }
#pragma unroll
        for (int k = 0; k < 8; ++k)
#pragma unroll
            for (int i = 0; i < N; ++i)
                if (s + k < n) v[i] += u[k][i];
    }
}

}  // namespace ee
