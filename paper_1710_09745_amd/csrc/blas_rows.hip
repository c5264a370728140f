// Block BLAS in the row layout (rows.h).
#include <type_traits>
#include <utility>

#include "internal.h"
#include "rows.h"

namespace bcg {

// Canonical [N][Vh][3] <-> rows [Vh][3][N], FP64: a workgroup takes 16 sites of all
// columns through LDS, so that both sides move whole runs (48 complex numbers of a
// column on one, 48 N contiguous ones on the other).  Column n sits at n * 49, so that
// the 16-byte reads across columns fall into different banks.
template <bool TO_ROWS>
__global__ void __launch_bounds__(256)
k_canon_rows(const double2* __restrict__ src, double2* __restrict__ dst, int N, int Vh) {
    extern __shared__ double2 tile[];  // [N][49]
    const int s0 = blockIdx.x * 16;
    const int m = 3 * (Vh - s0 < 16 ? Vh - s0 : 16);  // (site, colour) rows of this block
    const long r0 = 3L * s0;
    const float rn = 1.0f / (float)N;
    if constexpr (TO_ROWS) {
        for (int e = threadIdx.x; e < 48 * N; e += 256) {
            const int n = e / 48, r = e - 48 * n;
            if (r < m) tile[n * 49 + r] = src[(long)n * 3 * Vh + r0 + r];
        }
        __syncthreads();
        for (int e = threadIdx.x; e < m * N; e += 256) {
            const int r = (int)(((float)e + 0.5f) * rn), n = e - r * N;
            dst[r0 * N + e] = tile[n * 49 + r];
        }
    } else {
        for (int e = threadIdx.x; e < m * N; e += 256) {
            const int r = (int)(((float)e + 0.5f) * rn), n = e - r * N;
            tile[n * 49 + r] = src[r0 * N + e];
        }
        __syncthreads();
        for (int e = threadIdx.x; e < 48 * N; e += 256) {
            const int n = e / 48, r = e - 48 * n;
            if (r < m) dst[(long)n * 3 * Vh + r0 + r] = tile[n * 49 + r];
        }
    }
}

hipError_t launch_canon_to_rows(const double2* src, double2* dst, int N, int Vh, hipStream_t s) {
    hipLaunchKernelGGL(k_canon_rows<true>, dim3((Vh + 15) / 16), dim3(256), (size_t)N * 49 * 16, s, src, dst, N, Vh);
    return hipGetLastError();
}
hipError_t launch_rows_to_canon(const double2* src, double2* dst, int N, int Vh, hipStream_t s) {
    hipLaunchKernelGGL(k_canon_rows<false>, dim3((Vh + 15) / 16), dim3(256), (size_t)N * 49 * 16, s, src, dst, N, Vh);
    return hipGetLastError();
}

}  // namespace bcg
