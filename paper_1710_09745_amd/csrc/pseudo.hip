// Pseudo-block CG (the prior work of Sec. 2): N independent CG recurrences that
// share every stencil application.  The hop kernels apply A to all N search
// directions at once (each link read once per site for the whole block); the
// scalar recurrences of the columns stay separate: per column
//   alpha_i = |r_i|^2 / p_i^H A p_i,  x_i += alpha_i p_i,  r_i -= alpha_i A p_i,
//   beta_i = |r_i,new|^2 / |r_i|^2,   p_i = r_i + beta_i p_i.
// A column whose iterated relative residual meets tol stops moving (alpha = 0)
// while the others go on.  FP64 storage, block vectors [N][3][Vh] pairs.
//
// Reductions are deterministic: one partial per (column, workgroup), summed in
// a fixed order by a single-workgroup kernel (16 to 128 lanes per column).
//
// x is updated together with p, whose old value both need: the iteration reads P, X, R, AP
// once each for 8 block transfers instead of 9 (update1 and update2 at 16^3 x 48, N = 24:
// 117 + 56 -> 61 + 89 us).
//
// In the row layout ([Vh][3][N]) a thread keeps one column for all of its rows (the
// threads of a workgroup cover whole rows), so that the loads of a workgroup are one
// contiguous run and the per-column scalars stay in registers; p^H A p comes from the hop.
#include "device_common.h"
#include "internal.h"
#include "rows.h"

namespace bcg {

static int pb_blocks(int Vh) {
    const int g = (Vh + 255) / 256;
    return g < NORM_BLOCKS ? g : NORM_BLOCKS;
}

// workgroup sum of v (256 threads); the total on thread 0
__device__ double pb_block_sum(double v, double* red) {
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
    __syncthreads();
    return red[0] + red[1] + red[2] + red[3];
}

// partials[j][b] = Re sum over the sites of workgroup b of conj(P_j) AP_j; grid (blocks, N)
__global__ void __launch_bounds__(256)
k_pb_dot(const double2* __restrict__ P, const double2* __restrict__ AP, int Vh, double* __restrict__ partials,
         const PbState* __restrict__ st) {
    if (st->halt) return;
    const int j = blockIdx.y;
    __shared__ double red[4];
    double s = 0.0;
    if (st->active[j]) {
        for (long i = (long)blockIdx.x * 256 + threadIdx.x; i < Vh; i += (long)gridDim.x * 256)
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                const long o = ((long)j * 3 + c) * Vh + i;
                const double2 p = P[o], a = AP[o];
                s += p.x * a.x + p.y * a.y;
            }
    }
    s = pb_block_sum(s, red);
    if (threadIdx.x == 0) partials[(long)j * gridDim.x + blockIdx.x] = s;
}

// Lanes per column of the 1024-thread sums: 16 for 64 columns, up to 128 for 8 or fewer.
__device__ __forceinline__ int pb_lanes(int N) { return N <= 8 ? 128 : (N <= 16 ? 64 : (N <= 32 ? 32 : 16)); }

// Sum over b of partials[j][b] for column j = threadIdx.x / pb_lanes(N), in a fixed order:
// lane g of the column takes b = g, g + lanes, ... (eight loads in flight), then the
// lanes are added in order.  Valid on lane 0 of each column; red: 1024 doubles.
__device__ double pb_column_sum(const double* __restrict__ partials, int nb, int N, double* red) {
    const int ln = pb_lanes(N), j = threadIdx.x / ln, g = threadIdx.x & (ln - 1);
    double v = 0.0;
    if (j < N)
        for (int b0 = g; b0 < nb; b0 += 8 * ln) {
            double t[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) t[u] = b0 + u * ln < nb ? partials[(long)j * nb + b0 + u * ln] : 0.0;
#pragma unroll
            for (int u = 0; u < 8; ++u) v += t[u];
        }
    for (int off = 8; off > 0; off >>= 1) v += __shfl_xor(v, off, 16);
    red[threadIdx.x] = v;
    __syncthreads();
    double s = 0.0;
    if (g == 0)
        for (int q = 0; q < ln; q += 16) s += red[threadIdx.x + q];
    return s;
}

// alpha_j = rr_j / p_j^H A p_j for the active columns (0 for the others)
__global__ void __launch_bounds__(1024) k_pb_alpha(const double* __restrict__ partials, int nb, int N, PbState* st) {
    if (st->halt) {
        if (threadIdx.x == 0) st->step = 0;
        return;
    }
    __shared__ double red[1024];
    const int ln = pb_lanes(N), j = threadIdx.x / ln;
    const double pap = pb_column_sum(partials, nb, N, red);
    if (threadIdx.x == 0) st->step = 1;
    __syncthreads();
    if (j < N && (threadIdx.x & (ln - 1)) == 0) {
        double a = 0.0;
        if (st->active[j]) {
            if (!(pap > 0.0)) {
                st->halt = 1;
                st->reason = HALT_BREAKDOWN_G;
                st->step = 0;
            } else {
                a = st->rr[j] / pap;
            }
        }
        st->alpha[j] = a;
    }
}

// r_j -= alpha_j Ap_j; partials[j][b] = |r_j|^2 over workgroup b's sites
__global__ void __launch_bounds__(256)
k_pb_update1(double2* __restrict__ R, const double2* __restrict__ AP, int Vh, double* __restrict__ partials, const PbState* __restrict__ st) {
    if (st->halt) return;
    const int j = blockIdx.y;
    __shared__ double red[4];
    double s = 0.0;
    if (st->active[j]) {
        const double a = st->alpha[j];
        for (long i = (long)blockIdx.x * 256 + threadIdx.x; i < Vh; i += (long)gridDim.x * 256)
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                const long o = ((long)j * 3 + c) * Vh + i;
                const double2 ap = AP[o];
                double2 r = R[o];
                r.x = fma(-a, ap.x, r.x);
                r.y = fma(-a, ap.y, r.y);
                R[o] = r;
                s += r.x * r.x + r.y * r.y;
            }
    }
    s = pb_block_sum(s, red);
    if (threadIdx.x == 0) partials[(long)j * gridDim.x + blockIdx.x] = s;
}

// beta_j, the iterated residuals and the convergence of each column
__global__ void __launch_bounds__(1024) k_pb_beta(const double* __restrict__ partials, int nb, int N, PbState* st) {
    if (st->halt) return;
    __shared__ int still;
    __shared__ double red[1024];
    if (threadIdx.x == 0) still = 0;
    __syncthreads();
    const int ln = pb_lanes(N), j = threadIdx.x / ln;
    const double rr = pb_column_sum(partials, nb, N, red);
    if (j < N && (threadIdx.x & (ln - 1)) == 0 && st->active[j]) {
        st->beta[j] = rr / st->rr[j];
        st->rr[j] = rr;
        st->relres[j] = sqrt(rr) / st->bnorm[j];
        st->col_iters[j] += 1;
        if (st->relres[j] <= st->tol) st->active[j] = 0;
        else atomicAdd(&still, 1);
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        st->iters += 1;
        if (still == 0) {
            st->halt = 1;
            st->reason = HALT_CONVERGED;
        }
    }
}

// x_j += alpha_j p_j (alpha = 0: no step), then p_j = r_j + beta_j p_j for the columns
// still active; after a halt that came with a step, x alone
__global__ void __launch_bounds__(256)
k_pb_update2(double2* __restrict__ X, double2* __restrict__ P, const double2* __restrict__ R, int Vh,
             const PbState* __restrict__ st) {
    if (!st->step) return;
    const int j = blockIdx.y;
    const double a = st->alpha[j], b = st->beta[j];
    if (a == 0.0) return;
    const bool go = st->active[j];
    for (long i = (long)blockIdx.x * 256 + threadIdx.x; i < Vh; i += (long)gridDim.x * 256)
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            const long o = ((long)j * 3 + c) * Vh + i;
            double2 p = P[o], x = X[o];
            x.x = fma(a, p.x, x.x);
            x.y = fma(a, p.y, x.y);
            X[o] = x;
            if (go) {
                const double2 r = R[o];
                p.x = fma(b, p.x, r.x);
                p.y = fma(b, p.y, r.y);
                P[o] = p;
            }
        }
}

// Loads and stores with a streaming hint: x is touched once an iteration and A p has its
// last use in update1, and both would only push p, r and the links out of the Infinity Cache.
typedef double pair_t __attribute__((ext_vector_type(2)));
__device__ __forceinline__ double2 ld_stream(const double2* p) {
    return __builtin_bit_cast(double2, __builtin_nontemporal_load(reinterpret_cast<const pair_t*>(p)));
}
__device__ __forceinline__ void st_stream(double2* p, double2 v) {
    __builtin_nontemporal_store(__builtin_bit_cast(pair_t, v), reinterpret_cast<pair_t*>(p));
}

// The same three steps in the row layout.  tp = 256 / N rows of N threads; thread
// (row, column) strides over the 3 Vh rows of the block; the workgroup's sums per column
// are added in order of the row (partials [j][b] as above).
__device__ __forceinline__ void pb_rows_sum(double v, double* red, int N, int tp, double* __restrict__ partials) {
    red[threadIdx.x] = v;
    __syncthreads();
    if (threadIdx.x < N) {
        double s = 0.0;
        for (int q = 0; q < tp; ++q) s += red[q * N + threadIdx.x];
        partials[(long)threadIdx.x * gridDim.x + blockIdx.x] = s;
    }
}

// partials of p^H A p per column from the block sums of the hop (dots[nb][N])
constexpr int PB_DOT_PARTS = 64;
__global__ void __launch_bounds__(256)
k_pb_dot_sum(const double* __restrict__ dots, int N, long nb, double* __restrict__ partials,
             const PbState* __restrict__ st) {
    if (st->halt) return;
    __shared__ double red[256];
    const int tp = 256 / N, j = threadIdx.x % N;
    double s = 0.0;
    if (threadIdx.x < tp * N) {
        const long step = (long)gridDim.x * tp;
#pragma unroll 4
        for (long b = (long)blockIdx.x * tp + threadIdx.x / N; b < nb; b += step) s += dots[b * N + j];
    }
    pb_rows_sum(s, red, N, tp, partials);
}

__global__ void __launch_bounds__(256)
k_pb_update1_rows(double2* __restrict__ R, const double2* __restrict__ AP, int N, long rows,
                  double* __restrict__ partials, const PbState* __restrict__ st) {
    if (st->halt) return;
    __shared__ double red[256];
    const int tp = 256 / N, j = threadIdx.x % N;
    double s = 0.0;
    if (threadIdx.x < tp * N && st->active[j]) {
        const double a = st->alpha[j];
        const long step = (long)gridDim.x * tp;
#pragma unroll 4
        for (long r0 = (long)blockIdx.x * tp + threadIdx.x / N; r0 < rows; r0 += step) {
            const long o = r0 * N + j;
            const double2 ap = ld_stream(AP + o);
            double2 r = R[o];
            r.x = fma(-a, ap.x, r.x);
            r.y = fma(-a, ap.y, r.y);
            R[o] = r;
            s += r.x * r.x + r.y * r.y;
        }
    }
    pb_rows_sum(s, red, N, tp, partials);
}

__global__ void __launch_bounds__(256)
k_pb_update2_rows(double2* __restrict__ X, double2* __restrict__ P, const double2* __restrict__ R, int N, long rows,
                  const PbState* __restrict__ st) {
    if (!st->step) return;
    const int tp = 256 / N, j = threadIdx.x % N;
    if (threadIdx.x >= tp * N) return;
    const double a = st->alpha[j], b = st->beta[j];
    if (a == 0.0) return;
    const bool go = st->active[j];
    const long step = (long)gridDim.x * tp;
#pragma unroll 4
    for (long r0 = (long)blockIdx.x * tp + threadIdx.x / N; r0 < rows; r0 += step) {
        const long o = r0 * N + j;
        double2 p = P[o], x = ld_stream(X + o);
        const double2 r = go ? R[o] : p;
        x.x = fma(a, p.x, x.x);
        x.y = fma(a, p.y, x.y);
        st_stream(X + o, x);
        p.x = fma(b, p.x, r.x);
        p.y = fma(b, p.y, r.y);
        if (go) P[o] = p;
    }
}

// R and P from the true residual Rt on the columns that restart
__global__ void __launch_bounds__(256)
k_pb_restart_rows(double2* __restrict__ R, double2* __restrict__ P, const double2* __restrict__ Rt, int N, long n,
                  const int* __restrict__ restart) {
    for (long t = (long)blockIdx.x * 256 + threadIdx.x; t < n; t += (long)gridDim.x * 256)
        if (restart[t % N]) R[t] = P[t] = Rt[t];
}

// start (or restart from the true residual) the columns whose flag is set:
// rr_j = |r_j|^2 from the colnorm partials [b][N]; the others keep their state
__global__ void k_pb_start(const double* __restrict__ partials, int nb, int N, PbState* st,
                           const int* __restrict__ restart, double tol, int first) {
    const int j = threadIdx.x;
    if (threadIdx.x == 0) {
        st->halt = 0;
        st->reason = HALT_NONE;
        st->tol = tol;
        if (first) st->iters = 0;
    }
    if (j < N) {
        if (first || restart[j]) {
            double rr = 0.0;
            for (int b = 0; b < nb; ++b) rr += partials[(long)b * N + j];
            st->rr[j] = rr;
            if (first) {
                st->bnorm[j] = sqrt(rr);
                st->col_iters[j] = 0;
            }
            st->relres[j] = sqrt(rr) / st->bnorm[j];
            st->active[j] = 1;
        } else {
            st->active[j] = 0;
        }
        st->alpha[j] = 0.0;
        st->beta[j] = 0.0;
    }
}

// workgroups of the row kernels: the same count as partials per column as the planes'
static dim3 pb_rows_grid(int Vh) { return dim3(pb_blocks(Vh)); }

hipError_t launch_pb_dot(const double2* P, const double2* AP, int N, int Vh, double* partials, const PbState* st,
                         hipStream_t s) {
    hipLaunchKernelGGL(k_pb_dot, dim3(pb_blocks(Vh), N), dim3(256), 0, s, P, AP, Vh, partials, st);
    return hipGetLastError();
}
hipError_t launch_pb_dot_sum(const double* dots, int N, int Vh, double* partials, const PbState* st, hipStream_t s) {
    hipLaunchKernelGGL(k_pb_dot_sum, dim3(PB_DOT_PARTS), dim3(256), 0, s, dots, N, row_blocks(N, Vh), partials, st);
    return hipGetLastError();
}
hipError_t launch_pb_alpha(const double* partials, int N, int Vh, bool rows, PbState* st, hipStream_t s) {
    hipLaunchKernelGGL(k_pb_alpha, dim3(1), dim3(1024), 0, s, partials, rows ? PB_DOT_PARTS : pb_blocks(Vh), N, st);
    return hipGetLastError();
}
hipError_t launch_pb_update1(double2* R, const double2* AP, int N, int Vh, bool rows, double* partials,
                             const PbState* st, hipStream_t s) {
    if (rows) hipLaunchKernelGGL(k_pb_update1_rows, pb_rows_grid(Vh), dim3(256), 0, s, R, AP, N, 3L * Vh, partials, st);
    else hipLaunchKernelGGL(k_pb_update1, dim3(pb_blocks(Vh), N), dim3(256), 0, s, R, AP, Vh, partials, st);
    return hipGetLastError();
}
hipError_t launch_pb_beta(const double* partials, int N, int Vh, PbState* st, hipStream_t s) {
    hipLaunchKernelGGL(k_pb_beta, dim3(1), dim3(1024), 0, s, partials, pb_blocks(Vh), N, st);
    return hipGetLastError();
}
hipError_t launch_pb_update2(double2* X, double2* P, const double2* R, int N, int Vh, bool rows, const PbState* st,
                             hipStream_t s) {
    if (rows) hipLaunchKernelGGL(k_pb_update2_rows, dim3(4 * pb_blocks(Vh)), dim3(256), 0, s, X, P, R, N, 3L * Vh, st);
    else hipLaunchKernelGGL(k_pb_update2, dim3(pb_blocks(Vh), N), dim3(256), 0, s, X, P, R, Vh, st);
    return hipGetLastError();
}
hipError_t launch_pb_restart_rows(double2* R, double2* P, const double2* Rt, int N, int Vh, const int* restart,
                                  hipStream_t s) {
    hipLaunchKernelGGL(k_pb_restart_rows, dim3(4 * pb_blocks(Vh)), dim3(256), 0, s, R, P, Rt, N, 3L * Vh * N, restart);
    return hipGetLastError();
}
hipError_t launch_pb_start(const double* colnorm_partials, int N, int Vh, PbState* st, const int* restart,
                           double tol, int first, hipStream_t s) {
    hipLaunchKernelGGL(k_pb_start, dim3(1), dim3(64), 0, s, colnorm_partials, pb_blocks(Vh), N, st, restart, tol,
                       first);
    return hipGetLastError();
}

}  // namespace bcg
