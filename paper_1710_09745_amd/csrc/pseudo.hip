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
// 117 + 56 -> 61 + 89 us).  On planes of up to 16384 sites, where a transfer costs nothing
// beside a kernel's start, x goes with r: the longer chain of loads is the first kernel's,
// which waits for its sum anyway (4^4, N = 1, an iteration 24.5 -> 23.5 us).
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

// Partials of a sum per column: number b of column j at j * sj + b * sb, nb of them, by ln
// lanes a column (a power of two from 16 to 128).
struct PbSum {
    const double* p;
    int nb, sj, sb, ln;
};

// The sum of column j = threadIdx.x / ln in a fixed order: lane g of the column takes
// b = g, g + ln, ... (eight loads in flight), 16 lanes meet in a butterfly, the groups of 16
// in order.  Valid on lane 0 of each column; red: a double per thread.
__device__ __forceinline__ double pb_column_sum(const PbSum& t, int N, double* red) {
    const int j = threadIdx.x / t.ln, g = threadIdx.x & (t.ln - 1);
    double v = 0.0;
    if (j < N)
        for (int b0 = g; b0 < t.nb; b0 += 8 * t.ln) {
            double x[8];
#pragma unroll
            for (int u = 0; u < 8; ++u)
                x[u] = b0 + u * t.ln < t.nb ? t.p[(long)j * t.sj + (long)(b0 + u * t.ln) * t.sb] : 0.0;
#pragma unroll
            for (int u = 0; u < 8; ++u) v += x[u];
        }
    for (int off = 8; off > 0; off >>= 1) v += __shfl_xor(v, off, 16);
    if (t.ln == 16) return v;
    red[threadIdx.x] = v;
    __syncthreads();
    double s = 0.0;
    if (g == 0)
        for (int q = 0; q < t.ln; q += 16) s += red[threadIdx.x + q];
    return s;
}

// alpha_j = rr_j / p_j^H A p_j for the active columns (0 for the others)
__global__ void __launch_bounds__(1024) k_pb_alpha(PbSum dots, int N, PbState* st) {
    if (st->halt) {
        if (threadIdx.x == 0) st->step = 0;
        return;
    }
    __shared__ double red[1024];
    const int j = threadIdx.x / dots.ln;
    const double pap = pb_column_sum(dots, N, red);
    if (threadIdx.x == 0) st->step = 1;
    __syncthreads();
    if (j < N && (threadIdx.x & (dots.ln - 1)) == 0) {
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
// (XNOW: and x_j += alpha_j p_j)
template <bool XNOW>
__global__ void __launch_bounds__(256)
k_pb_update1(double2* __restrict__ X, double2* __restrict__ R, const double2* __restrict__ P,
             const double2* __restrict__ AP, int Vh, double* __restrict__ partials, const PbState* __restrict__ st) {
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
                if constexpr (XNOW) {
                    const double2 p = P[o];
                    double2 x = X[o];
                    x.x = fma(a, p.x, x.x);
                    x.y = fma(a, p.y, x.y);
                    X[o] = x;
                }
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
__global__ void __launch_bounds__(1024) k_pb_beta(PbSum rrs, int N, PbState* st) {
    if (st->halt) return;
    __shared__ int still;
    __shared__ double red[1024];
    if (threadIdx.x == 0) still = 0;
    __syncthreads();
    const int j = threadIdx.x / rrs.ln;
    const double rr = pb_column_sum(rrs, N, red);
    if (j < N && (threadIdx.x & (rrs.ln - 1)) == 0 && st->active[j]) {
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

// x_j += alpha_j p_j (alpha = 0: no step; XNOW: done already), then p_j = r_j + beta_j p_j
// for the columns still active; after a halt that came with a step, x alone
template <bool XNOW>
__global__ void __launch_bounds__(256)
k_pb_update2(double2* __restrict__ X, double2* __restrict__ P, const double2* __restrict__ R, int Vh,
             const PbState* __restrict__ st) {
    const int j = blockIdx.y, moved = st->step;
    const double a = st->alpha[j], b = st->beta[j];
    const bool go = st->active[j] && !st->halt;
    if (XNOW ? !go : (!moved || a == 0.0)) return;
    for (long i = (long)blockIdx.x * 256 + threadIdx.x; i < Vh; i += (long)gridDim.x * 256)
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            const long o = ((long)j * 3 + c) * Vh + i;
            double2 p = P[o];
            if constexpr (!XNOW) {
                double2 x = X[o];
                x.x = fma(a, p.x, x.x);
                x.y = fma(a, p.y, x.y);
                X[o] = x;
            }
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
// are added in a fixed order (partials [j][b] as above).
__device__ __forceinline__ void pb_rows_sum(double v, double* red, int N, int tp, double* __restrict__ partials) {
    red[threadIdx.x] = v;
    __syncthreads();
    // rows q, q + 8, ... by the threads of row q < 8, then those eight in order
    if (tp >= 16) {
        double s = 0.0;
        if (threadIdx.x < 8 * N)
            for (int r = threadIdx.x; r < tp * N; r += 8 * N) s += red[r];
        __syncthreads();
        red[threadIdx.x] = s;
        __syncthreads();
        tp = 8;
    }
    if (threadIdx.x < N) {
        double s = 0.0;
        for (int q = 0; q < tp; ++q) s += red[q * N + threadIdx.x];
        partials[(long)threadIdx.x * gridDim.x + blockIdx.x] = s;
    }
}

// partials of p^H A p per column from the block sums of the hop (dots[nb][N]), where they
// are more than the one workgroup of k_pb_alpha reads in the time of another launch
constexpr int PB_DOT_PARTS = 64, PB_DOTS_DIRECT = 512;
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
    const int tp = 256 / N, j = threadIdx.x % N, moved = st->step;
    const double a = st->alpha[j], b = st->beta[j];
    const bool go = st->active[j];
    if (!moved || a == 0.0 || threadIdx.x >= tp * N) return;
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

// Workgroups of the row kernels, from the numbers of a block: one a thread for up to two
// workgroups per CU, then four, and at most `most` (by sites alone most of the chip was idle
// on small lattices: both updates at 8^4, N = 32 49 -> 12 us, 16^4, N = 24 71 -> 50).
static int pb_rows_blocks(int N, int Vh, int most) {
    const long tp = 256 / N, one = (3L * Vh + tp - 1) / tp, four = (one + 3) / 4;
    const long g = one < 512 ? one : (four < 512 ? 512 : four);
    return (int)(g < most ? g : most);
}
// (at most what the memory of the partials holds, and few enough for the one workgroup that sums them)
static int pb_update1_parts(int N, int Vh, bool rows) {
    const int most = NORM_BLOCKS * MAXN / N;
    return rows ? pb_rows_blocks(N, Vh, most < 1024 ? most : 1024) : pb_blocks(Vh);
}

// planes: x together with r instead of with p
static bool pb_xnow(int Vh) { return Vh <= 16384; }

// lanes a column for nb partials: more than 16 where each would add more than eight
static int pb_lanes(int N, int nb) {
    int ln = 16;
    while (ln < 128 && 2 * ln * N <= 1024 && 8 * ln < nb) ln *= 2;
    return ln;
}
static dim3 pb_sum_threads(const PbSum& t, int N) { return dim3((t.ln * N + 63) / 64 * 64); }

hipError_t launch_pb_dot(const double2* P, const double2* AP, int N, int Vh, double* partials, const PbState* st,
                         hipStream_t s) {
    hipLaunchKernelGGL(k_pb_dot, dim3(pb_blocks(Vh), N), dim3(256), 0, s, P, AP, Vh, partials, st);
    return hipGetLastError();
}
hipError_t launch_pb_alpha(const double* dots, double* partials, int N, int Vh, bool rows, PbState* st, hipStream_t s) {
    PbSum t{dots, pb_blocks(Vh), pb_blocks(Vh), 1, 0};
    if (rows) {
        const int nb = row_blocks(N, Vh);
        t = PbSum{dots, nb, 1, N, 0};
        if (nb > PB_DOTS_DIRECT) {
            hipLaunchKernelGGL(k_pb_dot_sum, dim3(PB_DOT_PARTS), dim3(256), 0, s, dots, N, nb, partials, st);
            t = PbSum{partials, PB_DOT_PARTS, PB_DOT_PARTS, 1, 0};
        }
    }
    t.ln = pb_lanes(N, t.nb);
    hipLaunchKernelGGL(k_pb_alpha, dim3(1), pb_sum_threads(t, N), 0, s, t, N, st);
    return hipGetLastError();
}
hipError_t launch_pb_update1(double2* X, double2* R, const double2* P, const double2* AP, int N, int Vh, bool rows, double* partials,
                             const PbState* st, hipStream_t s) {
    const int nb = pb_update1_parts(N, Vh, rows);
    const dim3 grid(nb, N);
    if (rows) hipLaunchKernelGGL(k_pb_update1_rows, dim3(nb), dim3(256), 0, s, R, AP, N, 3L * Vh, partials, st);
    else if (pb_xnow(Vh)) hipLaunchKernelGGL(k_pb_update1<true>, grid, dim3(256), 0, s, X, R, P, AP, Vh, partials, st);
    else hipLaunchKernelGGL(k_pb_update1<false>, grid, dim3(256), 0, s, X, R, P, AP, Vh, partials, st);
    return hipGetLastError();
}
hipError_t launch_pb_beta(const double* partials, int N, int Vh, bool rows, PbState* st, hipStream_t s) {
    const int nb = pb_update1_parts(N, Vh, rows);
    const PbSum t{partials, nb, nb, 1, pb_lanes(N, nb)};
    hipLaunchKernelGGL(k_pb_beta, dim3(1), pb_sum_threads(t, N), 0, s, t, N, st);
    return hipGetLastError();
}
hipError_t launch_pb_update2(double2* X, double2* P, const double2* R, int N, int Vh, bool rows, const PbState* st,
                             hipStream_t s) {
    if (rows)
        hipLaunchKernelGGL(k_pb_update2_rows, dim3(pb_rows_blocks(N, Vh, 2048)), dim3(256), 0, s, X, P, R, N, 3L * Vh,
                           st);
    else if (pb_xnow(Vh)) hipLaunchKernelGGL(k_pb_update2<true>, dim3(pb_blocks(Vh), N), dim3(256), 0, s, X, P, R, Vh, st);
    else hipLaunchKernelGGL(k_pb_update2<false>, dim3(pb_blocks(Vh), N), dim3(256), 0, s, X, P, R, Vh, st);
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
