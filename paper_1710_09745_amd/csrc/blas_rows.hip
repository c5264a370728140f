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

// ---------------------------------------------------------------------------------------------
// Streaming kernels.  A wave takes 4 sites (half rows: 8) and all N columns, NT tiles of
// 16 (half rows: one tile of 8); lane (site, column) holds the three colours of its
// column, so a product with an N x N matrix needs the other columns of the same site:
// the DPP row broadcasts of mac3 supply them, and the coefficients M[l][j] are one LDS
// read per 12 or 36 multiply-adds.  The same lane layout is the operand layout of
// v_mfma_f64_16x16x4f64 (lane l supplies A[l % 16][l / 16]) with the four sites as the
// contraction index, so a Gram product needs neither LDS nor a second read of its block.
// ---------------------------------------------------------------------------------------------
// one wave's sites and columns
template <typename S, int NT, bool HR> struct RowLane {
    int i;         // site (clamped)
    bool live;     // a real site
    int cl;        // column within the tile
    __device__ __forceinline__ void at(int sb, int w, int lane, int Vh) {
        const int i0 = sb * row_block_sites<HR>() + (w & 3) * (row_block_sites<HR>() / 4) + row_lane_site<HR>(lane);
        live = i0 < Vh;
        i = live ? i0 : Vh - 1;
        cl = row_lane_col<HR>(lane);
    }
    __device__ __forceinline__ int col(int t) const { return t * 16 + cl; }
    // row_cs of column tile t, and its byte offset, in storage T (columns past N: column N - 1)
    template <typename T> __device__ __forceinline__ unsigned cs(int t, int N) const {
        return row_cs<T>(N, col(t) < N ? col(t) : N - 1);
    }
    template <typename T> __device__ __forceinline__ unsigned off(int t, int N) const {
        const int c = col(t) < N ? col(t) : N - 1;
        return (unsigned)i * row_ss<T>(N) + (unsigned)c * row_col_bytes<T>();
    }
};

// acc += (values of columns 0 .. M - 1 of the tile held in v) x the coefficients m(l),
// l = 0 .. M - 1, of the lane's output column
template <bool HR, int M, typename R, typename F>
__device__ __forceinline__ void row_product_m(C2<R> acc[3], const C2<R> v[3], F&& m) {
    static_for<M>([&](auto lc) {
        constexpr int l = decltype(lc)::value;
        const C2<R> b = m(l);
        if constexpr (HR) {
            mac3<l, 0x3>(acc, v[0], v[1], v[2], b);
            mac3<8 + l, 0xc>(acc, v[0], v[1], v[2], b);
        } else {
            mac3<l, 0xf>(acc, v[0], v[1], v[2], b);
        }
    });
}
// all columns of a tile: 8 in a half row, and in the last of several tiles (T8) that has
// at most 8, else 16.  At 17 to 24 columns the passes are bound by these multiply-adds, and
// three eighths of a 32 x 32 product is padding that the shorter tile halves (24^4, N = 24,
// 16-bit: pass A 128 -> 113, pass B 201 -> 167 us)
template <bool HR, bool T8, typename R, typename F>
__device__ __forceinline__ void row_product(C2<R> acc[3], const C2<R> v[3], bool last, F&& m) {
    if (HR || (T8 && last)) row_product_m<HR, 8>(acc, v, m);
    else row_product_m<HR, HR ? 8 : 16>(acc, v, m);
}
// Arithmetic of the passes' products and sums on NT tiles: that of the storage, but FP64 for
// FP32 storage on two tiles, with one rounding as a result is stored: sums over 17 to 32
// columns in FP32 leave errors of 2e-7 in the iterates, which with FP64 sums are those of the
// stored numbers alone.  (An iteration, us, FP32 / FP64 sums: 16^3 x 48, N = 32 526 / 560,
// 24^4, N = 24 716 / 761; with the plane kernels, whose products are FP64, 778 and 1138.)
template <typename S, int NT> struct PassReal { using type = typename S::real; };
template <> struct PassReal<F32, 2> { using type = double; };
template <typename S, typename R> __device__ __forceinline__ void row_get(const RowRaw<S>& raw, C2<R> o[3]) {
    C2<typename S::real> v[3];
    raw.get(v);
#pragma unroll
    for (int c = 0; c < 3; ++c) o[c] = C2<R>{(R)v[c].re, (R)v[c].im};
}
// Waves of a Gram workgroup: four from three tiles on, whose accumulators need more
// than the 256 registers a lane has in a workgroup of eight.
constexpr int row_gram_nw(int nt) { return nt <= 2 ? ROW_NW : 4; }

// Gram partials of A^H B (SAME: of A^H A), one per workgroup.  Bound by its reads up to
// N = 32, by the matrix cores beyond.
template <typename S, int NT, bool HR, bool SAME>
__global__ void __launch_bounds__(64 * row_gram_nw(NT))
k_gram_rows(const char* __restrict__ A, const char* __restrict__ B, int N, int Vh, RowOrder ord, int nb, int ld,
            double2* __restrict__ partials, const int* __restrict__ halt) {
    constexpr int NW = row_gram_nw(NT);
    extern __shared__ double red[];
    if (halt != nullptr && *halt) return;
    const int lane = threadIdx.x & 63;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const rsrc_t ra = make_rsrc(A), rb = make_rsrc(B);
    RowGram<NT, SAME> G;
    G.zero();
    RowLane<S, NT, HR> L;
    RowRaw<S> a[NT], b[SAME ? 1 : NT];
    bool live;
    auto fetch = [&](int sb) {
        L.at(sb, w, lane, Vh);
        live = L.live;
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            const unsigned o = L.template off<S>(t, N);
            a[t].load(ra, o, L.template cs<S>(t, N));
            if constexpr (!SAME) b[t].load(rb, o, L.template cs<S>(t, N));
        }
    };
    int it = 0;
    int sb = row_turn(0, blockIdx.x, gridDim.x, NW / 4, w >> 2, nb, ord);
    if (sb >= 0) fetch(sb);
    while (sb >= 0) {
        C2<typename S::real> va[NT][3], vb[SAME ? 1 : NT][3];
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            a[t].get(va[t]);
            if constexpr (!SAME) b[t].get(vb[t]);
        }
        const bool ok = live;
        sb = row_turn(++it, blockIdx.x, gridDim.x, NW / 4, w >> 2, nb, ord);
        if (sb >= 0) fetch(sb);
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            double ar[NT], ai[NT], br[NT], bi[NT];
#pragma unroll
            for (int t = 0; t < NT; ++t) {
                ar[t] = ok ? (double)va[t][c].re : 0.0;
                ai[t] = ok ? (double)va[t][c].im : 0.0;
                br[t] = SAME ? ar[t] : (double)vb[SAME ? 0 : t][c].re;
                bi[t] = SAME ? ai[t] : (double)vb[SAME ? 0 : t][c].im;
            }
            G.add(ar, ai, br, bi);
        }
    }
    G.template finish<NW, HR>(red, partials + (long)blockIdx.x * ld * ld, ld);
}

// Pass A: Q <- Q - AP beta and, with GR, the partials of H = Qt^H Qt of the stored Qt
// (its own kernel for three and four tiles, whose accumulators would not leave room).
// Bound by the read of Q and AP and the write of Q.
template <typename S, int NT, bool HR, bool T8, bool GR>
__global__ void __launch_bounds__(64 * ROW_NW)
k_pass_a_rows(char* __restrict__ Q, const char* __restrict__ AP, const double2* __restrict__ beta, int N, int Vh,
              RowOrder ord, int nb, int ld, double2* __restrict__ partials, const int* __restrict__ halt) {
    using R = typename PassReal<S, NT>::type;
    constexpr int NP = HR ? 8 : 16 * NT;
    extern __shared__ unsigned char lds[];
    C2<R>* cf = reinterpret_cast<C2<R>*>(lds);  // [NP][NP], zero outside N x N
    if (halt != nullptr && *halt) return;
    const int lane = threadIdx.x & 63;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    for (int e = threadIdx.x; e < NP * NP; e += 64 * ROW_NW) {
        const int l = e / NP, j = e % NP;
        const double2 b = (l < N && j < N) ? beta[l * MAXN + j] : make_double2(0.0, 0.0);
        cf[e] = C2<R>{(R)b.x, (R)b.y};
    }
    __syncthreads();
    const rsrc_t rq = make_rsrc(Q), ra = make_rsrc(AP);
    RowGram<GR ? NT : 1, true> G;
    if constexpr (GR) G.zero();
    RowLane<S, NT, HR> L;
    if constexpr (NT <= 2) {
        RowRaw<S> a[NT], q[NT];
        int it = 0;
        int sb = row_turn(0, blockIdx.x, gridDim.x, ROW_NW / 4, w >> 2, nb, ord);
        auto fetch = [&]() {
            L.at(sb, w, lane, Vh);
#pragma unroll
            for (int t = 0; t < NT; ++t) {
                const unsigned o = L.template off<S>(t, N);
                a[t].load(ra, o, L.template cs<S>(t, N));
                q[t].load(rq, o, L.template cs<S>(t, N));
            }
        };
        if (sb >= 0) fetch();
        while (sb >= 0) {
            C2<R> av[NT][3], qv[NT][3];
#pragma unroll
            for (int t = 0; t < NT; ++t) {
                row_get<S>(a[t], av[t]);
                row_get<S>(q[t], qv[t]);
            }
            const RowLane<S, NT, HR> M = L;
            sb = row_turn(++it, blockIdx.x, gridDim.x, ROW_NW / 4, w >> 2, nb, ord);
            if (sb >= 0) fetch();
#pragma unroll
            for (int t = 0; t < NT; ++t) {
                C2<R> acc[3] = {c2<R>(0, 0), c2<R>(0, 0), c2<R>(0, 0)};
#pragma unroll
                for (int lt = 0; lt < NT; ++lt)
                    row_product<HR, T8>(acc, av[lt], lt == NT - 1, [&](int l) { return cf[(lt * 16 + l) * NP + t * 16 + M.cl]; });
#pragma unroll
                for (int c = 0; c < 3; ++c) {
                    qv[t][c].re -= acc[c].re;
                    qv[t][c].im -= acc[c].im;
                }
                const bool st = M.live && M.col(t) < N;
                row_store_rt<S, R>(Q, M.template off<S>(t, N), M.template cs<S>(t, N), qv[t], st);
            }
            if constexpr (GR) {
#pragma unroll
                for (int c = 0; c < 3; ++c) {
                    double xr[NT], xi[NT];
#pragma unroll
                    for (int t = 0; t < NT; ++t) {
                        xr[t] = M.live ? (double)qv[t][c].re : 0.0;
                        xi[t] = M.live ? (double)qv[t][c].im : 0.0;
                    }
                    G.add(xr, xi, xr, xi);
                }
            }
        }
    } else {
        // three or four tiles: one output tile at a time, the operand tiles re-read from L1
        int it = 0;
        for (int sb; (sb = row_turn(it, blockIdx.x, gridDim.x, ROW_NW / 4, w >> 2, nb, ord)) >= 0; ++it) {
            L.at(sb, w, lane, Vh);
#pragma unroll 1
            for (int t = 0; t < NT; ++t) {
                RowRaw<S> qr;
                qr.load(rq, L.template off<S>(t, N), L.template cs<S>(t, N));
                C2<R> acc[3] = {c2<R>(0, 0), c2<R>(0, 0), c2<R>(0, 0)};
#pragma unroll 1
                for (int lt = 0; lt < NT; ++lt) {
                    RowRaw<S> ar;
                    ar.load(ra, L.template off<S>(lt, N), L.template cs<S>(lt, N));
                    C2<R> av[3];
                    row_get<S>(ar, av);
                    const C2<R>* m = cf + lt * 16 * NP + t * 16 + L.cl;
                    row_product<HR, T8>(acc, av, lt == NT - 1, [&](int l) { return m[l * NP]; });
                }
                C2<R> qv[3];
                row_get<S>(qr, qv);
#pragma unroll
                for (int c = 0; c < 3; ++c) {
                    qv[c].re -= acc[c].re;
                    qv[c].im -= acc[c].im;
                }
                row_store_rt<S, R>(Q, L.template off<S>(t, N), L.template cs<S>(t, N), qv, L.live && L.col(t) < N);
            }
        }
    }
    if constexpr (GR) G.template finish<ROW_NW, HR>(reinterpret_cast<double*>(lds), partials + (long)blockIdx.x * ld * ld, ld);
}

// Pass B: X += P (beta C) in FP64, Qn = Qt S^{-1}, Pn = Qn + P S^H, as pb_mode selects.
// Qn and Pn may be Qt and P up to two tiles, whose columns of a site are all loaded before
// any is stored.  X is touched by this kernel alone, once an iteration, so its loads and
// stores carry the streaming hint: with that and the update in place, the vectors of the
// hops stay in the Infinity Cache (an iteration, us: 16^4, N = 16, FP64 160 -> 148, of
// which both hops 78.5 -> 71; 16^3 x 48, N = 32, FP32 550 -> 535).
// LDS: beta C whole, the upper tiles of S^{-1} and the lower tiles of S^H (the others
// are zero), [l][j] within a tile.
template <typename S, int NT, bool HR, bool T8>
__global__ void __launch_bounds__(64 * ROW_NW)
k_pass_b_rows(double2* __restrict__ X, const char* Qt, const char* P, char* Qn, char* Pn,
              const double2* __restrict__ betaC, const double2* __restrict__ Sinv, const double2* __restrict__ SH, int N,
              int Vh, RowOrder ord, int nb, const SolveState* __restrict__ stt) {
    using R = typename PassReal<S, NT>::type;
    constexpr int TW = HR ? 8 : 16, NP = TW * NT, TE = TW * TW, NUP = NT * (NT + 1) / 2;
    extern __shared__ unsigned char lds[];
    C2<double>* cx = reinterpret_cast<C2<double>*>(lds);         // [NP][NP]
    C2<R>* ci = reinterpret_cast<C2<R>*>(cx + NP * NP);          // tile (lt <= jt) at jt (jt + 1) / 2 + lt
    C2<R>* ch = ci + NUP * TE;                                   // tile (lt >= jt) at lt (lt + 1) / 2 + jt
    const int mode = stt->pb_mode;
    if (mode == PB_SKIP) return;
    const bool full = mode == PB_FULL;
    const int lane = threadIdx.x & 63;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    for (int e = threadIdx.x; e < NP * NP; e += 64 * ROW_NW) {
        const int l = e / NP, j = e % NP, lt = l / TW, jt = j / TW;
        const bool in = l < N && j < N;
        const double2 z = make_double2(0.0, 0.0);
        const double2 b = in ? betaC[l * MAXN + j] : z;
        cx[e] = C2<double>{b.x, b.y};
        const int k = (l % TW) * TW + j % TW;
        if (lt <= jt) {
            const double2 v = in && l <= j ? Sinv[l * MAXN + j] : z;
            ci[(jt * (jt + 1) / 2 + lt) * TE + k] = C2<R>{(R)v.x, (R)v.y};
        }
        if (lt >= jt) {
            const double2 v = in && l >= j ? SH[l * MAXN + j] : z;
            ch[(lt * (lt + 1) / 2 + jt) * TE + k] = C2<R>{(R)v.x, (R)v.y};
        }
    }
    __syncthreads();
    const rsrc_t rq = make_rsrc(Qt), rp = make_rsrc(P), rx = make_rsrc(X);
    RowLane<S, NT, HR> L;
    // one operand tile into the sums of output tile jt
    auto tile = [&](int lt, int jt, const C2<R> pv[3], const C2<R> qv[3], C2<double> xa[3], C2<R> pa[3], C2<R> qa[3]) {
        C2<double> pd[3];
#pragma unroll
        for (int c = 0; c < 3; ++c) pd[c] = C2<double>{(double)pv[c].re, (double)pv[c].im};
        const C2<double>* mx = cx + lt * TW * NP + jt * TW + L.cl;
        row_product<HR, T8>(xa, pd, lt == NT - 1, [&](int l) { return mx[l * NP]; });
        if (!full) return;
        if (lt >= jt) {
            const C2<R>* m = ch + (lt * (lt + 1) / 2 + jt) * TE + L.cl;
            row_product<HR, T8>(pa, pv, lt == NT - 1, [&](int l) { return m[l * TW]; });
        }
        if (lt <= jt) {
            const C2<R>* m = ci + (jt * (jt + 1) / 2 + lt) * TE + L.cl;
            row_product<HR, T8>(qa, qv, lt == NT - 1, [&](int l) { return m[l * TW]; });
        }
    };
    auto store = [&](int jt, const RowRaw<F64>& xr, C2<double> xa[3], C2<R> pa[3], C2<R> qa[3]) {
        if (!(L.live && L.col(jt) < N)) return;
        const unsigned o = L.template off<S>(jt, N), ox = L.template off<F64>(jt, N);
        C2<double> x[3];
        xr.get(x);
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            x[c].re += xa[c].re;
            x[c].im += xa[c].im;
        }
        row_store_nt(X, ox, L.template cs<F64>(jt, N), x);
        if (!full) return;
        C2<R> qs[3] = {qa[0], qa[1], qa[2]};
        row_store_rt<S, R>(Qn, o, L.template cs<S>(jt, N), qs, true);
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            // with sums finer than the storage, P' is formed from Q' as stored
            const C2<R> q = std::is_same<R, typename S::real>::value ? qa[c] : qs[c];
            pa[c].re += q.re;
            pa[c].im += q.im;
        }
        row_store<S, R>(Pn, o, L.template cs<S>(jt, N), pa);
    };
    if constexpr (NT <= 2) {
        RowRaw<S> p[NT], q[NT];
        RowRaw<F64> x[NT];
        int it = 0;
        int sb = row_turn(0, blockIdx.x, gridDim.x, ROW_NW / 4, w >> 2, nb, ord);
        while (sb >= 0) {
            L.at(sb, w, lane, Vh);
#pragma unroll
            for (int t = 0; t < NT; ++t) {
                const unsigned o = L.template off<S>(t, N);
                p[t].load(rp, o, L.template cs<S>(t, N));
                q[t].load(rq, o, L.template cs<S>(t, N));
                x[t].template load<AUX_NT>(rx, L.template off<F64>(t, N), L.template cs<F64>(t, N));
            }
            C2<R> pv[NT][3], qv[NT][3];
#pragma unroll
            for (int t = 0; t < NT; ++t) {
                row_get<S>(p[t], pv[t]);
                row_get<S>(q[t], qv[t]);
            }
#pragma unroll
            for (int jt = 0; jt < NT; ++jt) {
                C2<double> xa[3] = {};
                C2<R> pa[3] = {}, qa[3] = {};
#pragma unroll
                for (int lt = 0; lt < NT; ++lt) tile(lt, jt, pv[lt], qv[lt], xa, pa, qa);
                store(jt, x[jt], xa, pa, qa);
            }
            sb = row_turn(++it, blockIdx.x, gridDim.x, ROW_NW / 4, w >> 2, nb, ord);
        }
    } else {
        int it = 0;
        for (int sb; (sb = row_turn(it, blockIdx.x, gridDim.x, ROW_NW / 4, w >> 2, nb, ord)) >= 0; ++it) {
            L.at(sb, w, lane, Vh);
#pragma unroll 1
            for (int jt = 0; jt < NT; ++jt) {
                RowRaw<F64> xr;
                xr.template load<AUX_NT>(rx, L.template off<F64>(jt, N), L.template cs<F64>(jt, N));
                C2<double> xa[3] = {};
                C2<R> pa[3] = {}, qa[3] = {};
#pragma unroll 1
                for (int lt = 0; lt < NT; ++lt) {
                    RowRaw<S> pr, qr;
                    const unsigned o = L.template off<S>(lt, N);
                    pr.load(rp, o, L.template cs<S>(lt, N));
                    if (lt <= jt) qr.load(rq, o, L.template cs<S>(lt, N));
                    C2<R> pv[3], qv[3];
                    row_get<S>(pr, pv);
                    row_get<S>(qr, qv);
                    tile(lt, jt, pv, qv, xa, pa, qa);
                }
                store(jt, xr, xa, pa, qa);
            }
        }
    }
}

// Y <- Z + X M in FP64 arithmetic (Z may be NULL; M NULL: the identity, X in another
// storage), all buffers distinct
template <typename SX, typename SY, bool HR>
__global__ void __launch_bounds__(64 * ROW_NW)
k_bmul_rows(const char* __restrict__ X, const char* __restrict__ Z, char* __restrict__ Y,
            const double2* __restrict__ M, int N, int Vh, RowOrder ord, int nb, const int* __restrict__ skip) {
    extern __shared__ unsigned char lds[];
    C2<double>* cf = reinterpret_cast<C2<double>*>(lds);  // [np][np]
    if (skip != nullptr && *skip) return;
    const int lane = threadIdx.x & 63;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int nt = HR ? 1 : (N + 15) / 16, np = HR ? 8 : 16 * nt;
    for (int l = threadIdx.x / np; l < np && M != nullptr; l += 64 * ROW_NW / np) {
        const int j = threadIdx.x % np;
        if (threadIdx.x >= (64 * ROW_NW / np) * np) break;
        const double2 b = (l < N && j < N) ? M[l * MAXN + j] : make_double2(0.0, 0.0);
        cf[l * np + j] = C2<double>{b.x, b.y};
    }
    __syncthreads();
    const rsrc_t rx = make_rsrc(X), rz = make_rsrc(Z != nullptr ? Z : X);
    RowLane<SX, 4, HR> L;
    int it = 0;
    for (int sb; (sb = row_turn(it, blockIdx.x, gridDim.x, ROW_NW / 4, w >> 2, nb, ord)) >= 0; ++it) {
        L.at(sb, w, lane, Vh);
#pragma unroll 1
        for (int t = 0; t < nt; ++t) {
            C2<double> acc[3] = {};
#pragma unroll 1
            for (int lt = M != nullptr ? 0 : t; lt < (M != nullptr ? nt : t + 1); ++lt) {
                RowRaw<SX> xr;
                xr.load(rx, L.template off<SX>(lt, N), L.template cs<SX>(lt, N));
                C2<double> xd[3];
                row_get<SX>(xr, xd);
                if (M == nullptr) {
#pragma unroll
                    for (int c = 0; c < 3; ++c) acc[c] = xd[c];
                    break;
                }
                const C2<double>* m = cf + lt * 16 * np + t * 16 + L.cl;
                row_product<HR, false>(acc, xd, false, [&](int l) { return m[l * np]; });
            }
            if (!(L.live && L.col(t) < N)) continue;
            const unsigned o = L.template off<SY>(t, N);
            if (Z != nullptr) {
                RowRaw<SY> zr;
                zr.load(rz, o, L.template cs<SY>(t, N));
                C2<typename SY::real> z[3];
                zr.get(z);
#pragma unroll
                for (int c = 0; c < 3; ++c) {
                    acc[c].re += (double)z[c].re;
                    acc[c].im += (double)z[c].im;
                }
            }
            row_store<SY, double>(Y, o, L.template cs<SY>(t, N), acc);
        }
    }
}

// per-column sums of |V|^2 over each workgroup's rows (FP64): partials[b * N + j].  As many
// threads as a workgroup holds: the partials, and with them the workgroups, are a 256th of
// the sites.
constexpr int NORM_THREADS = 1024;
__global__ void __launch_bounds__(NORM_THREADS)
k_colnorm2_rows(const double2* __restrict__ V, int N, int cp, long rows, double* __restrict__ partials) {
    __shared__ double red[NORM_THREADS / 64][64];
    const int j = threadIdx.x & (cp - 1), rpw = NORM_THREADS / cp;
    double s = 0.0;
    if (j < N)
        for (long r = (long)blockIdx.x * rpw + threadIdx.x / cp; r < rows; r += (long)gridDim.x * rpw) {
            const double2 v = V[r * N + j];
            s += v.x * v.x + v.y * v.y;
        }
    for (int off = 32; off >= cp; off >>= 1) s += __shfl_xor(s, off, 64);  // cp: a power of two up to 64
    red[threadIdx.x >> 6][threadIdx.x & 63] = s;
    __syncthreads();
    if (threadIdx.x < cp && j < N) {
        double t = 0.0;
        for (int w = 0; w < NORM_THREADS / 64; ++w) t += red[w][j];
        partials[(long)blockIdx.x * N + j] = t;
    }
}

// ---------------------------------------------------------------------------------------------
// Launchers
// ---------------------------------------------------------------------------------------------
// the last of several tiles has at most 8 columns (row_product)
static bool last_tile_8(int N) { return N > 16 && (N - 1) % 16 < 8; }

static int gram_nw(int N) { return row_gram_nw(N <= 8 ? 1 : (N + 15) / 16); }
int gram_rows_parts(int N, int Vh, const RowOrder& o) { return row_grid(row_blocks(N, Vh), o, GRAM_BLOCKS, gram_nw(N)); }

template <typename S, bool SAME>
static void gram_rows_go(const void* A, const void* B, int N, int Vh, const RowOrder& o, double2* part,
                         const int* halt, hipStream_t s) {
    const int nb = row_blocks(N, Vh), ld = row_ld(N);
    const int nw = gram_nw(N);
    const dim3 grid(row_grid(nb, o, GRAM_BLOCKS, nw)), blk(64 * nw);
    const size_t lds = (size_t)nw * 512 * sizeof(double);
#define GO(NT, HR) \
    hipLaunchKernelGGL((k_gram_rows<S, NT, HR, SAME>), grid, blk, lds, s, (const char*)A, (const char*)B, N, Vh, o, nb, ld, part, halt)
    if (N <= 8) GO(1, true);
    else if (N <= 16) GO(1, false);
    else if (N <= 32) GO(2, false);
    else if (N <= 48) GO(3, false);
    else GO(4, false);
#undef GO
}

hipError_t launch_gram_rows(Prec prec, const void* A, const void* B, int N, int Vh, const RowOrder& o, double2* part,
                            const int* halt, hipStream_t s) {
#define GO(S)                                                            \
    if (A == B) gram_rows_go<S, true>(A, B, N, Vh, o, part, halt, s);    \
    else gram_rows_go<S, false>(A, B, N, Vh, o, part, halt, s)
    switch (prec) {
        case Prec::FP64: GO(F64); break;
        case Prec::FP32: GO(F32); break;
        case Prec::FP16: GO(H16); break;
        case Prec::BF16: GO(B16); break;
        case Prec::FX16: GO(X16); break;
    }
#undef GO
    return hipGetLastError();
}

bool pass_a_rows_gram(int N) { return N <= 32; }

// bytes of a coefficient in the arithmetic of the passes
template <typename S> static size_t pass_coef_bytes(int N) {
    return N > 16 && N <= 32 ? sizeof(C2<typename PassReal<S, 2>::type>) : sizeof(C2<typename S::real>);
}

template <typename S>
static void pass_a_rows_go(void* Q, const void* AP, const double2* beta, int N, int Vh, const RowOrder& o,
                           double2* part, const int* halt, hipStream_t s) {
    const int nb = row_blocks(N, Vh), ld = row_ld(N);
    const dim3 grid(row_grid(nb, o, GRAM_BLOCKS)), blk(64 * ROW_NW);
    const int np = N <= 8 ? 8 : (N + 15) / 16 * 16;
    const size_t cf = (size_t)np * np * pass_coef_bytes<S>(N), red = ROW_NW * 512 * sizeof(double);
    const size_t lds = pass_a_rows_gram(N) && red > cf ? red : cf;
#define GO(NT, HR, T8, GR)                                                                                         \
    hipLaunchKernelGGL((k_pass_a_rows<S, NT, HR, T8, GR>), grid, blk, lds, s, (char*)Q, (const char*)AP, beta, N, \
                       Vh, o, nb, ld, part, halt)
#define GO8(NT, GR)                                 \
    do {                                            \
        if (last_tile_8(N)) GO(NT, false, true, GR); \
        else GO(NT, false, false, GR);              \
    } while (0)
    if (N <= 8) GO(1, true, false, true);
    else if (N <= 16) GO(1, false, false, true);
    else if (N <= 32) GO8(2, true);
    else if (N <= 48) GO8(3, false);
    else GO8(4, false);
#undef GO8
#undef GO
}

hipError_t launch_pass_a_rows(Prec prec, void* Q, const void* AP, const double2* beta, int N, int Vh,
                              const RowOrder& o, double2* part, const int* halt, hipStream_t s) {
    switch (prec) {
        case Prec::FP64: pass_a_rows_go<F64>(Q, AP, beta, N, Vh, o, part, halt, s); break;
        case Prec::FP32: pass_a_rows_go<F32>(Q, AP, beta, N, Vh, o, part, halt, s); break;
        case Prec::FP16: pass_a_rows_go<H16>(Q, AP, beta, N, Vh, o, part, halt, s); break;
        case Prec::BF16: pass_a_rows_go<B16>(Q, AP, beta, N, Vh, o, part, halt, s); break;
        case Prec::FX16: pass_a_rows_go<X16>(Q, AP, beta, N, Vh, o, part, halt, s); break;
    }
    return hipGetLastError();
}

template <typename S>
static size_t pass_b_rows_lds(int N) {
    const int tw = N <= 8 ? 8 : 16, nt = N <= 8 ? 1 : (N + 15) / 16;
    return (size_t)nt * nt * tw * tw * sizeof(C2<double>) + (size_t)nt * (nt + 1) * tw * tw * pass_coef_bytes<S>(N);
}

template <typename S>
static void pass_b_rows_go(double2* X, const void* Qt, const void* P, void* Qn, void* Pn, const double2* betaC,
                           const double2* Sinv, const double2* SH, int N, int Vh, const RowOrder& o,
                           const SolveState* st, hipStream_t s) {
    const int nb = row_blocks(N, Vh);
    const size_t lds = pass_b_rows_lds<S>(N);
    const dim3 grid(row_grid(nb, o, 2048)), blk(64 * ROW_NW);
#define GO(NT, HR, T8)                                                                                         \
    hipLaunchKernelGGL((k_pass_b_rows<S, NT, HR, T8>), grid, blk, lds, s, X, (const char*)Qt, (const char*)P, \
                       (char*)Qn, (char*)Pn, betaC, Sinv, SH, N, Vh, o, nb, st)
#define GO8(NT)                                 \
    do {                                        \
        if (last_tile_8(N)) GO(NT, false, true); \
        else GO(NT, false, false);              \
    } while (0)
    if (N <= 8) GO(1, true, false);
    else if (N <= 16) GO(1, false, false);
    else if (N <= 32) GO8(2);
    else if (N <= 48) GO8(3);
    else GO8(4);
#undef GO8
#undef GO
}

hipError_t launch_pass_b_rows(Prec prec, double2* X, const void* Qt, const void* P, void* Qn, void* Pn,
                              const double2* betaC, const double2* Sinv, const double2* SH, int N, int Vh,
                              const RowOrder& o, const SolveState* st, hipStream_t s) {
    switch (prec) {
        case Prec::FP64: pass_b_rows_go<F64>(X, Qt, P, Qn, Pn, betaC, Sinv, SH, N, Vh, o, st, s); break;
        case Prec::FP32: pass_b_rows_go<F32>(X, Qt, P, Qn, Pn, betaC, Sinv, SH, N, Vh, o, st, s); break;
        case Prec::FP16: pass_b_rows_go<H16>(X, Qt, P, Qn, Pn, betaC, Sinv, SH, N, Vh, o, st, s); break;
        case Prec::BF16: pass_b_rows_go<B16>(X, Qt, P, Qn, Pn, betaC, Sinv, SH, N, Vh, o, st, s); break;
        case Prec::FX16: pass_b_rows_go<X16>(X, Qt, P, Qn, Pn, betaC, Sinv, SH, N, Vh, o, st, s); break;
    }
    return hipGetLastError();
}

template <typename SX, typename SY>
static void bmul_rows_go(const void* X, const void* Z, void* Y, const double2* M, int N, int Vh, const RowOrder& o,
                         const int* skip, hipStream_t s) {
    const int nb = row_blocks(N, Vh), np = N <= 8 ? 8 : (N + 15) / 16 * 16;
    const dim3 grid(row_grid(nb, o, 2048)), blk(64 * ROW_NW);
    const size_t lds = M != nullptr ? (size_t)np * np * sizeof(C2<double>) : 0;
    if (N <= 8)
        hipLaunchKernelGGL((k_bmul_rows<SX, SY, true>), grid, blk, lds, s, (const char*)X, (const char*)Z, (char*)Y, M,
                           N, Vh, o, nb, skip);
    else
        hipLaunchKernelGGL((k_bmul_rows<SX, SY, false>), grid, blk, lds, s, (const char*)X, (const char*)Z, (char*)Y, M,
                           N, Vh, o, nb, skip);
}

template <typename S>
static void bmul_rows_s(bool x64, bool y64, const void* X, const void* Z, void* Y, const double2* M, int N, int Vh,
                        const RowOrder& o, const int* skip, hipStream_t s) {
    if (x64) bmul_rows_go<F64, S>(X, Z, Y, M, N, Vh, o, skip, s);
    else if (y64) bmul_rows_go<S, F64>(X, Z, Y, M, N, Vh, o, skip, s);
    else bmul_rows_go<S, S>(X, Z, Y, M, N, Vh, o, skip, s);
}

hipError_t launch_bmul_rows(Prec px, const void* X, Prec py, const void* Z, void* Y, const double2* M, int N, int Vh,
                            const RowOrder& o, const int* skip, hipStream_t s) {
    const bool x64 = px == Prec::FP64, y64 = py == Prec::FP64;
    if (!x64 && !y64 && px != py) return hipErrorInvalidValue;
    switch (x64 ? py : px) {
        case Prec::FP64: bmul_rows_go<F64, F64>(X, Z, Y, M, N, Vh, o, skip, s); break;
        case Prec::FP32: bmul_rows_s<F32>(x64, y64, X, Z, Y, M, N, Vh, o, skip, s); break;
        case Prec::FP16: bmul_rows_s<H16>(x64, y64, X, Z, Y, M, N, Vh, o, skip, s); break;
        case Prec::BF16: bmul_rows_s<B16>(x64, y64, X, Z, Y, M, N, Vh, o, skip, s); break;
        case Prec::FX16: bmul_rows_s<X16>(x64, y64, X, Z, Y, M, N, Vh, o, skip, s); break;
    }
    return hipGetLastError();
}

// partials as launch_colnorm2 (the same count, reduced by launch_colnorm_reduce)
hipError_t launch_colnorm2_rows(const double2* V, int N, int Vh, double* partials, hipStream_t s) {
    const int g = (Vh + 255) / 256;
    hipLaunchKernelGGL(k_colnorm2_rows, dim3(g < NORM_BLOCKS ? g : NORM_BLOCKS), dim3(NORM_THREADS), 0, s, V, N, pad_n(N),
                       3L * Vh, partials);
    return hipGetLastError();
}

// dynamic LDS above the default limit
template <typename S> static hipError_t rows_setup_s() {
    hipError_t e = hipSuccess;
    auto big = [&](const void* f, int N) {
        const hipError_t r = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, (int)pass_b_rows_lds<S>(N));
        if (e == hipSuccess) e = r;
    };
    big(reinterpret_cast<const void*>(&k_pass_b_rows<S, 3, false, false>), 48);
    big(reinterpret_cast<const void*>(&k_pass_b_rows<S, 3, false, true>), 48);
    big(reinterpret_cast<const void*>(&k_pass_b_rows<S, 4, false, false>), 64);
    big(reinterpret_cast<const void*>(&k_pass_b_rows<S, 4, false, true>), 64);
    return e;
}
hipError_t blas_rows_setup() {
    for (hipError_t e : {rows_setup_s<F64>(), rows_setup_s<F32>(), rows_setup_s<H16>(), rows_setup_s<B16>(),
                         rows_setup_s<X16>()})
        if (e != hipSuccess) return e;
    return hipSuccess;
}

}  // namespace bcg
