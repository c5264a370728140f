// Link force: the gradient of the solve's loss with respect to the fat and long
// links (the backward of X = A^{-1} B; derived from dA = -(dD_eo D_oe + D_eo dD_oe)
// and D_eo^H = -D_oe).  For a link W_mu(x) of hop length k, y = x + k mu:
//   x even: grad = +eta_mu(x) sum_i [ Lam_i(x) Y_X,i(y)^H + X_i(x) Y_L,i(y)^H ]
//   x odd : grad = -eta_mu(x) sum_i [ Y_X,i(x) Lam_i(y)^H + Y_L,i(x) X_i(y)^H ]
// with Y_X = D_oe X, Y_L = D_oe Lam on the odd sites; output in the canonical
// [4][V][3][3] layout.
//
// k_link_force_rows (row layout): a wave takes 4 sites x 16
// columns per tile (half rows: 8 x 8), keeps the two vectors of its sites in registers
// for all directions, and sums the outer products of a lane's columns there; the lanes
// of a site meet through LDS, 16 bytes per entry and lane, and store a link's nine
// entries as one run.  k_link_force (plane layout): one thread per (site, direction).
#include "internal.h"
#include "rows.h"

namespace bcg {

__global__ void __launch_bounds__(256)
k_link_force(const double2* __restrict__ X, const double2* __restrict__ Lam,
             const double2* __restrict__ YX, const double2* __restrict__ YL, int N, Geom g,
             int improved, double2* __restrict__ gfat, double2* __restrict__ glong) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    const int mu = blockIdx.y;
    const int p = blockIdx.z;
    if (i >= g.Vh) return;
    int x[4];
    site_coords(g, i, p, x);
    const long Vh = g.Vh;
    const long V = 2 * Vh;
    const long lex = x[0] + (long)g.L[0] * (x[1] + (long)g.L[1] * (x[2] + (long)g.L[2] * x[3]));
    // fields at x (parity p) and at y (parity 1-p)
    const double2* U1 = p == 0 ? Lam : YX;
    const double2* U2 = p == 0 ? X : YL;
    const double2* V1 = p == 0 ? YX : Lam;
    const double2* V2 = p == 0 ? YL : X;
    const double s = (double)eta_sign(x, mu) * (p == 0 ? 1.0 : -1.0);
    for (int k = 1; k <= (improved ? 3 : 1); k += 2) {
        const int y = neighbour_cb(g, x, mu, k);
        C2<double> acc[9];
#pragma unroll
        for (int e = 0; e < 9; ++e) acc[e] = C2<double>{0.0, 0.0};
        for (int r = 0; r < N; ++r) {
            C2<double> u1[3], u2[3], v1[3], v2[3];
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                const long ox = ((long)r * 3 + c) * Vh + i, oy = ((long)r * 3 + c) * Vh + y;
                u1[c] = ld(U1 + ox);
                u2[c] = ld(U2 + ox);
                v1[c] = ld(V1 + oy);
                v2[c] = ld(V2 + oy);
            }
#pragma unroll
            for (int a = 0; a < 3; ++a)
#pragma unroll
                for (int b = 0; b < 3; ++b) {
                    // u v^H: (a, b) = u_a conj(v_b) = conj(v_b) u_a
                    cmac_conj(acc[3 * a + b], v1[b], u1[a]);
                    cmac_conj(acc[3 * a + b], v2[b], u2[a]);
                }
        }
        double2* out = (k == 1 ? gfat : glong) + ((long)mu * V + lex) * 9;
#pragma unroll
        for (int e = 0; e < 9; ++e) out[e] = make_double2(s * acc[e].re, s * acc[e].im);
    }
}

template <int ND, int NT, bool HR>
__global__ void __launch_bounds__(256)
k_link_force_rows(const char* __restrict__ X, const char* __restrict__ Lam, const char* __restrict__ YX,
                  const char* __restrict__ YL, int N, Geom g, RowOrder ord, double2* __restrict__ gfat,
                  double2* __restrict__ glong) {
    constexpr int SPB = row_block_sites<HR>(), SPR = HR ? 2 : 1, LPS = 16 / SPR;  // sites per row, lanes per site
    __shared__ C2<double> part[4][64 * 9];
    const int lane = threadIdx.x & 63;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int p = blockIdx.y;
    const int i_w = row_block(blockIdx.x, ord) * SPB + w * (SPB / 4);
    if (i_w >= g.Vh) return;
    const int i0 = i_w + row_lane_site<HR>(lane);
    const int i = i0 < g.Vh ? i0 : g.Vh - 1;
    int x[4];
    site_coords(g, i, p, x);
    const int st[4] = {1, g.L[0], g.L[0] * g.L[1], g.L[0] * g.L[1] * g.L[2]};
    const int lex = x[0] + st[1] * x[1] + st[2] * x[2] + st[3] * x[3];
    // fields at x (parity p) and at y (parity 1 - p)
    const rsrc_t ru1 = make_rsrc(p == 0 ? Lam : YX), ru2 = make_rsrc(p == 0 ? X : YL);
    const rsrc_t rv1 = make_rsrc(p == 0 ? YX : Lam), rv2 = make_rsrc(p == 0 ? YL : X);
    const unsigned cs = row_cs<F64>(N, 0), ss = row_ss<F64>(N);
    unsigned co[NT];
    C2<double> u1[NT][3], u2[NT][3];
    const bool last = (NT - 1) * 16 + row_lane_col<HR>(lane) < N;  // a column of the last tile
    auto keep = [&](C2<double>& z) { z = C2<double>{last ? z.re : 0.0, last ? z.im : 0.0}; };
#pragma unroll
    for (int t = 0; t < NT; ++t) {
        const int c = t * 16 + row_lane_col<HR>(lane);
        co[t] = (unsigned)(c < N ? c : N - 1) * 16u;
        RowRaw<F64> a, b;
        a.load(ru1, (unsigned)i * ss + co[t], cs);
        b.load(ru2, (unsigned)i * ss + co[t], cs);
#pragma unroll
        for (int q = 0; q < 3; ++q) {
            u1[t][q] = a.v[q];
            u2[t][q] = b.v[q];
            if (t == NT - 1) keep(u1[t][q]), keep(u2[t][q]);
        }
    }
    // step s: direction s / NT (mu = direction mod 4, hop 1 then 3), column tile s % NT
    auto fetch = [&](RowRaw<F64>& a, RowRaw<F64>& b, auto sc) {
        constexpr int dir = decltype(sc)::value / NT, t = decltype(sc)::value % NT;
        constexpr int mu = dir & 3, d = dir < 4 ? 1 : 3;
        const int L = g.L[mu], wrap = L * st[mu];
        int y = x[mu] + d, nbl = lex + d * st[mu];
        if (y >= L) { y -= L; nbl -= wrap; }
        if (d == 3 && y >= L) nbl -= wrap;
        const unsigned o = (unsigned)(nbl >> 1) * ss + co[t];
        a.load(rv1, o, cs);
        b.load(rv2, o, cs);
    };
    RowRaw<F64> v1[2], v2[2];
    fetch(v1[0], v2[0], std::integral_constant<int, 0>{});
    C2<double> acc[9];
    C2<double>* pw = part[w];
    static_for<ND * NT>([&](auto sc) {
        constexpr int s = decltype(sc)::value, dir = s / NT, t = s % NT;
        if constexpr (s + 1 < ND * NT) fetch(v1[(s + 1) & 1], v2[(s + 1) & 1], std::integral_constant<int, s + 1>{});
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (t == 0)
#pragma unroll
            for (int e = 0; e < 9; ++e) acc[e] = C2<double>{0.0, 0.0};
        if constexpr (t == NT - 1)  // lanes past the last column add nothing
#pragma unroll
            for (int b = 0; b < 3; ++b) keep(v1[s & 1].v[b]), keep(v2[s & 1].v[b]);
#pragma unroll
        for (int a = 0; a < 3; ++a)
#pragma unroll
            for (int b = 0; b < 3; ++b) {
                // u v^H: (a, b) = u_a conj(v_b) = conj(v_b) u_a
                cmac_conj(acc[3 * a + b], v1[s & 1].v[b], u1[t][a]);
                cmac_conj(acc[3 * a + b], v2[s & 1].v[b], u2[t][a]);
            }
        if constexpr (t == NT - 1) {
#pragma unroll
            for (int e = 0; e < 9; ++e) pw[lane * 9 + e] = acc[e];
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
            constexpr int mu = dir & 3;
            double2* out = dir < 4 ? gfat : glong;
#pragma unroll
            for (int q0 = 0; q0 < 9 * SPR; q0 += 16) {
                const int q = q0 + (lane & 15);
                if (q < 9 * SPR) {
                    const int sr = q / 9, e = q - 9 * sr;  // site of the row, entry
                    const int site = i_w + (lane >> 4) * SPR + sr;
                    const int l0 = (lane & 48) + sr * LPS;
                    C2<double> r{0.0, 0.0};
#pragma unroll
                    for (int n = 0; n < LPS; ++n) {
                        const C2<double> v = pw[(l0 + n) * 9 + e];
                        r.re += v.re;
                        r.im += v.im;
                    }
                    if (site < g.Vh) {
                        int xs[4];
                        site_coords(g, site, p, xs);
                        const long ls = xs[0] + (long)st[1] * xs[1] + (long)st[2] * xs[2] + (long)st[3] * xs[3];
                        const double sg = (double)eta_sign(xs, mu) * (p == 0 ? 1.0 : -1.0);
                        typedef double pair_t __attribute__((ext_vector_type(2)));
                        const pair_t v{sg * r.re, sg * r.im};
                        pair_t* o = reinterpret_cast<pair_t*>(out + ((long)mu * 2 * g.Vh + ls) * 9 + e);
                        // Half rows store 16 entries of two links, then the last two: parts of
                        // lines that L2 puts together unless they carry the streaming hint (us
                        // with / without: 16^4, N = 5 122 / 103, 16^3 x 32, N = 8 247 / 222; a
                        // whole row's, N = 16: 332 / 356)
                        if constexpr (HR) *o = v;
                        else __builtin_nontemporal_store(v, o);
                    }
                }
            }
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        }
    });
}

hipError_t launch_link_force_rows(const double2* X, const double2* Lam, const double2* YX, const double2* YL, int N,
                                  const Geom& g, const RowOrder& ord, int improved, double2* gfat, double2* glong,
                                  hipStream_t s) {
    if (!rows_fit(N, g.Vh)) return hipErrorInvalidValue;
    const int spb = N <= 8 ? 32 : 16;
    const dim3 grid((g.Vh + spb - 1) / spb, 2);
#define GO(ND, NT, HR)                                                                                              \
    hipLaunchKernelGGL((k_link_force_rows<ND, NT, HR>), grid, dim3(256), 0, s, (const char*)X, (const char*)Lam,    \
                       (const char*)YX, (const char*)YL, N, g, ord, gfat, glong)
#define GON(ND)                        \
    do {                               \
        if (N <= 8) GO(ND, 1, true);   \
        else if (N <= 16) GO(ND, 1, false); \
        else if (N <= 32) GO(ND, 2, false); \
        else if (N <= 48) GO(ND, 3, false); \
        else GO(ND, 4, false);         \
    } while (0)
    if (improved) GON(8);
    else GON(4);
#undef GON
#undef GO
    return hipGetLastError();
}

hipError_t launch_link_force(const double2* X, const double2* Lam, const double2* YX,
                             const double2* YL, int N, const Geom& g, int improved,
                             double2* gfat, double2* glong, hipStream_t s) {
    dim3 grid((g.Vh + 255) / 256, 4, 2);
    hipLaunchKernelGGL(k_link_force, grid, dim3(256), 0, s, X, Lam, YX, YL, N, g, improved, gfat, glong);
    return hipGetLastError();
}

}  // namespace bcg
