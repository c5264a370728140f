// Multi-right-hand-side staggered hop in the row layout (rows.h), for N > 4 columns.
//
// The hop is bound by what it moves: the 16 neighbour vectors of a site pass through
// L1 once each, and past L2 as often as the caches miss.  With lanes across columns a
// neighbour's 16 columns are one aligned run of 256 bytes (FP64), a wave holds 4 sites
// (not 64) so that the sites in flight on an XCD stay near each other, the folded
// links of a site are loaded once per 16 columns (9 loads of 16 lanes) and reach the
// columns through DPP row broadcasts, and the loads of the next D directions are kept
// in flight behind scheduling barriers (left to itself the compiler sinks each load to
// its use, for the occupancy, at 1.4 times the time in FP64).
#include <type_traits>
#include <utility>

#include "internal.h"
#include "rows.h"

namespace bcg {

// The folded link entries of a site as a row's lanes hold them: lane k matrix k.
template <typename S, int NL> struct RowLinks {
    C2<typename S::real> w[9];
    // base: links of the wave's first site (uniform), site: offset of the lane's site
    __device__ __forceinline__ void load(rsrc_t r, unsigned site, int lane) {
        const unsigned k = (unsigned)lane & (NL - 1);
        if constexpr (!S::scaled) {
            const unsigned o = site * (9u * NL * S::bytes) + k * S::bytes;
#pragma unroll
            for (int e = 0; e < 9; ++e) w[e] = buf_pair<AUX_NONE>(r, o, e * (NL * S::bytes), (typename S::real)0);
        } else {
            const unsigned o = site * (10u * NL * 4u) + k * 4u;
            unsigned u[10];
#pragma unroll
            for (int e = 0; e < 10; ++e) u[e] = __builtin_amdgcn_raw_buffer_load_b32(r, o, e * (NL * 4), AUX_NONE);
            const float s = __builtin_bit_cast(float, u[9]);
#pragma unroll
            for (int e = 0; e < 9; ++e)
                w[e] = C2<float>{S::dec((unsigned short)(u[e] & 0xffffu)) * s, S::dec((unsigned short)(u[e] >> 16)) * s};
        }
    }
};

template <int K, int BM, typename R>
__device__ __forceinline__ void row_matvec(C2<R> acc[3], const C2<R> w[9], const C2<R> v[3]) {
    mac3<K, BM>(acc, w[0], w[3], w[6], v[0]);
    mac3<K, BM>(acc, w[1], w[4], w[7], v[1]);
    mac3<K, BM>(acc, w[2], w[5], w[8], v[2]);
}

// The hop at one block of sites (four waves) and column tile ct: acc = D in, or with MASS
// acc = m2 * ctr - D in and z = ctr, at the lane's site and column.  D directions are in
// flight at a time.
template <typename S, int NL, bool MASS, bool HR, int D>
__device__ __forceinline__ void hop_rows_block(const char* __restrict__ W, const char* __restrict__ in,
                                               const char* __restrict__ ctr, double m2d, int N, const Geom& g,
                                               int out_parity, int sb, int w, int ct, int lane,
                                               C2<typename S::real> acc[3], C2<typename S::real> z[3], bool& stores,
                                               size_t& out_off) {
    using R = typename S::real;
    constexpr int SPB = row_block_sites<HR>(), SPW = SPB / 4;
    constexpr unsigned WB = S::scaled ? 40u * NL : 9u * NL * S::bytes;  // link bytes of a site
    const int i_w = sb * SPB + w * SPW;               // first site of the wave
    const int base = i_w < g.Vh ? i_w : g.Vh - 1;
    const int i0 = i_w + row_lane_site<HR>(lane);
    const bool live = i0 < g.Vh;
    const int i = live ? i0 : g.Vh - 1;               // spare lanes work on the last site and store nothing
    const int c0 = ct * 16 + row_lane_col<HR>(lane);
    stores = live && c0 < N;
    const int c = c0 < N ? c0 : N - 1;
    const rsrc_t wr = make_rsrc(W + (size_t)base * WB), vr = make_rsrc(in);
    const unsigned cs = row_cs<S>(N), ss = row_ss<S>(N), co = (unsigned)c * row_col_bytes<S>();
    RowLinks<S, NL> la, lb;
    if constexpr (HR) {
        const int p0 = base + (lane >> 4) * 2;         // the row's two sites
        la.load(wr, (unsigned)((p0 < g.Vh ? p0 : g.Vh - 1) - base), lane & 15);
        lb.load(wr, (unsigned)((p0 + 1 < g.Vh ? p0 + 1 : g.Vh - 1) - base), lane & 15);
    } else {
        la.load(wr, (unsigned)(i - base), lane & 15);
    }
    int x[4];
    site_coords(g, i, out_parity, x);
    const int st[4] = {1, g.L[0], g.L[0] * g.L[1], g.L[0] * g.L[1] * g.L[2]};
    const int lex = x[0] + st[1] * x[1] + st[2] * x[2] + st[3] * x[3];
    auto fetch = [&](RowRaw<S>& v, auto kc) {
        constexpr int k = decltype(kc)::value;
        constexpr int mu = hop_mu<NL>(k), d = hop_d<NL>(k);
        const int L = g.L[mu], wrap = L * st[mu];
        int y = x[mu] + d, nbl = lex + d * st[mu];
        if constexpr (d > 0) {
            if (y >= L) { y -= L; nbl -= wrap; }
            if (d == 3 && y >= L) nbl -= wrap;
        } else {
            if (y < 0) { y += L; nbl += wrap; }
            if (d == -3 && y < 0) nbl += wrap;
        }
        v.load(vr, (unsigned)(nbl >> 1) * ss + co, cs);
    };
    RowRaw<S> v[D];
    static_for<D>([&](auto k) { fetch(v[k.value], k); });
#pragma unroll
    for (int a = 0; a < 3; ++a) acc[a] = c2<R>(0, 0);
    static_for<NL>([&](auto kc) {
        constexpr int k = decltype(kc)::value;
        __builtin_amdgcn_sched_barrier(0);
        C2<R> u[3];
        v[k % D].get(u);
        if constexpr (HR) {
            row_matvec<k, 0x3>(acc, la.w, u);
            row_matvec<k, 0xc>(acc, lb.w, u);
        } else {
            row_matvec<k, 0xf>(acc, la.w, u);
        }
        if constexpr (k + D < NL) fetch(v[k % D], std::integral_constant<int, k + D>{});
    });
    out_off = (size_t)i * ss + co;
    if constexpr (MASS) {
        const R m2 = (R)m2d;
        RowRaw<S> zr;
        zr.load(make_rsrc(ctr), (unsigned)i * ss + co, cs);
        zr.get(z);
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            acc[a].re = m2 * z[a].re - acc[a].re;
            acc[a].im = m2 * z[a].im - acc[a].im;
        }
    }
}

// out = D in (MASS: m2 * ctr - D in) on one parity, at least WPS waves per SIMD.  Grid:
// (site blocks) x (tiles of 16 columns), the tiles of a block next to each other on one XCD.
template <typename S, int NL, bool MASS, bool HR, int D, int WPS>
__global__ void __launch_bounds__(256, WPS)
k_hop_rows(const char* __restrict__ W, const char* __restrict__ in, char* __restrict__ out,
           const char* __restrict__ ctr, double m2d, int N, int nct, Geom g, RowOrder ord, int out_parity,
           const int* __restrict__ halt) {
    using R = typename S::real;
    if (halt != nullptr && *halt) return;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    int sb, ct;
    if (ord.on) {
        const int q = blockIdx.x >> 3;
        ct = q % nct;
        sb = row_block((q / nct) * 8 + (blockIdx.x & 7), ord);
    } else {
        sb = blockIdx.x / nct;
        ct = blockIdx.x - sb * nct;
    }
    C2<R> acc[3], z[3];
    bool stores;
    size_t o;
    hop_rows_block<S, NL, MASS, HR, D>(W, in, ctr, m2d, N, g, out_parity, sb, w, ct, threadIdx.x & 63, acc, z, stores, o);
    if (stores) row_store<S, R>(out, o, row_cs<S>(N), acc);
}

// out = m2 * ctr - D in and the Gram partials of ctr^H out (as stored), N <= 16: a lane
// holds the two numbers of its (site, column) when it stores out, which is the operand
// layout of the matrix instruction, so the Gram costs neither a launch nor a second read
// of both blocks.  Persistent workgroups of NW waves over the site blocks.
template <typename S, int NL, bool HR, int D, int WPS, int NW>
__global__ void __launch_bounds__(64 * NW, WPS)
k_hop_gram_rows(const char* __restrict__ W, const char* __restrict__ in, char* __restrict__ out,
                const char* __restrict__ ctr, double m2d, int N, Geom g, RowOrder ord, int nb, int out_parity,
                double2* __restrict__ partials, const int* __restrict__ halt) {
    using R = typename S::real;
    __shared__ double red[NW * 512];
    if (halt != nullptr && *halt) return;
    const int lane = threadIdx.x & 63;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    RowGram<1, false> G;
    G.zero();
    int it = 0;
    for (int sb; (sb = row_turn(it, blockIdx.x, gridDim.x, NW / 4, w >> 2, nb, ord)) >= 0; ++it) {
        C2<R> acc[3], z[3];
        bool stores;
        size_t o;
        hop_rows_block<S, NL, true, HR, D>(W, in, ctr, m2d, N, g, out_parity, sb, w & 3, 0, lane, acc, z, stores, o);
        row_store_rt<S, R>(out, o, row_cs<S>(N), acc, stores);
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            const double zr = stores ? (double)z[c].re : 0.0, zi = stores ? (double)z[c].im : 0.0;
            const double ar = (double)acc[c].re, ai = (double)acc[c].im;
            G.add(&zr, &zi, &ar, &ai);
        }
    }
    constexpr int LD = HR ? 8 : 16;
    G.template finish<NW, HR>(red, partials + (long)blockIdx.x * LD * LD, LD);
}

// Row-layout FP64 links of one parity from the canonical ones: a row of lanes per
// site, lane k folded matrix k (as k_pack_links).
template <int NL>
__global__ void __launch_bounds__(256)
k_pack_links_rows(const double2* __restrict__ fat, const double2* __restrict__ lng, double2* __restrict__ W, Geom g,
                  int parity) {
    const long t = (long)blockIdx.x * 256 + threadIdx.x;
    const int i = (int)(t / NL), k = (int)(t % NL);
    if (i >= g.Vh) return;
    int x[4];
    site_coords(g, i, parity, x);
    const int mu = hop_mu<NL>(k), d = hop_d<NL>(k);
    const bool bwd = d < 0, three = d == 3 || d == -3;
    const double2* U = three ? lng : fat;
    int y[4] = {x[0], x[1], x[2], x[3]};
#pragma unroll
    for (int m = 0; m < 4; ++m)
        if (bwd && m == mu) {
            y[m] += d;
            while (y[m] < 0) y[m] += g.L[m];
        }
    const long lex = y[0] + (long)g.L[0] * (y[1] + (long)g.L[1] * (y[2] + (long)g.L[2] * y[3]));
    const double2* u = U + ((long)mu * 2 * g.Vh + lex) * 9;
    const double s = (double)eta_sign(x, mu) * (bwd ? -1.0 : 1.0);
    double2 e[9];
#pragma unroll
    for (int q = 0; q < 9; ++q) e[q] = u[q];
    double2* o = W + (long)i * 9 * NL + k;
#pragma unroll
    for (int a = 0; a < 3; ++a)
#pragma unroll
        for (int b = 0; b < 3; ++b) {
            const double2 v = bwd ? e[3 * b + a] : e[3 * a + b];
            o[(3 * a + b) * NL] = make_double2(s * v.x, bwd ? -s * v.y : s * v.y);
        }
}

// FP64 links [Vh][9][NL] -> the plane layout [NL][9][Vh], 16 sites of all 9 NL planes
// per workgroup through LDS (whole runs on both sides; entry q of site t at q * 17 + t)
__global__ void __launch_bounds__(256)
k_row_links_to_planes(const double2* __restrict__ src, double2* __restrict__ dst, int nl, long Vh) {
    extern __shared__ double2 tile[];  // [9 nl][17]
    const long s0 = (long)blockIdx.x * 16;
    const int ne = 9 * nl, ns = Vh - s0 < 16 ? (int)(Vh - s0) : 16;
    for (int e = threadIdx.x; e < ns * ne; e += 256) {
        const int t = e / ne, q = e - t * ne;
        tile[q * 17 + t] = src[s0 * ne + e];
    }
    __syncthreads();
    const int t = threadIdx.x & 15;
    if (t < ns)
        for (int r = threadIdx.x >> 4; r < ne; r += 16) {
            const int k = r / 9, e = r - 9 * k;
            dst[(long)r * Vh + s0 + t] = tile[(e * nl + k) * 17 + t];
        }
}

// row-layout links in another storage from the FP64 ones, one lane per (site, matrix)
template <typename S>
__global__ void __launch_bounds__(256)
k_row_links_from64(const double2* __restrict__ src, char* __restrict__ dst, long n, int nl) {
    const long t = (long)blockIdx.x * 256 + threadIdx.x;
    if (t >= n) return;
    const long i = t / nl;
    const int k = (int)(t - i * nl);
    const double2* s = src + i * 9 * nl + k;
    double2 e[9];
#pragma unroll
    for (int q = 0; q < 9; ++q) e[q] = s[(long)q * nl];
    if constexpr (!S::scaled) {
        typename S::pair* d = reinterpret_cast<typename S::pair*>(dst) + i * 9 * nl + k;
#pragma unroll
        for (int q = 0; q < 9; ++q) {
            typename S::pair p;
            p.x = (typename S::real)e[q].x;
            p.y = (typename S::real)e[q].y;
            d[(long)q * nl] = p;
        }
    } else {
        unsigned* d = reinterpret_cast<unsigned*>(dst) + i * 10 * nl + k;
        float m = 0.0f;
#pragma unroll
        for (int q = 0; q < 9; ++q) m = fmaxf(m, fmaxf(fabsf((float)e[q].x), fabsf((float)e[q].y)));
        const float inv = m > 0.0f ? 1.0f / m : 0.0f;
#pragma unroll
        for (int q = 0; q < 9; ++q) {
            const unsigned lo = S::enc((float)e[q].x * inv), hi = S::enc((float)e[q].y * inv);
            d[(long)q * nl] = lo | (hi << 16);
        }
        d[(long)9 * nl] = __builtin_bit_cast(unsigned, m);
    }
}

// ---------------------------------------------------------------------------------------------
hipError_t pack_links_rows(const void* fat, const void* lng, void* W, const Geom& g, int parity, int nl,
                           hipStream_t s) {
    const dim3 grid((unsigned)(((long)g.Vh * nl + 255) / 256));
    if (nl == 16)
        hipLaunchKernelGGL(k_pack_links_rows<16>, grid, dim3(256), 0, s, (const double2*)fat, (const double2*)lng,
                           (double2*)W, g, parity);
    else
        hipLaunchKernelGGL(k_pack_links_rows<8>, grid, dim3(256), 0, s, (const double2*)fat, (const double2*)lng,
                           (double2*)W, g, parity);
    return hipGetLastError();
}

hipError_t row_links_to_planes(const void* Wr, void* Wp, int nl, long Vh, hipStream_t s) {
    hipLaunchKernelGGL(k_row_links_to_planes, dim3((unsigned)((Vh + 15) / 16)), dim3(256), (size_t)9 * nl * 17 * 16, s,
                       (const double2*)Wr, (double2*)Wp, nl, Vh);
    return hipGetLastError();
}

hipError_t row_links_from64(Prec pd, const void* W64, void* Wd, int nl, long Vh, hipStream_t s) {
    const long n = Vh * nl;
    const dim3 grid((unsigned)((n + 255) / 256));
#define GO(S) hipLaunchKernelGGL(k_row_links_from64<S>, grid, dim3(256), 0, s, (const double2*)W64, (char*)Wd, n, nl)
    switch (pd) {
        case Prec::FP32: GO(F32); break;
        case Prec::FP16: GO(H16); break;
        case Prec::BF16: GO(B16); break;
        case Prec::FX16: GO(X16); break;
        default: return hipErrorInvalidValue;
    }
#undef GO
    return hipGetLastError();
}

bool rows_fit(int N, long Vh) {
    return N >= 2 && N <= MAXN && (N > 4 || Vh <= ROWS_SMALL_SITES) && (double)Vh * 3.0 * N * 16.0 < 4294967296.0;
}

RowOrder row_order(const Geom& g, int N) {
    RowOrder o{};
    const int spb = N <= 8 ? 32 : 16;
    const long plane = (long)g.L[0] * g.L[1] / 2;
    if (plane % spb) return o;
    const long bpp = plane / spb, nb = bpp * g.L[2] * g.L[3];
    if (nb % 8) return o;
    // cells of up to 4 x 8 (z, t) that divide the lattice and each XCD's eighth
    for (int bt : {8, 6, 4, 2, 1})
        for (int bz : {4, 2, 1}) {
            if (g.L[3] % bt || g.L[2] % bz || (nb / 8) % (bpp * bz * bt)) continue;
            o.on = 1;
            o.bpp = o.by = (int)bpp;
            o.bz = bz;
            o.bt = bt;
            o.lz = g.L[2];
            o.nb = (int)nb;
            return o;
        }
    return o;
}

template <typename S, int NL, bool MASS>
static void hop_rows_go(const void* W, const void* in, void* out, const void* ctr, double m2, int N, const Geom& g,
                        const RowOrder& ord, int out_parity, const int* halt, hipStream_t s) {
    constexpr bool F = std::is_same<S, F64>::value;
    const bool hr = N <= 8;
    const int nct = hr ? 1 : (N + 15) / 16;
    const long nb = (g.Vh + (hr ? 31 : 15)) / (hr ? 32 : 16);
    const dim3 grid((unsigned)(nb * nct));
#define GO(HRV, DV, WV)                                                                                          \
    BCG_TIMED_LAUNCH((k_hop_rows<S, NL, MASS, HRV, DV, WV>), grid, dim3(256), 0, s, (const char*)W, (const char*)in, \
                     (char*)out, (const char*)ctr, m2, N, nct, g, ord, out_parity, halt)
    if (hr) GO(true, F ? 4 : 8, F ? 3 : 4);
    else GO(false, F ? 4 : 8, 4);
#undef GO
}

constexpr int HOP_GRAM_NW = 8;
// The fused Gram saves a launch and a read of both blocks, but its persistent workgroups
// give up the overlap of one workgroup's start with another's end: 16^4, N = 16, FP64
// 39 + 11.6 us apart, 41.3 us fused (N = 8: 24.4 + 6.9, 28.6); at 32^3 x 64, N = 16,
// FP32 701 + 154 us apart and 825 to 909 us fused at any grid.
bool hop_rows_gram(int N, int Vh) { return N <= 16 && Vh <= 65536; }
int hop_gram_parts(int N, int Vh, const RowOrder& ord) {
    return row_grid(row_blocks(N, Vh), ord, GRAM_BLOCKS, HOP_GRAM_NW);
}

template <typename S, int NL>
static void hop_gram_rows_go(const void* W, const void* in, void* out, const void* ctr, double m2, int N,
                             const Geom& g, const RowOrder& ord, int out_parity, double2* partials, const int* halt,
                             hipStream_t s) {
    constexpr bool F = std::is_same<S, F64>::value;
    constexpr int NW = HOP_GRAM_NW;
    const int nb = row_blocks(N, g.Vh);
    const dim3 grid(hop_gram_parts(N, g.Vh, ord));
#define GO(HRV, DV, WV)                                                                                            \
    BCG_TIMED_LAUNCH((k_hop_gram_rows<S, NL, HRV, DV, WV, NW>), grid, dim3(64 * NW), 0, s, (const char*)W,         \
                     (const char*)in, (char*)out, (const char*)ctr, m2, N, g, ord, nb, out_parity, partials, halt)
    if (N <= 8) GO(true, F ? 2 : 8, F ? 2 : 4);
    else GO(false, F ? 2 : 8, 4);
#undef GO
}

hipError_t launch_hop_gram_rows(Prec prec, int nl, const void* W, const void* in, void* out, const void* ctr,
                                double m2, int N, const Geom& g, const RowOrder& ord, int out_parity,
                                double2* partials, const int* halt, hipStream_t s) {
    if (!rows_fit(N, g.Vh) || !hop_rows_gram(N, g.Vh) || ctr == nullptr) return hipErrorInvalidValue;
#define GO(S)                                                                                                       \
    do {                                                                                                            \
        if (nl == 16) hop_gram_rows_go<S, 16>(W, in, out, ctr, m2, N, g, ord, out_parity, partials, halt, s);       \
        else hop_gram_rows_go<S, 8>(W, in, out, ctr, m2, N, g, ord, out_parity, partials, halt, s);                 \
    } while (0)
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

hipError_t launch_hop_rows(Prec prec, int nl, const void* W, const void* in, void* out, const void* ctr, double m2,
                           int N, const Geom& g, const RowOrder& ord, int out_parity, const int* halt, hipStream_t s) {
    if (!rows_fit(N, g.Vh)) return hipErrorInvalidValue;
#define GO(S)                                                                                                   \
    do {                                                                                                        \
        if (nl == 16) {                                                                                         \
            if (ctr) hop_rows_go<S, 16, true>(W, in, out, ctr, m2, N, g, ord, out_parity, halt, s);             \
            else hop_rows_go<S, 16, false>(W, in, out, ctr, m2, N, g, ord, out_parity, halt, s);                \
        } else {                                                                                                \
            if (ctr) hop_rows_go<S, 8, true>(W, in, out, ctr, m2, N, g, ord, out_parity, halt, s);              \
            else hop_rows_go<S, 8, false>(W, in, out, ctr, m2, N, g, ord, out_parity, halt, s);                 \
        }                                                                                                       \
    } while (0)
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

}  // namespace bcg
