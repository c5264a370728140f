// Multi-right-hand-side staggered hop in the row layout (rows.h).
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
template <typename S, int NL, bool NT> struct RowLinks {
    static constexpr int AUX = NT ? AUX_NT : AUX_NONE;
    C2<typename S::real> w[9];
    // base: links of the wave's first site (uniform), site: offset of the lane's site
    __device__ __forceinline__ void load(rsrc_t r, unsigned site, int lane) {
        const unsigned k = (unsigned)lane & (NL - 1);
        if constexpr (!S::scaled) {
            const unsigned o = site * (9u * NL * S::bytes) + k * S::bytes;
#pragma unroll
            for (int e = 0; e < 9; ++e) w[e] = buf_pair<AUX>(r, o, e * (NL * S::bytes), (typename S::real)0);
        } else {
            const unsigned o = site * (10u * NL * 4u) + k * 4u;
            unsigned u[10];
#pragma unroll
            for (int e = 0; e < 10; ++e) u[e] = __builtin_amdgcn_raw_buffer_load_b32(r, o, e * (NL * 4), AUX);
            const float s = row_scale<S>(__builtin_bit_cast(float, u[9]));
#pragma unroll
            for (int e = 0; e < 9; ++e)
                w[e] = C2<float>{row_dec<S>((unsigned short)(u[e] & 0xffffu)) * s, row_dec<S>((unsigned short)(u[e] >> 16)) * s};
        }
    }
};

// Directions at which the sum over them starts another chain.  The lengths, 2 3 3 4 4 (naive
// operator 1 1 2 2 2), give fewer roundings of large sums than four chains of NL / 4 added in
// pairs, the plane kernel's (error of A x against extended precision, FP64: one chain of 6 NL
// multiply-adds 3.8e-16, the lane-split plane kernel 1.9e-16, these 1.9e-16; FP32 storage
// 2.1e-7, 1.1e-7, 1.1e-7).  Two chains in the 16-bit formats, whose storage leaves 2.8e-5 and
// more whatever the chains: the vector unit is busy throughout there (24^4, N = 16, A x: two
// chains 302 us, six 328 us).
template <typename S, int NL> __host__ __device__ constexpr bool chain_start(int k) {
    if (S::scaled) return k == NL / 2;
    return NL == 16 ? (k == 2 || k == 5 || k == 8 || k == 12) : (k == 1 || k == 2 || k == 4 || k == 6);
}
template <typename S, int NL> __host__ __device__ constexpr int chain_second() {
    int k = 1;
    while (!chain_start<S, NL>(k)) ++k;
    return k;
}

// The hop at one block of sites (four waves) and the NT column tiles from column ct0 on:
// acc = D in, or with MASS acc = m2 * ctr - D in and z = ctr, at the lane's site and
// columns.  D directions are in flight at a time.  Two tiles share the links, the site's
// coordinates and the neighbour offsets (16^3 x 48, N = 32, FP32: 217 -> 185 us for both
// hops).
template <typename S, int NL, bool MASS, bool HR, int NT, int D, bool LNT>
__device__ __forceinline__ void hop_rows_block(const char* __restrict__ W, const char* __restrict__ in,
                                               const char* __restrict__ ctr, double m2d, int N, const Geom& g,
                                               int out_parity, int sb, int w, int ct0, int lane,
                                               C2<typename S::real> acc[NT][3], C2<typename S::real> z[NT][3],
                                               bool stores[NT], size_t out_off[NT], unsigned cs[NT]) {
    using R = typename S::real;
    constexpr int SPB = row_block_sites<HR>(), SPW = SPB / 4;
    constexpr unsigned WB = S::scaled ? 40u * NL : 9u * NL * S::bytes;  // link bytes of a site
    const int i_w = sb * SPB + w * SPW;               // first site of the wave
    const int base = i_w < g.Vh ? i_w : g.Vh - 1;
    const int i0 = i_w + row_lane_site<HR>(lane);
    const bool live = i0 < g.Vh;
    const int i = live ? i0 : g.Vh - 1;               // spare lanes work on the last site and store nothing
    const rsrc_t wr = make_rsrc(W + (size_t)base * WB), vr = make_rsrc(in);
    RowLinks<S, NL, LNT> la, lb;
    if constexpr (HR) {
        const int p0 = base + (lane >> 4) * 2;         // the row's two sites
        la.load(wr, (unsigned)((p0 < g.Vh ? p0 : g.Vh - 1) - base), lane & 15);
        lb.load(wr, (unsigned)((p0 + 1 < g.Vh ? p0 + 1 : g.Vh - 1) - base), lane & 15);
    } else {
        la.load(wr, (unsigned)(i - base), lane & 15);
    }
    int x[4];
    site_coords(g, i, out_parity, x);
    const unsigned ss = row_ss<S>(N);
    unsigned co[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t) {
        const int c0 = ct0 + 16 * t + row_lane_col<HR>(lane);
        const int c = c0 < N ? c0 : N - 1;
        stores[t] = live && c0 < N;
        co[t] = (unsigned)c * row_col_bytes<S>();
        cs[t] = row_cs<S>(N, c);
    }
    // Byte offset of a neighbour's first column: the site's own plus one of two uniform
    // steps, the second around the lattice.  Along x the neighbours' pair index depends on
    // whether x0 is odd.  (An extent of 2 takes the three-hop neighbour one hop away.)
    const unsigned own = (unsigned)i * ss, own_x = own + ((x[0] & 1) ? ss : 0u);
    const int half[4] = {0, g.L[0] / 2, g.L[0] / 2 * g.L[1], g.L[0] / 2 * g.L[1] * g.L[2]};
    auto fetch = [&](RowRaw<S> v[NT], auto kc) {
        constexpr int k = decltype(kc)::value;
        constexpr int mu = hop_mu<NL>(k), d0 = hop_d<NL>(k), sg = d0 > 0 ? 1 : -1;
        const int L = g.L[mu], d = (d0 == 3 || d0 == -3) && L == 2 ? sg : d0;
        const bool around = d0 > 0 ? x[mu] >= L - d : x[mu] < -d;
        unsigned o;
        if constexpr (mu == 0) {
            const int step = d > 0 ? (d - 1) / 2 : -((1 - d) / 2);
            o = own_x + (around ? (unsigned)(step - sg * (L / 2)) * ss : (unsigned)step * ss);
        } else {
            const unsigned step = (unsigned)(d * half[mu]) * ss, back = (unsigned)((d - sg * L) * half[mu]) * ss;
            o = own + (around ? back : step);
        }
#pragma unroll
        for (int t = 0; t < NT; ++t) v[t].load(vr, o + co[t], cs[t]);
    };
    RowRaw<S> v[D][NT];
    static_for<D>([&](auto k) { fetch(v[k.value], k); });
    // The sum over directions in chains (chain_start), added as they end
    C2<R> part[NT][3];
    static_for<NL>([&](auto kc) {
        constexpr int k = decltype(kc)::value;
        constexpr bool first = k < chain_second<S, NL>(), start = k == 0 || chain_start<S, NL>(k);
        C2<R>(*sum)[3] = first ? acc : part;
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            if constexpr (start)
#pragma unroll
                for (int a = 0; a < 3; ++a) sum[t][a] = c2<R>(0, 0);
            C2<R> u[3];
            v[k % D][t].get(u);
            if constexpr (HR) {
                row_matvec<k, 0x3>(sum[t], la.w, u);
                row_matvec<k, 0xc>(sum[t], lb.w, u);
            } else {
                row_matvec<k, 0xf>(sum[t], la.w, u);
            }
            if constexpr (!first && (k == NL - 1 || chain_start<S, NL>(k + 1)))
#pragma unroll
                for (int a = 0; a < 3; ++a) {
                    acc[t][a].re += part[t][a].re;
                    acc[t][a].im += part[t][a].im;
                    // here, not sunk into the branch of the store with `part` kept for it
                    asm volatile("" : "+v"(acc[t][a].re), "+v"(acc[t][a].im));
                }
        }
        if constexpr (k + D < NL) fetch(v[k % D], std::integral_constant<int, k + D>{});
    });
#pragma unroll
    for (int t = 0; t < NT; ++t) {
        out_off[t] = (size_t)i * ss + co[t];
        if constexpr (MASS) {
            const R m2 = (R)m2d;
            RowRaw<S> zr;
            zr.load(make_rsrc(ctr), (unsigned)i * ss + co[t], cs[t]);
            zr.get(z[t]);
#pragma unroll
            for (int a = 0; a < 3; ++a) {
                acc[t][a].re = m2 * z[t][a].re - acc[t][a].re;
                acc[t][a].im = m2 * z[t][a].im - acc[t][a].im;
            }
        }
    }
}

// out = D in (MASS: m2 * ctr - D in) on one parity, at least WPS waves per SIMD.  Grid:
// (site blocks) x (groups of NT tiles of 16 columns), the groups of a block next to each
// other on one XCD; a last group of one tile takes the one-tile code.
//
// ROWS_DOT: also Re ctr^H out of each column over the block's sites, to dots[block][N],
// while both are in registers (16^3 x 48, N = 24, FP64: the hop 167 -> 169 us, in place of a
// 39 us pass over both blocks).
//
// ROWS_CANON: out in the canonical layout [N][V/2][3], through LDS so that a column's
// sites of the block are one run (768 bytes), in place of a kernel that reads and writes
// the block once more (apply, us: 4^4, N = 4 14.5 -> 11-13, 16^4,
// N = 16 95 -> 86, 32^3 x 64, N = 12 2505 -> 2287).
enum { ROWS_PLAIN = 0, ROWS_DOT = 1, ROWS_CANON = 2 };
template <typename S, int NL, bool MASS, bool HR, int NT, int D, int WPS, bool LNT, int EPI>
__global__ void __launch_bounds__(256, WPS)
k_hop_rows(const char* __restrict__ W, const char* __restrict__ in, char* __restrict__ out,
           const char* __restrict__ ctr, double m2d, int N, int nct, Geom g, RowOrder ord, int out_parity,
           double* __restrict__ dots, const int* __restrict__ halt) {
    using R = typename S::real;
    constexpr int TW = HR ? 8 : 16, RW = 3 * row_block_sites<HR>();  // columns of a tile, numbers a column has
    __shared__ double red[EPI == ROWS_DOT ? 4 * NT * 16 : 1];
    __shared__ C2<R> tile[EPI == ROWS_CANON ? NT * TW * (RW + 1) : 1];
    if (halt != nullptr && *halt) return;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    // the tiles of a site block eight workgroups apart, on one XCD (an odd rest of blocks:
    // next to each other)
    const int nb = gridDim.x / nct, whole = (nb & ~7) * nct, q = blockIdx.x >> 3, rest = (int)blockIdx.x - whole;
    const int ct = rest < 0 ? q % nct : rest % nct;
    int sb = rest < 0 ? (q / nct) * 8 + (blockIdx.x & 7) : (nb & ~7) + rest / nct;
    if (ord.on) sb = row_block(sb, ord);
    auto tiles = [&](auto ntc) {
        constexpr int T = decltype(ntc)::value;
        C2<R> acc[T][3], z[T][3];
        bool stores[T];
        size_t o[T];
        unsigned cs[T];
        hop_rows_block<S, NL, MASS, HR, T, T == NT ? D : 2 * D, LNT>(W, in, ctr, m2d, N, g, out_parity, sb, w,
                                                                     16 * NT * ct, threadIdx.x & 63, acc, z, stores, o, cs);
#pragma unroll
        for (int t = 0; t < T; ++t)
            if (EPI != ROWS_CANON && stores[t]) row_store<S, R>(out, o[t], cs[t], acc[t]);
        const int lane = threadIdx.x & 63;
        if constexpr (EPI == ROWS_CANON) {
            const int r0 = 3 * (w * (row_block_sites<HR>() / 4) + row_lane_site<HR>(lane));
#pragma unroll
            for (int t = 0; t < T; ++t)
#pragma unroll
                for (int c = 0; c < 3; ++c) tile[(t * TW + row_lane_col<HR>(lane)) * (RW + 1) + r0 + c] = acc[t][c];
            __syncthreads();
            const long rows = 3L * g.Vh, b0 = (long)sb * RW;
            const int m = rows - b0 < RW ? (int)(rows - b0) : RW;
            C2<R>* dst = reinterpret_cast<C2<R>*>(out) + b0;
            for (int e = threadIdx.x; e < T * TW * RW; e += 256) {
                const int j = e / RW, r = e - RW * j, c = 16 * NT * ct + j;
                if (c < N && r < m) dst[(long)c * rows + r] = tile[j * (RW + 1) + r];
            }
        }
        if constexpr (EPI == ROWS_DOT) {
#pragma unroll
            for (int t = 0; t < T; ++t) {
                double d = 0.0;
#pragma unroll
                for (int c = 0; c < 3; ++c) d += (double)z[t][c].re * acc[t][c].re + (double)z[t][c].im * acc[t][c].im;
                if (!stores[t]) d = 0.0;
#pragma unroll
                for (int off = 32; off >= TW; off >>= 1) d += __shfl_xor(d, off, 64);
                if (lane < TW) red[(t * 4 + w) * 16 + lane] = d;
            }
            __syncthreads();
            const int t = threadIdx.x / TW, j = threadIdx.x % TW, c = 16 * (NT * ct + t) + j;
            if (t < T && c < N) {
                const double* r = red + t * 64 + j;
                dots[(long)sb * N + c] = (r[0] + r[16]) + (r[32] + r[48]);
            }
        }
    };
    if constexpr (NT == 2) {
        if (16 * NT * ct + 16 >= N) return tiles(std::integral_constant<int, 1>{});
    }
    tiles(std::integral_constant<int, NT>{});
}

// out = m2 * ctr - D in and the Gram partials of ctr^H out (as stored), N <= 16: a lane
// holds the two numbers of its (site, column) when it stores out, which is the operand
// layout of the matrix instruction, so the Gram costs neither a launch nor a second read
// of both blocks.  Persistent workgroups of NW waves over the site blocks.
template <typename S, int NL, bool HR, int D, int WPS, int NW, bool LNT>
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
        C2<R> acc[1][3], z[1][3];
        bool stores[1];
        size_t o[1];
        unsigned cs[1];
        hop_rows_block<S, NL, true, HR, 1, D, LNT>(W, in, ctr, m2d, N, g, out_parity, sb, w & 3, 0, lane, acc, z,
                                                     stores, o, cs);
        row_store_rt<S, R>(out, o[0], cs[0], acc[0], stores[0]);
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            const double zr = stores[0] ? (double)z[0][c].re : 0.0, zi = stores[0] ? (double)z[0][c].im : 0.0;
            const double ar = (double)acc[0][c].re, ai = (double)acc[0][c].im;
            G.add(&zr, &zi, &ar, &ai);
        }
    }
    constexpr int LD = HR ? 8 : 16;
    G.template finish<NW, HR>(red, partials + (long)blockIdx.x * LD * LD, LD);
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
    // Cells of up to 4 x 8 (z, t) that divide the lattice and each XCD's eighth, in y the
    // whole plane while a cell's vectors fit an XCD's 4 MB L2 at 16 FP64 columns, else 4
    // rows (both hops, us, whole planes / 4 rows: 16^4, N = 16, FP64 78.5 / 81.5, 16^3 x 48,
    // N = 32 416 / 425; 24^4, N = 24 597 / 590, 32^3 x 64, N = 16, FP64 2653 / 2547, FP32
    // 1217 / 1204)
    const int y4 = (int)((2L * g.L[0] + spb - 1) / spb);  // blocks of 4 rows
    for (int by : {bpp * spb > 256 ? y4 : (int)bpp, (int)bpp})
        for (int bt : {8, 6, 4, 2, 1})
            for (int bz : {4, 2, 1}) {
                if (bpp % by || g.L[3] % bt || g.L[2] % bz || (nb / 8) % ((long)by * bz * bt)) continue;
                o.on = 1;
                o.bpp = (int)bpp;
                o.by = by;
                o.bz = bz;
                o.bt = bt;
                o.lz = g.L[2];
                o.nb = (int)nb;
                return o;
            }
    return o;
}

// Links past the caches: with both parities' links beyond 200 MB (of 256 MB) no link stays
// in the Infinity Cache from one hop of a parity to the next, and streaming loads leave
// the room to the vectors (both hops, us, kept / streamed: 16^4, N = 16, FP64, 151 MB 69 /
// 73; 16^3 x 48, N = 32, FP32, 226 MB 191 / 179; 32^3 x 64, N = 16, FP32 1241 / 1198).
static bool stream_links(Prec p, int nl, long Vh) {
    return 2.0 * nl * Vh * (p == Prec::FP64 ? 144 : (p == Prec::FP32 ? 72 : 40)) > 200e6;
}

template <typename S, int NL, bool MASS, bool LNT>
static void hop_rows_go(const void* W, const void* in, void* out, const void* ctr, double m2, int N, const Geom& g,
                        const RowOrder& ord, int out_parity, double* dots, bool canon, const int* halt, hipStream_t s) {
    constexpr bool F = std::is_same<S, F64>::value;
    const long nb = row_blocks(N, g.Vh);
#define GO2(HRV, NTV, DV, WV, EPI)                                                                                   \
    do {                                                                                                             \
        const int nct = (N + 16 * NTV - 1) / (16 * NTV);                                                             \
        const dim3 grid((unsigned)(nb * nct));                                                                       \
        BCG_TIMED_LAUNCH((k_hop_rows<S, NL, MASS, HRV, NTV, DV, WV, LNT, EPI>), grid, dim3(256), 0, s,               \
                         (const char*)W, (const char*)in, (char*)out, (const char*)ctr, m2, N, nct, g, ord,          \
                         out_parity, dots, halt);                                                                    \
    } while (0)
#define GO(HRV, NTV, DV, WV)                                              \
    do {                                                                  \
        if constexpr (F) {                                                \
            if (canon) GO2(HRV, NTV, DV, WV, ROWS_CANON);                 \
            else if (MASS && dots) GO2(HRV, NTV, DV, WV, MASS ? ROWS_DOT : ROWS_PLAIN); \
            else GO2(HRV, NTV, DV, WV, ROWS_PLAIN);                       \
        } else {                                                          \
            GO2(HRV, NTV, DV, WV, ROWS_PLAIN);                            \
        }                                                                 \
    } while (0)
    // FP64 on more than one tile: two at a time with three directions in flight at two waves
    // per SIMD, but one at a time (four directions, three waves) where the third tile would be
    // left alone and up to 8192 sites, whose workgroups are few (an application, us, one /
    // two: 16^3 x 48, N = 40 654 / 768, N = 64 1152 / 963, N = 28 511 / 388, 24^4, N = 32 942 /
    // 794; 8^4, N = 24 20 / 25; two at three or four waves with two directions or one: 4 to 13 %
    // longer than these)
    const bool one = N <= 16 || (F && ((N > 32 && N <= 48) || g.Vh <= 8192));
    if (N <= 8) GO(true, 1, F ? 4 : 8, F ? 2 : 4);
    else if (one) GO(false, 1, F ? 4 : 8, F ? 3 : 4);
    else GO(false, 2, F ? 3 : 4, F ? 2 : 4);
#undef GO
#undef GO2
}

constexpr int HOP_GRAM_NW = 8;
bool hop_rows_gram(int N) { return N <= 16; }
// The fused Gram saves a launch and a read of both blocks (apart / fused, us: 16^4, N = 16,
// FP64 39 + 12 / 41, N = 8 24 + 7 / 29; 32^3 x 64, N = 16, FP32 619 + 157 / 671).  Whole
// rounds of the 512 workgroups that fit the chip, of 8 turns each or more: one round of many
// turns lets the workgroups of an XCD drift apart in the lattice (32^3 x 64: 738 us at 512
// workgroups, 705 at 2048, 671 at 4096), a part of a round leaves CUs idle at the end
// (24^4, N = 16, 16-bit, an iteration: 431 us apart, 428 at 1024, 442 at 1296).  Above 16
// columns the accumulators of three tiles spill (16^3 x 48, N = 32, FP32: 99 + 39 us apart,
// 138 to 182 fused; 24^4, N = 24, 16-bit 137 + 63 and 213).
int hop_gram_parts(int N, int Vh, const RowOrder& ord) {
    const int nb = row_blocks(N, Vh), rounds = nb / 16 / GRAM_BLOCKS;
    return row_grid(nb, ord, GRAM_BLOCKS * (rounds < 1 ? 1 : (rounds < 8 ? rounds : 8)), HOP_GRAM_NW);
}

template <typename S, int NL>
static void hop_gram_rows_go(const void* W, const void* in, void* out, const void* ctr, double m2, int N,
                             const Geom& g, const RowOrder& ord, int out_parity, double2* partials, bool lnt,
                             const int* halt, hipStream_t s) {
    constexpr bool F = std::is_same<S, F64>::value;
    constexpr int NW = HOP_GRAM_NW;
    const int nb = row_blocks(N, g.Vh);
    const dim3 grid(hop_gram_parts(N, g.Vh, ord));
#define GO2(HRV, DV, WV, LNT)                                                                                      \
    BCG_TIMED_LAUNCH((k_hop_gram_rows<S, NL, HRV, DV, WV, NW, LNT>), grid, dim3(64 * NW), 0, s, (const char*)W,    \
                     (const char*)in, (char*)out, (const char*)ctr, m2, N, g, ord, nb, out_parity, partials, halt)
#define GO(HRV, DV, WV)                     \
    do {                                    \
        if (lnt) GO2(HRV, DV, WV, true);    \
        else GO2(HRV, DV, WV, false);       \
    } while (0)
    if (N <= 8) GO(true, F ? 2 : 8, F ? 2 : 4);
    else GO(false, F ? 2 : 8, 4);
#undef GO
#undef GO2
}

hipError_t launch_hop_gram_rows(Prec prec, int nl, const void* W, const void* in, void* out, const void* ctr,
                                double m2, int N, const Geom& g, const RowOrder& ord, int out_parity,
                                double2* partials, const int* halt, hipStream_t s) {
    if (!rows_fit(N, g.Vh) || !hop_rows_gram(N) || ctr == nullptr) return hipErrorInvalidValue;
    const bool lnt = stream_links(prec, nl, g.Vh);
#define GO(S)                                                                                                       \
    do {                                                                                                            \
        if (nl == 16) hop_gram_rows_go<S, 16>(W, in, out, ctr, m2, N, g, ord, out_parity, partials, lnt, halt, s);  \
        else hop_gram_rows_go<S, 8>(W, in, out, ctr, m2, N, g, ord, out_parity, partials, lnt, halt, s);            \
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
                           int N, const Geom& g, const RowOrder& ord, int out_parity, const int* halt, hipStream_t s,
                           double* dots, bool canon) {
    if (!rows_fit(N, g.Vh) || (dots && (prec != Prec::FP64 || !ctr || canon)) || (canon && prec != Prec::FP64))
        return hipErrorInvalidValue;
    const bool lnt = stream_links(prec, nl, g.Vh);
#define GO3(S, NL, MASS)                                                                                  \
    do {                                                                                                  \
        if (lnt) hop_rows_go<S, NL, MASS, true>(W, in, out, ctr, m2, N, g, ord, out_parity, dots, canon, halt, s);  \
        else hop_rows_go<S, NL, MASS, false>(W, in, out, ctr, m2, N, g, ord, out_parity, dots, canon, halt, s);     \
    } while (0)
#define GO(S)                               \
    do {                                    \
        if (nl == 16) {                     \
            if (ctr) GO3(S, 16, true);      \
            else GO3(S, 16, false);         \
        } else {                            \
            if (ctr) GO3(S, 8, true);       \
            else GO3(S, 8, false);          \
        }                                   \
    } while (0)
    switch (prec) {
        case Prec::FP64: GO(F64); break;
        case Prec::FP32: GO(F32); break;
        case Prec::FP16: GO(H16); break;
        case Prec::BF16: GO(B16); break;
        case Prec::FX16: GO(X16); break;
    }
#undef GO3
#undef GO
    return hipGetLastError();
}

}  // namespace bcg
