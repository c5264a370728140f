// Row layout of block vectors and links, and the wave mapping its kernels share.
//
// The three colours of a site hold their N columns next to each other:
//   vectors  FP64        [V/2][3][N] pairs
//            FP32        [V/2] of {[N] of {c0, c1}, [N] of c2}: 16 and 8 bytes a column
//            16-bit      [V/2][N] of {c0, c1, c2, scale}: the three packed colour
//                        pairs of a (site, column) and their FP32 scale in 16 bytes
//            (16 bytes to a lane where they can be: L1 answers four 128-byte runs of
//            8 bytes a lane in some 23 cycles, eight of 16 bytes in some 33; both FP32
//            hops at 32^3 x 64, N = 16: 1335 -> 1241 us)
//   links    FP64, FP32  [V/2][9][NL] pairs: entry e = 3 a + b of the NL folded
//                        matrices of a site side by side
//            16-bit      [V/2][10][NL] words: the nine packed entries, then the scale
//
// A row of 16 lanes takes one site and 16 of its columns (so a wave takes 4 sites),
// or, with at most 8 columns (half rows), two sites of 8 columns each.  Every load of
// a vector is then a contiguous, aligned run of columns whatever neighbour it belongs
// to, and a number that all columns of a site need (an entry of a folded matrix, or
// the value of another column in a product with an N x N matrix) sits in one lane of
// the row and reaches the others through the DPP row broadcast inside the multiply-add
// itself: it costs no load, no LDS access and no extra instruction.
#pragma once
#include <type_traits>
#include <utility>

#include "device_common.h"
#include "internal.h"
#include "storage.h"

namespace bcg {

// acc[i] += w_i(lane K of the row) * v for the three complex numbers w_i, on the lanes
// whose bank (group of four lanes of a row) is set in BM.  The leading s_nop covers
// the two wait states between a vector write of w and its use as a DPP operand.
#define BCG_MAC3(T, BM)                                                                     \
    asm("s_nop 1\n\t"                                                                       \
        "v_fmac_" T "_dpp %0, %6, %12 row_newbcast:%14 row_mask:0xf bank_mask:" BM "\n\t"   \
        "v_fmac_" T "_dpp %2, %8, %12 row_newbcast:%14 row_mask:0xf bank_mask:" BM "\n\t"   \
        "v_fmac_" T "_dpp %4, %10, %12 row_newbcast:%14 row_mask:0xf bank_mask:" BM "\n\t"  \
        "v_fmac_" T "_dpp %1, %6, %13 row_newbcast:%14 row_mask:0xf bank_mask:" BM "\n\t"   \
        "v_fmac_" T "_dpp %3, %8, %13 row_newbcast:%14 row_mask:0xf bank_mask:" BM "\n\t"   \
        "v_fmac_" T "_dpp %5, %10, %13 row_newbcast:%14 row_mask:0xf bank_mask:" BM "\n\t"  \
        "v_fmac_" T "_dpp %0, -%7, %13 row_newbcast:%14 row_mask:0xf bank_mask:" BM "\n\t"  \
        "v_fmac_" T "_dpp %2, -%9, %13 row_newbcast:%14 row_mask:0xf bank_mask:" BM "\n\t"  \
        "v_fmac_" T "_dpp %4, -%11, %13 row_newbcast:%14 row_mask:0xf bank_mask:" BM "\n\t" \
        "v_fmac_" T "_dpp %1, %7, %12 row_newbcast:%14 row_mask:0xf bank_mask:" BM "\n\t"   \
        "v_fmac_" T "_dpp %3, %9, %12 row_newbcast:%14 row_mask:0xf bank_mask:" BM "\n\t"   \
        "v_fmac_" T "_dpp %5, %11, %12 row_newbcast:%14 row_mask:0xf bank_mask:" BM         \
        : "+&v"(acc[0].re), "+&v"(acc[0].im), "+&v"(acc[1].re), "+&v"(acc[1].im), "+&v"(acc[2].re), "+&v"(acc[2].im) \
        : "v"(w0.re), "v"(w0.im), "v"(w1.re), "v"(w1.im), "v"(w2.re), "v"(w2.im), "v"(v.re), "v"(v.im), "n"(K))
template <int K, int BM>
__device__ __forceinline__ void mac3(C2<double> acc[3], C2<double> w0, C2<double> w1, C2<double> w2, C2<double> v) {
    if constexpr (BM == 0xf) BCG_MAC3("f64", "0xf");
    else if constexpr (BM == 0x3) BCG_MAC3("f64", "0x3");
    else BCG_MAC3("f64", "0xc");
}
template <int K, int BM>
__device__ __forceinline__ void mac3(C2<float> acc[3], C2<float> w0, C2<float> w1, C2<float> w2, C2<float> v) {
    if constexpr (BM == 0xf) BCG_MAC3("f32", "0xf");
    else if constexpr (BM == 0x3) BCG_MAC3("f32", "0x3");
    else BCG_MAC3("f32", "0xc");
}
#undef BCG_MAC3

// acc += W v for the 3 x 3 matrix W that lane K of the row holds, as one block of 36
// multiply-adds with one wait for all of them (24^4, N = 24, 16-bit, where the vector unit
// is busy throughout: with the cheaper neighbour offsets 307 -> 284 us for both hops)
#define BCG_MATVEC(T, BM)                                                                   \
    asm("s_nop 1\n\t"                                                                       \
        "v_fmac_" T "_dpp %0, %6, %24 row_newbcast:%30 row_mask:0xf bank_mask:" BM "\n\t" \
        "v_fmac_" T "_dpp %2, %12, %24 row_newbcast:%30 row_mask:0xf bank_mask:" BM "\n\t" \
        "v_fmac_" T "_dpp %4, %18, %24 row_newbcast:%30 row_mask:0xf bank_mask:" BM "\n\t" \
        "v_fmac_" T "_dpp %1, %6, %25 row_newbcast:%30 row_mask:0xf bank_mask:" BM "\n\t" \
        "v_fmac_" T "_dpp %3, %12, %25 row_newbcast:%30 row_mask:0xf bank_mask:" BM "\n\t" \
        "v_fmac_" T "_dpp %5, %18, %25 row_newbcast:%30 row_mask:0xf bank_mask:" BM "\n\t" \
        "v_fmac_" T "_dpp %0, -%7, %25 row_newbcast:%30 row_mask:0xf bank_mask:" BM "\n\t" \
        "v_fmac_" T "_dpp %2, -%13, %25 row_newbcast:%30 row_mask:0xf bank_mask:" BM "\n\t" \
        "v_fmac_" T "_dpp %4, -%19, %25 row_newbcast:%30 row_mask:0xf bank_mask:" BM "\n\t" \
        "v_fmac_" T "_dpp %1, %7, %24 row_newbcast:%30 row_mask:0xf bank_mask:" BM "\n\t" \
        "v_fmac_" T "_dpp %3, %13, %24 row_newbcast:%30 row_mask:0xf bank_mask:" BM "\n\t" \
        "v_fmac_" T "_dpp %5, %19, %24 row_newbcast:%30 row_mask:0xf bank_mask:" BM "\n\t" \
        "v_fmac_" T "_dpp %0, %8, %26 row_newbcast:%30 row_mask:0xf bank_mask:" BM "\n\t" \
        "v_fmac_" T "_dpp %2, %14, %26 row_newbcast:%30 row_mask:0xf bank_mask:" BM "\n\t" \
        "v_fmac_" T "_dpp %4, %20, %26 row_newbcast:%30 row_mask:0xf bank_mask:" BM "\n\t" \
        "v_fmac_" T "_dpp %1, %8, %27 row_newbcast:%30 row_mask:0xf bank_mask:" BM "\n\t" \
        "v_fmac_" T "_dpp %3, %14, %27 row_newbcast:%30 row_mask:0xf bank_mask:" BM "\n\t" \
        "v_fmac_" T "_dpp %5, %20, %27 row_newbcast:%30 row_mask:0xf bank_mask:" BM "\n\t" \
        "v_fmac_" T "_dpp %0, -%9, %27 row_newbcast:%30 row_mask:0xf bank_mask:" BM "\n\t" \
        "v_fmac_" T "_dpp %2, -%15, %27 row_newbcast:%30 row_mask:0xf bank_mask:" BM "\n\t" \
        "v_fmac_" T "_dpp %4, -%21, %27 row_newbcast:%30 row_mask:0xf bank_mask:" BM "\n\t" \
        "v_fmac_" T "_dpp %1, %9, %26 row_newbcast:%30 row_mask:0xf bank_mask:" BM "\n\t" \
        "v_fmac_" T "_dpp %3, %15, %26 row_newbcast:%30 row_mask:0xf bank_mask:" BM "\n\t" \
        "v_fmac_" T "_dpp %5, %21, %26 row_newbcast:%30 row_mask:0xf bank_mask:" BM "\n\t" \
        "v_fmac_" T "_dpp %0, %10, %28 row_newbcast:%30 row_mask:0xf bank_mask:" BM "\n\t" \
        "v_fmac_" T "_dpp %2, %16, %28 row_newbcast:%30 row_mask:0xf bank_mask:" BM "\n\t" \
        "v_fmac_" T "_dpp %4, %22, %28 row_newbcast:%30 row_mask:0xf bank_mask:" BM "\n\t" \
        "v_fmac_" T "_dpp %1, %10, %29 row_newbcast:%30 row_mask:0xf bank_mask:" BM "\n\t" \
        "v_fmac_" T "_dpp %3, %16, %29 row_newbcast:%30 row_mask:0xf bank_mask:" BM "\n\t" \
        "v_fmac_" T "_dpp %5, %22, %29 row_newbcast:%30 row_mask:0xf bank_mask:" BM "\n\t" \
        "v_fmac_" T "_dpp %0, -%11, %29 row_newbcast:%30 row_mask:0xf bank_mask:" BM "\n\t" \
        "v_fmac_" T "_dpp %2, -%17, %29 row_newbcast:%30 row_mask:0xf bank_mask:" BM "\n\t" \
        "v_fmac_" T "_dpp %4, -%23, %29 row_newbcast:%30 row_mask:0xf bank_mask:" BM "\n\t" \
        "v_fmac_" T "_dpp %1, %11, %28 row_newbcast:%30 row_mask:0xf bank_mask:" BM "\n\t" \
        "v_fmac_" T "_dpp %3, %17, %28 row_newbcast:%30 row_mask:0xf bank_mask:" BM "\n\t" \
        "v_fmac_" T "_dpp %5, %23, %28 row_newbcast:%30 row_mask:0xf bank_mask:" BM \
        : "+&v"(acc[0].re), "+&v"(acc[0].im), "+&v"(acc[1].re), "+&v"(acc[1].im), "+&v"(acc[2].re), "+&v"(acc[2].im) \
        : "v"(w[0].re), "v"(w[0].im), "v"(w[1].re), "v"(w[1].im), "v"(w[2].re), "v"(w[2].im), "v"(w[3].re), "v"(w[3].im), "v"(w[4].re), "v"(w[4].im), "v"(w[5].re), "v"(w[5].im), "v"(w[6].re), "v"(w[6].im), "v"(w[7].re), "v"(w[7].im), "v"(w[8].re), "v"(w[8].im), \
          "v"(v[0].re), "v"(v[0].im), "v"(v[1].re), "v"(v[1].im), "v"(v[2].re), "v"(v[2].im), "n"(K))
template <int K, int BM, typename R>
__device__ __forceinline__ void row_matvec(C2<R> acc[3], const C2<R> w[9], const C2<R> v[3]) {
    if constexpr (std::is_same<R, double>::value) {
        if constexpr (BM == 0xf) BCG_MATVEC("f64", "0xf");
        else if constexpr (BM == 0x3) BCG_MATVEC("f64", "0x3");
        else BCG_MATVEC("f64", "0xc");
    } else {
        if constexpr (BM == 0xf) BCG_MATVEC("f32", "0xf");
        else if constexpr (BM == 0x3) BCG_MATVEC("f32", "0x3");
        else BCG_MATVEC("f32", "0xc");
    }
}
#undef BCG_MATVEC

// f(integral_constant<int, 0>), ..., f(integral_constant<int, M - 1>)
template <int... I, typename F> __device__ __forceinline__ void static_for_(std::integer_sequence<int, I...>, F&& f) {
    (f(std::integral_constant<int, I>{}), ...);
}
template <int M, typename F> __device__ __forceinline__ void static_for(F&& f) {
    static_for_(std::make_integer_sequence<int, M>{}, f);
}

// The three colours of one (site, column): as loaded, and decoded to the arithmetic
// type.  off: byte offset of (site, column), cs: bytes from there to the next colour
// (FP64) or to the third (FP32), see row_cs.
template <typename S> struct RowRaw {
    C2<typename S::real> v[3];
    template <int AUX = AUX_NONE> __device__ __forceinline__ void load(rsrc_t r, unsigned off, unsigned cs) {
#pragma unroll
        for (int c = 0; c < 3; ++c) v[c] = buf_pair<AUX>(r, off, c * cs, (typename S::real)0);
    }
    __device__ __forceinline__ void get(C2<typename S::real> o[3]) const {
#pragma unroll
        for (int c = 0; c < 3; ++c) o[c] = v[c];
    }
};
// 16-bit components: stored number x group scale, with the unit 1 / 32767 of the fixed-point
// format taken into the scale (one product per component instead of two)
template <typename S> __device__ __forceinline__ float row_dec(unsigned short u) {
    if constexpr (std::is_same<S, X16>::value) return (float)(short)u;
    else return S::dec(u);
}
template <typename S> __device__ __forceinline__ float row_scale(float s) {
    return std::is_same<S, X16>::value ? s * (1.0f / 32767.0f) : s;
}
template <typename S> struct RowRaw16 {
    uint4 u;
    __device__ __forceinline__ void load(rsrc_t r, unsigned off, unsigned) {
        u = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, AUX_NONE));
    }
    __device__ __forceinline__ void get(C2<float> o[3]) const {
        const float s = row_scale<S>(__builtin_bit_cast(float, u.w));
        const unsigned p[3] = {u.x, u.y, u.z};
#pragma unroll
        for (int c = 0; c < 3; ++c)
            o[c] = C2<float>{row_dec<S>((unsigned short)(p[c] & 0xffffu)) * s, row_dec<S>((unsigned short)(p[c] >> 16)) * s};
    }
};
struct __attribute__((packed, aligned(8))) RowPair32 { float a, b, c, d; };  // {c0, c1} of a column
template <> struct RowRaw<F32> {
    C2<float> v[3];
    __device__ __forceinline__ void load(rsrc_t r, unsigned off, unsigned cs) {
        const float4 p = __builtin_bit_cast(float4, __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, AUX_NONE));
        v[0] = C2<float>{p.x, p.y};
        v[1] = C2<float>{p.z, p.w};
        v[2] = buf_pair<AUX_NONE>(r, off + cs, 0, 0.0f);
    }
    __device__ __forceinline__ void get(C2<float> o[3]) const {
#pragma unroll
        for (int c = 0; c < 3; ++c) o[c] = v[c];
    }
};
template <> struct RowRaw<H16> : RowRaw16<H16> {};
template <> struct RowRaw<B16> : RowRaw16<B16> {};
template <> struct RowRaw<X16> : RowRaw16<X16> {};

// bytes between the columns of a site, from column c's entry to its next colour (FP32: its
// third), and between sites
template <typename S> __device__ __forceinline__ constexpr unsigned row_col_bytes() { return 16u; }
template <typename S> __device__ __forceinline__ unsigned row_cs(int N, int c) {
    if constexpr (S::scaled) return 0u;
    else if constexpr (S::bytes == 8) return 16u * (unsigned)N - 8u * (unsigned)c;
    else return 16u * (unsigned)N;
}
template <typename S> __device__ __forceinline__ unsigned row_ss(int N) { return (S::scaled ? 16u : 3u * S::bytes) * (unsigned)N; }

// Store the three colours of a (site, column) in storage S if `st`; v becomes the
// values as stored, so that a fused product sees what later kernels will load.
template <typename S, typename R>
__device__ __forceinline__ void row_store_rt(void* base, size_t off, unsigned cs, C2<R> v[3], bool st) {
    char* p = reinterpret_cast<char*>(base) + off;
    if constexpr (!S::scaled) {
        typename S::pair w[3];
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            w[c].x = (typename S::real)v[c].re;
            w[c].y = (typename S::real)v[c].im;
            v[c] = C2<R>{(R)w[c].x, (R)w[c].y};
        }
        if constexpr (S::bytes == 8) {
            if (st) {
                *reinterpret_cast<RowPair32*>(p) = RowPair32{w[0].x, w[0].y, w[1].x, w[1].y};
                *reinterpret_cast<float2*>(p + cs) = w[2];
            }
        } else if (st) {
#pragma unroll
            for (int c = 0; c < 3; ++c) *reinterpret_cast<typename S::pair*>(p + c * cs) = w[c];
        }
    } else {
        float m = 0.0f;
#pragma unroll
        for (int c = 0; c < 3; ++c) m = fmaxf(m, fmaxf(fabsf((float)v[c].re), fabsf((float)v[c].im)));
        const float inv = m > 0.0f ? 1.0f / m : 0.0f;
        unsigned u[3];
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            const unsigned short lo = S::enc((float)v[c].re * inv), hi = S::enc((float)v[c].im * inv);
            u[c] = (unsigned)lo | ((unsigned)hi << 16);
            v[c] = C2<R>{(R)(row_dec<S>(lo) * row_scale<S>(m)), (R)(row_dec<S>(hi) * row_scale<S>(m))};
        }
        if (st) *reinterpret_cast<uint4*>(p) = make_uint4(u[0], u[1], u[2], __builtin_bit_cast(unsigned, m));
    }
}
template <typename S, typename R>
__device__ __forceinline__ void row_store(void* base, size_t off, unsigned cs, const C2<R> v[3]) {
    C2<R> w[3] = {v[0], v[1], v[2]};
    row_store_rt<S, R>(base, off, cs, w, true);
}

// FP64 with a streaming hint
__device__ __forceinline__ void row_store_nt(void* base, size_t off, unsigned cs, const C2<double> v[3]) {
    typedef double pair_t __attribute__((ext_vector_type(2)));
    char* p = reinterpret_cast<char*>(base) + off;
#pragma unroll
    for (int c = 0; c < 3; ++c) __builtin_nontemporal_store(pair_t{v[c].re, v[c].im}, reinterpret_cast<pair_t*>(p + c * cs));
}

// Site of a lane: blocks of 16 sites (half rows: 32), four waves of 4 (8) sites.
template <bool HR> __device__ __forceinline__ constexpr int row_block_sites() { return HR ? 32 : 16; }
template <bool HR> __device__ __forceinline__ int row_lane_site(int lane) { return HR ? lane >> 3 : lane >> 4; }
template <bool HR> __device__ __forceinline__ int row_lane_col(int lane) { return HR ? lane & 7 : lane & 15; }

// Site block of workgroup (or task) b of nb.  Workgroup b runs on XCD b mod 8; with an
// order given, XCD x takes the x-th eighth of a walk through four-dimensional cells of
// (planes of by blocks) x bz x bt, so that the sites one L2 serves at a time are near
// each other in all four directions.
__device__ __forceinline__ int row_block(int b, const RowOrder& o) {
    if (!o.on) return b;
    const int lin = (b & 7) * (o.nb >> 3) + (b >> 3);
    const int cell = o.by * o.bz * o.bt;
    const int k = lin / cell, r = lin - k * cell;
    const int ny = o.bpp / o.by, nz = o.lz / o.bz;
    const int y0 = k % ny, z0 = (k / ny) % nz, t0 = k / (ny * nz);
    const int y = r % o.by, z = (r / o.by) % o.bz, t = r / (o.by * o.bz);
    return (y0 * o.by + y) + o.bpp * ((z0 * o.bz + z) + o.lz * (t0 * o.bt + t));
}

typedef double dvec4 __attribute__((ext_vector_type(4)));

// Site block of turn `it` of wave quad `wb` (of NWB) of workgroup g (of G): with an
// order, the blocks of workgroup g's XCD.  -1 past the end.
__device__ __forceinline__ int row_turn(int it, int g, int G, int NWB, int wb, int nb, const RowOrder& o) {
    const int b = o.on ? ((it * (G >> 3) + (g >> 3)) * NWB + wb) * 8 + (g & 7) : (it * G + g) * NWB + wb;
    return b < nb ? row_block(b, o) : -1;
}

// Upper tiles of a Gram product A^H B (SAME: A = B), accumulated over sites.
template <int NT, bool SAME> struct RowGram {
    static constexpr int NUP = NT * (NT + 1) / 2;
    dvec4 re[NUP], im[NUP];
    __device__ __forceinline__ void zero() {
#pragma unroll
        for (int u = 0; u < NUP; ++u) re[u] = im[u] = dvec4{0.0, 0.0, 0.0, 0.0};
    }
    // one colour of four sites (half rows: eight), tile t in ar[t], ai[t] and br, bi
    __device__ __forceinline__ void add(const double* ar, const double* ai, const double* br, const double* bi) {
        int u = 0;
#pragma unroll
        for (int a = 0; a < NT; ++a)
#pragma unroll
            for (int b = a; b < NT; ++b, ++u) {
                re[u] = __builtin_amdgcn_mfma_f64_16x16x4f64(ar[a], br[b], re[u], 0, 0, 0);
                re[u] = __builtin_amdgcn_mfma_f64_16x16x4f64(ai[a], bi[b], re[u], 0, 0, 0);
                im[u] = __builtin_amdgcn_mfma_f64_16x16x4f64(ar[a], bi[b], im[u], 0, 0, 0);
                // A = B: the diagonal tile keeps M = Xr^T Xi, Im G = M - M^T at the end
                if (!(SAME && a == b)) im[u] = __builtin_amdgcn_mfma_f64_16x16x4f64(-ai[a], br[b], im[u], 0, 0, 0);
            }
    }
    // fixed-order sum of the workgroup's NW waves and the partial of this workgroup,
    // leading dimension ld; red: NW x 512 doubles of LDS.  Half rows: the two 8 x 8
    // diagonal blocks (the two sites of a row) are added.
    template <int NW, bool HR>
    __device__ __forceinline__ void finish(double* red, double2* __restrict__ out, int ld) {
        const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
        int u = 0;
#pragma unroll
        for (int a = 0; a < NT; ++a)
#pragma unroll
            for (int b = a; b < NT; ++b, ++u) {
                __syncthreads();
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int e = (4 * r + (lane >> 4)) * 16 + (lane & 15);
                    red[w * 512 + e] = re[u][r];
                    red[w * 512 + 256 + e] = im[u][r];
                }
                __syncthreads();
                if (threadIdx.x < 256) {
                    const int i = threadIdx.x >> 4, j = threadIdx.x & 15;
                    if (!HR || (i < 8 && j < 8)) {
                        double sr = 0.0, si = 0.0;
#pragma unroll
                        for (int h = 0; h < (HR ? 2 : 1); ++h) {
                            const int e = (i + 8 * h) * 16 + j + 8 * h, et = (j + 8 * h) * 16 + i + 8 * h;
                            for (int v = 0; v < NW; ++v) {
                                sr += red[v * 512 + e];
                                si += (SAME && a == b) ? red[v * 512 + 256 + e] - red[v * 512 + 256 + et]
                                                       : red[v * 512 + 256 + e];
                            }
                        }
                        const int gi = 16 * a + i, gj = 16 * b + j;
                        out[gi * ld + gj] = make_double2(sr, si);
                        if (a != b) out[gj * ld + gi] = make_double2(sr, -si);
                    }
                }
            }
    }
};

constexpr int ROW_NW = 8;  // waves per workgroup of the streaming kernels

// ---- host side ------------------------------------------------------------------------------
inline int row_blocks(int N, int Vh) { return N <= 8 ? (Vh + 31) / 32 : (Vh + 15) / 16; }

// workgroups: at most `most`, a multiple of 8 when the blocks are walked per XCD
inline int row_grid(int nb, const RowOrder& o, int most, int nw = ROW_NW) {
    const int nwb = nw / 4, g = (nb + nwb - 1) / nwb;
    if (!o.on) return g < most ? g : most;
    const int per = (nb / 8 + nwb - 1) / nwb;  // turns of one XCD
    return 8 * (per < most / 8 ? per : most / 8);
}


}  // namespace bcg
