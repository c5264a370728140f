// Register arithmetic on 16 x 16 complex matrices spread over a row of 16 lanes: lane j
// holds column j, register i row i, so that entry (i, K) reaches every lane of the row
// through the DPP row broadcast of lane K inside the multiply-add (v_fmac_f64_dpp,
// row_newbcast), without LDS, shuffles or barriers.  In a factorisation all four rows of a
// wave do the same, in a product each may hold rows of w of its own.
// Each block opens with the two wait states that a vector write of a DPP operand needs,
// and its outputs are early-clobber, as later lines still read the inputs.
#pragma once
#include <type_traits>
#include <utility>

#include "device_common.h"

namespace bcg {

// acc[r] += w[r](lane K) * v, r < 1
template <int K> __device__ __forceinline__ void row_mac1(C2<double>* acc, const C2<double>* w, C2<double> v) {
    asm("s_nop 1\n\t"
        "v_fmac_f64_dpp %0, %2, %4 row_newbcast:%6 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %1, %2, %5 row_newbcast:%6 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %0, -%3, %5 row_newbcast:%6 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %1, %3, %4 row_newbcast:%6 row_mask:0xf bank_mask:0xf"
        : "+&v"(acc[0].re), "+&v"(acc[0].im)
        : "v"(w[0].re), "v"(w[0].im), "v"(v.re), "v"(v.im), "n"(K));
}
// acc[r] += w[r](lane K) * v, r < 2
template <int K> __device__ __forceinline__ void row_mac2(C2<double>* acc, const C2<double>* w, C2<double> v) {
    asm("s_nop 1\n\t"
        "v_fmac_f64_dpp %0, %4, %8 row_newbcast:%10 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %2, %6, %8 row_newbcast:%10 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %1, %4, %9 row_newbcast:%10 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %3, %6, %9 row_newbcast:%10 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %0, -%5, %9 row_newbcast:%10 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %2, -%7, %9 row_newbcast:%10 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %1, %5, %8 row_newbcast:%10 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %3, %7, %8 row_newbcast:%10 row_mask:0xf bank_mask:0xf"
        : "+&v"(acc[0].re), "+&v"(acc[0].im), "+&v"(acc[1].re), "+&v"(acc[1].im)
        : "v"(w[0].re), "v"(w[0].im), "v"(w[1].re), "v"(w[1].im), "v"(v.re), "v"(v.im), "n"(K));
}
// acc[r] += w[r](lane K) * v, r < 3
template <int K> __device__ __forceinline__ void row_mac3(C2<double>* acc, const C2<double>* w, C2<double> v) {
    asm("s_nop 1\n\t"
        "v_fmac_f64_dpp %0, %6, %12 row_newbcast:%14 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %2, %8, %12 row_newbcast:%14 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %4, %10, %12 row_newbcast:%14 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %1, %6, %13 row_newbcast:%14 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %3, %8, %13 row_newbcast:%14 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %5, %10, %13 row_newbcast:%14 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %0, -%7, %13 row_newbcast:%14 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %2, -%9, %13 row_newbcast:%14 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %4, -%11, %13 row_newbcast:%14 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %1, %7, %12 row_newbcast:%14 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %3, %9, %12 row_newbcast:%14 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %5, %11, %12 row_newbcast:%14 row_mask:0xf bank_mask:0xf"
        : "+&v"(acc[0].re), "+&v"(acc[0].im), "+&v"(acc[1].re), "+&v"(acc[1].im), "+&v"(acc[2].re), "+&v"(acc[2].im)
        : "v"(w[0].re), "v"(w[0].im), "v"(w[1].re), "v"(w[1].im), "v"(w[2].re), "v"(w[2].im), "v"(v.re), "v"(v.im), "n"(K));
}
// acc[r] += w[r](lane K) * v, r < 4
template <int K> __device__ __forceinline__ void row_mac4(C2<double>* acc, const C2<double>* w, C2<double> v) {
    asm("s_nop 1\n\t"
        "v_fmac_f64_dpp %0, %8, %16 row_newbcast:%18 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %2, %10, %16 row_newbcast:%18 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %4, %12, %16 row_newbcast:%18 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %6, %14, %16 row_newbcast:%18 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %1, %8, %17 row_newbcast:%18 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %3, %10, %17 row_newbcast:%18 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %5, %12, %17 row_newbcast:%18 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %7, %14, %17 row_newbcast:%18 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %0, -%9, %17 row_newbcast:%18 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %2, -%11, %17 row_newbcast:%18 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %4, -%13, %17 row_newbcast:%18 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %6, -%15, %17 row_newbcast:%18 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %1, %9, %16 row_newbcast:%18 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %3, %11, %16 row_newbcast:%18 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %5, %13, %16 row_newbcast:%18 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %7, %15, %16 row_newbcast:%18 row_mask:0xf bank_mask:0xf"
        : "+&v"(acc[0].re), "+&v"(acc[0].im), "+&v"(acc[1].re), "+&v"(acc[1].im), "+&v"(acc[2].re), "+&v"(acc[2].im), "+&v"(acc[3].re), "+&v"(acc[3].im)
        : "v"(w[0].re), "v"(w[0].im), "v"(w[1].re), "v"(w[1].im), "v"(w[2].re), "v"(w[2].im), "v"(w[3].re), "v"(w[3].im), "v"(v.re), "v"(v.im), "n"(K));
}
// a[r] -= a[r](lane K) * m, r < 4.  m must be 0 on lane K, whose numbers then stay as they
// are; three instructions lie between a write of a number and its next broadcast.
template <int K> __device__ __forceinline__ void row_elim4(C2<double>* a, C2<double> m) {
    asm("s_nop 1\n\t"
        "v_fmac_f64_dpp %0, -%0, %8 row_newbcast:%10 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %2, -%2, %8 row_newbcast:%10 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %4, -%4, %8 row_newbcast:%10 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %6, -%6, %8 row_newbcast:%10 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %0, %1, %9 row_newbcast:%10 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %2, %3, %9 row_newbcast:%10 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %4, %5, %9 row_newbcast:%10 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %6, %7, %9 row_newbcast:%10 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %1, -%0, %9 row_newbcast:%10 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %3, -%2, %9 row_newbcast:%10 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %5, -%4, %9 row_newbcast:%10 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %7, -%6, %9 row_newbcast:%10 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %1, -%1, %8 row_newbcast:%10 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %3, -%3, %8 row_newbcast:%10 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %5, -%5, %8 row_newbcast:%10 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %7, -%7, %8 row_newbcast:%10 row_mask:0xf bank_mask:0xf"
        : "+&v"(a[0].re), "+&v"(a[0].im), "+&v"(a[1].re), "+&v"(a[1].im), "+&v"(a[2].re), "+&v"(a[2].im), "+&v"(a[3].re), "+&v"(a[3].im)
        : "v"(m.re), "v"(m.im), "n"(K));
}

template <int R, int K> __device__ __forceinline__ void row_mac(C2<double>* acc, const C2<double>* w, C2<double> v) {
    if constexpr (R == 1) row_mac1<K>(acc, w, v);
    else if constexpr (R == 2) row_mac2<K>(acc, w, v);
    else if constexpr (R == 3) row_mac3<K>(acc, w, v);
    else row_mac4<K>(acc, w, v);
}

// The value of lane K of each row of 16 lanes (in assembly, with the wait states, as x may
// come straight from one of the blocks above)
template <int K> __device__ __forceinline__ double row_bcast(double x) {
    const int2 u = __builtin_bit_cast(int2, x);
    int2 r;
    asm("s_nop 1\n\t"
        "v_mov_b32_dpp %0, %2 row_newbcast:%4 row_mask:0xf bank_mask:0xf\n\t"
        "v_mov_b32_dpp %1, %3 row_newbcast:%4 row_mask:0xf bank_mask:0xf"
        : "=&v"(r.x), "=&v"(r.y)
        : "v"(u.x), "v"(u.y), "n"(K));
    return __builtin_bit_cast(double, r);
}

}  // namespace bcg
