// Wave helpers of the FP64 kernels: multiply-adds whose one operand is
// broadcast within each 16-lane row by DPP (gfx950 row_newbcast), the plain
// broadcast of such a value, and the order of an XCD's work.
#pragma once
#include <hip/hip_runtime.h>

namespace sht {

// acc[c] += x_c * p for c < N (N even), where x_c is the value that lane
// C0 + c of the lane's 16-lane row holds in rv: each FP64 FMA reads rv
// through the DPP broadcast (row_newbcast), so the per-row operands need
// neither one LDS broadcast read per value nor a register each.  In each asm
// block the leading s_nop gives the two wait states that a DPP read needs
// after a vector-ALU write of rv, and nothing can be scheduled inside it.  The
// accumulators are early-clobbered: an accumulator that starts from p or rv
// would else share its register, which the block's later FMAs still read.
#define SHT_FMAC_BC(c, o) "v_fmac_f64_dpp %" #o ", %[rv], %[p] row_newbcast:" #c " row_mask:0xf bank_mask:0xf\n"
template <int N, int C0 = 0>
__device__ __forceinline__ void fmac_row_bcast(double *acc, double rv, double p) {
    static_assert(N % 2 == 0 && C0 % 2 == 0 && C0 + N <= 16, "lanes of one row, in pairs");
    if constexpr (N > 8) {
        fmac_row_bcast<8, C0>(acc, rv, p);
        fmac_row_bcast<N - 8, C0 + 8>(acc + 8, rv, p);
    } else if constexpr (C0 == 8) {
        if constexpr (N == 2)
            asm("s_nop 1\n" SHT_FMAC_BC(8, 0) SHT_FMAC_BC(9, 1)
                : "+&v"(acc[0]), "+&v"(acc[1]) : [rv] "v"(rv), [p] "v"(p));
        else if constexpr (N == 4)
            asm("s_nop 1\n" SHT_FMAC_BC(8, 0) SHT_FMAC_BC(9, 1) SHT_FMAC_BC(10, 2) SHT_FMAC_BC(11, 3)
                : "+&v"(acc[0]), "+&v"(acc[1]), "+&v"(acc[2]), "+&v"(acc[3])
                : [rv] "v"(rv), [p] "v"(p));
        else if constexpr (N == 6)
            asm("s_nop 1\n" SHT_FMAC_BC(8, 0) SHT_FMAC_BC(9, 1) SHT_FMAC_BC(10, 2) SHT_FMAC_BC(11, 3) SHT_FMAC_BC(12, 4)
                    SHT_FMAC_BC(13, 5)
                : "+&v"(acc[0]), "+&v"(acc[1]), "+&v"(acc[2]), "+&v"(acc[3]), "+&v"(acc[4]), "+&v"(acc[5])
                : [rv] "v"(rv), [p] "v"(p));
        else if constexpr (N == 8)
            asm("s_nop 1\n" SHT_FMAC_BC(8, 0) SHT_FMAC_BC(9, 1) SHT_FMAC_BC(10, 2) SHT_FMAC_BC(11, 3) SHT_FMAC_BC(12, 4)
                    SHT_FMAC_BC(13, 5) SHT_FMAC_BC(14, 6) SHT_FMAC_BC(15, 7)
                : "+&v"(acc[0]), "+&v"(acc[1]), "+&v"(acc[2]), "+&v"(acc[3]), "+&v"(acc[4]), "+&v"(acc[5]),
                  "+&v"(acc[6]), "+&v"(acc[7])
                : [rv] "v"(rv), [p] "v"(p));
        else
            static_assert(N == 2, "unsupported lane count");
    } else {
        static_assert(C0 == 0, "rows are read from lane 0 or 8");
        if constexpr (N == 2)
            asm("s_nop 1\n" SHT_FMAC_BC(0, 0) SHT_FMAC_BC(1, 1)
                : "+&v"(acc[0]), "+&v"(acc[1]) : [rv] "v"(rv), [p] "v"(p));
        else if constexpr (N == 4)
            asm("s_nop 1\n" SHT_FMAC_BC(0, 0) SHT_FMAC_BC(1, 1) SHT_FMAC_BC(2, 2) SHT_FMAC_BC(3, 3)
                : "+&v"(acc[0]), "+&v"(acc[1]), "+&v"(acc[2]), "+&v"(acc[3])
                : [rv] "v"(rv), [p] "v"(p));
        else if constexpr (N == 6)
            asm("s_nop 1\n" SHT_FMAC_BC(0, 0) SHT_FMAC_BC(1, 1) SHT_FMAC_BC(2, 2) SHT_FMAC_BC(3, 3) SHT_FMAC_BC(4, 4)
                    SHT_FMAC_BC(5, 5)
                : "+&v"(acc[0]), "+&v"(acc[1]), "+&v"(acc[2]), "+&v"(acc[3]), "+&v"(acc[4]), "+&v"(acc[5])
                : [rv] "v"(rv), [p] "v"(p));
        else
            asm("s_nop 1\n" SHT_FMAC_BC(0, 0) SHT_FMAC_BC(1, 1) SHT_FMAC_BC(2, 2) SHT_FMAC_BC(3, 3) SHT_FMAC_BC(4, 4)
                    SHT_FMAC_BC(5, 5) SHT_FMAC_BC(6, 6) SHT_FMAC_BC(7, 7)
                : "+&v"(acc[0]), "+&v"(acc[1]), "+&v"(acc[2]), "+&v"(acc[3]), "+&v"(acc[4]), "+&v"(acc[5]),
                  "+&v"(acc[6]), "+&v"(acc[7])
                : [rv] "v"(rv), [p] "v"(p));
    }
}
#undef SHT_FMAC_BC

// The value of lane K of each 16-lane row, in every lane of that row.
template <int K>
__device__ __forceinline__ double row_bcast(double x) {
    return __builtin_amdgcn_mov_dpp(x, 0x150 + K, 0xF, 0xF, false);
}

// x + the value of the lane N to the right, cyclic within each row of 16
template <int N>
__device__ __forceinline__ double row_ror_add(double x) {
    const long long v = __builtin_bit_cast(long long, x);
    const int lo = __builtin_amdgcn_mov_dpp((int)v, 0x120 + N, 0xF, 0xF, false);
    const int hi = __builtin_amdgcn_mov_dpp((int)(v >> 32), 0x120 + N, 0xF, 0xF, false);
    return x + __builtin_bit_cast(double, ((long long)hi << 32) | (long long)(unsigned)lo);
}

// Order m of item s of XCD xcd (workgroups are dealt to the 8 XCDs round
// robin): eight consecutive orders of each 64, so that the XCD's L2 serves an
// order's coefficient and a_lm stream to all its blocks, and gathers the 16
// bytes per map of neighbouring orders of a ring into whole lines.  Every
// other 64 orders are dealt in reverse, which evens out the chain lengths.
// Low orders (the longest chains) come first.  Orders past L are skipped by
// the caller; items go up to (L + 64) / 64 * 8.
__device__ __forceinline__ int xcd_order(int xcd, int s) {
    const int j = s >> 3;
    return 64 * j + 8 * (j & 1 ? 7 - xcd : xcd) + (s & 7);
}

}  // namespace sht
