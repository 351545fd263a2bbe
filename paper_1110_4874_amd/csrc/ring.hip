// Ring stage of synthesis (Wavemoth paper, Sec. 2.3 Eqs. 8-11) and of its
// adjoint, for gfx950.
//
// For ring k with J pixels at phi_j = pi (2j + s) / J:
//   f_j = sum_{m=-L}^{L} q_m e^{i m phi_j},   q_{-m} = conj(q_m)
//       = sum_{b=0}^{J-1} X_b e^{2 pi i b j / J},
//   X_b = sum_{m = b mod J} q_m e^{i pi m s / J}        (phase shift + wrap)
// X is Hermitian, so f is the real backward DFT of X; it is computed as a
// complex DFT of half length n = J/2 (even and odd pixels in the real and
// imaginary parts) after the usual pre-twiddle.
//
// Bin b collects the m of its two residue classes m = b + jJ and m = jJ - b;
// all of them share the phase e^{i pi b s/J} up to the sign (-1)^{js}.  Rings
// with J > L have at most two orders per bin; shorter rings sum theirs
// straight from q, several threads per bin when the ring has fewer bins than
// threads, reduced through LDS in a fixed order (deterministic, no atomics).
//
// The half-length DFT of size S = 2^lg (S = n for a power of two) keeps 16
// points a thread in registers: a thread group of max(64, S / 16) threads, so
// up to S = 1024 one wavefront, which needs no barrier.  Two or three
// passes of up to four radix-2 stages each (RingShape) go through LDS between
// them; the first reads its input in bit-reversed order, the last stores its
// results straight to the map.  Other n are 2h (J is a multiple of 4): the
// even and the odd half, two length-h DFTs one after the other, by Bluestein's
// chirp convolution of size S >= 2h-1: forward decimation in frequency, whose
// last pass meets the pointwise product with the plan's chirp spectrum and
// the first pass of the backward decimation in time in registers.  The first
// pass has zeros in its upper half and the last needs only its lower half, so
// each half costs four LDS exchanges; both halves' results stay in the
// registers of the thread that combines them, z_p = A_p + w^p B_p, z_{p+h} =
// A_p - w^p B_p with w = e^{2 pi i/n}.  LDS indices are padded by one entry
// per 16.  Global loads are issued in batches before their first use.
// The maps of a ring are adjacent in the ring-major q layout; up to S = 1024
// they share a workgroup (a wavefront each), and else run back to back on
// one XCD (dispatch is round-robin over 8 XCDs), so lines read from HBM serve
// them all from L2.
#include <mutex>
#include <set>
#include <utility>

#include <cstring>

#include "internal.h"

namespace sht {

// Complex product with a fixed rounding pattern (explicit fused multiply-adds):
// whichever way the compiler would contract the plain expression, the kernels
// of one plan (several maps per workgroup, one, or the batch queue) agree bit
// for bit.
__device__ __forceinline__ double2 cmul(double2 a, double2 b) {
    return make_double2(__builtin_fma(a.x, b.x, -(a.y * b.y)), __builtin_fma(a.x, b.y, a.y * b.x));
}
__device__ __forceinline__ double2 cconj(double2 a) { return make_double2(a.x, -a.y); }
__device__ __forceinline__ double2 cadd(double2 a, double2 b) { return make_double2(a.x + b.x, a.y + b.y); }
__device__ __forceinline__ double2 csub(double2 a, double2 b) { return make_double2(a.x - b.x, a.y - b.y); }
__device__ __forceinline__ double2 expipi(double x) {  // e^{i pi x}
    double s, c;
    sincospi(x, &s, &c);
    return make_double2(c, s);
}
// x * i conj(y): with y = e^{i pi k/J} and n = J/2, e^{i pi (n - k)/J} = i conj(y)
__device__ __forceinline__ double2 i_conj(double2 y) { return make_double2(y.y, y.x); }
__device__ __forceinline__ int ilog2_dev(int n) { return 31 - __clz(n); }
__device__ __forceinline__ int bitrev(int k, int lg) { return lg == 0 ? 0 : (int)(__brev((unsigned)k) >> (32 - lg)); }
__device__ __forceinline__ int pidx(int i) { return i + (i >> 4); }
// v where on, else 0, without a branch around the load that made v
__device__ __forceinline__ double2 keep(double2 v, bool on) {
    const long long mask = on ? -1LL : 0LL;
    return make_double2(__builtin_bit_cast(double, __builtin_bit_cast(long long, v.x) & mask),
                        __builtin_bit_cast(double, __builtin_bit_cast(long long, v.y) & mask));
}

// Workgroup -> work item, grouping 8 consecutive items on one XCD.
__device__ __forceinline__ int xcd_item(int wg) { return (wg & ~63) + ((wg & 7) << 3) + ((wg >> 3) & 7); }

// Orders LDS accesses between the threads of a group of T: a wavefront's LDS
// operations complete in order, more need the workgroup's barrier.
template <int T>
__device__ __forceinline__ void group_sync() {
    if constexpr (T > 64) {
        __syncthreads();
    } else {
        asm volatile("" ::: "memory");
        __builtin_amdgcn_wave_barrier();
    }
}

// x * e^{2 pi i j / 16} (exact constants)
__device__ __forceinline__ double2 rot16(double2 x, int j) {
    const double r = 0.70710678118654752440, c = 0.92387953251128675613, s = 0.38268343236508977173;
    switch (j & 15) {
        case 0: return x;
        case 1: return cmul(x, make_double2(c, s));
        case 2: return make_double2(r * (x.x - x.y), r * (x.x + x.y));
        case 3: return cmul(x, make_double2(s, c));
        case 4: return make_double2(-x.y, x.x);
        case 5: return cmul(x, make_double2(-s, c));
        case 6: return make_double2(-r * (x.x + x.y), r * (x.x - x.y));
        case 7: return cmul(x, make_double2(-c, s));
        case 8: return make_double2(-x.x, -x.y);
        case 9: return cmul(x, make_double2(-c, -s));
        case 10: return make_double2(r * (x.y - x.x), -r * (x.x + x.y));
        case 11: return cmul(x, make_double2(-s, -c));
        case 12: return make_double2(x.y, -x.x);
        case 13: return cmul(x, make_double2(s, -c));
        case 14: return make_double2(r * (x.x + x.y), r * (x.y - x.x));
        default: return cmul(x, make_double2(c, -s));
    }
}

// x[k] *= w^{bitrev(k)} (CONJ: its conjugate), k < 2^r, from w by products of
// at most five factors.  The empty asm keeps the compiler from computing the
// powers once and holding them across passes (60 registers).
template <int r, bool CONJ>
__device__ __forceinline__ void twiddle(double2 (&x)[1 << r], double2 w) {
    asm volatile("" : "+v"(w.x), "+v"(w.y));
    if (CONJ) w = cconj(w);
    double2 lo[4], hi = make_double2(1.0, 0.0), w4 = hi;
    lo[1] = w;
    if (r > 1) {
        lo[2] = cmul(w, w);
        lo[3] = cmul(lo[2], w);
        if (r > 2) w4 = cmul(lo[2], lo[2]);
    }
#pragma unroll
    for (int e = 1; e < (1 << r); e++) {
        if ((e & 3) == 0) hi = e == 4 ? w4 : e == 8 ? cmul(w4, w4) : cmul(hi, w4);
        const double2 f = e < 4 ? lo[e] : (e & 3) ? cmul(hi, lo[e & 3]) : hi;
        int k = 0;
#pragma unroll
        for (int b = 0; b < r; b++) k |= (e >> b & 1) << (r - 1 - b);
        x[k] = cmul(x[k], f);
    }
}

// r radix-2 stages on R = 2^r elements base + k h, h = 2^(s-1), pos = base mod h.
// Decimation in time, sign +1 (backward): sub-stage u combines k and k + 2^u
// with the twiddle e^{+2 pi i (pos + j h) / (2^(u+1) h)}, j = k mod 2^u.  The
// parts of pos gather on the inputs as wt^{bitrev(k)}, wt = e^{2 pi i pos / (R h)}
// (TRIV: h = 1, wt = 1), which leaves constants between the sub-stages.
// HALF: only the lower half of the results is wanted.
template <int r, bool TRIV, bool HALF>
__device__ __forceinline__ void dit_regs(double2 (&x)[1 << r], double2 wt) {
    if constexpr (!TRIV) twiddle<r, false>(x, wt);
#pragma unroll
    for (int u = 0; u < r; u++) {
        const int span = 1 << u;
#pragma unroll
        for (int k = 0; k < (1 << r); k++) {
            if (k & span) continue;
            const double2 t = rot16(x[k + span], (k & (span - 1)) * (8 >> u));
            if (!(HALF && u == r - 1)) x[k + span] = csub(x[k], t);
            x[k] = cadd(x[k], t);
        }
    }
}

// Decimation in frequency, sign -1 (forward): the sub-stages in reverse order,
// conjugate twiddles after the difference.  HALF: the upper half of the input
// is zero (and not read).
template <int r, bool TRIV, bool HALF>
__device__ __forceinline__ void dif_regs(double2 (&x)[1 << r], double2 wt) {
#pragma unroll
    for (int u = r - 1; u >= 0; u--) {
        const int span = 1 << u;
#pragma unroll
        for (int k = 0; k < (1 << r); k++) {
            if (k & span) continue;
            double2 d = x[k];
            if (!(HALF && u == r - 1)) {
                d = csub(x[k], x[k + span]);
                x[k] = cadd(x[k], x[k + span]);
            }
            x[k + span] = rot16(d, 16 - (k & (span - 1)) * (8 >> u));
        }
    }
    if constexpr (!TRIV) twiddle<r, true>(x, wt);
}

// The transform of size S = 2^LG by T threads: passes of r1 (outermost), r2 and
// r3 (innermost) radix-2 stages; up to S = 16 one thread does it all.
template <int LG, int T>
struct RingFft {
    static constexpr int S = 1 << LG, r1 = ring_shape(LG).r1, r2 = ring_shape(LG).r2, r3 = ring_shape(LG).r3;
    static constexpr int RO = r1 ? r1 : r3;         // stages of the pass that meets input and output
    static constexpr int NO = 1 << RO, ST = S >> RO;  // its points per thread and their stride
    static_assert(ST <= T && (S >> r3) <= T, "one outer and one inner group per thread");
    int tid;
    double2 *buf;
    double2 w1, w2;  // top twiddles of the outer and the middle pass

    __device__ __forceinline__ RingFft(int tid_, double2 *buf_, const double2 *__restrict__ tw, int tw_log)
        : tid(tid_), buf(buf_) {
        w1 = w2 = make_double2(1.0, 0.0);
        if (r1) w1 = tw[min(tid, ST - 1) << (tw_log - LG)];
        if (r2) w2 = tw[(tid & ((1 << r3) - 1)) << (tw_log - r3 - r2)];
    }
    __device__ __forceinline__ bool active() const { return ST == T || tid < ST; }
    __device__ __forceinline__ bool inner() const { return (S >> r3) == T || tid < (S >> r3); }

    // middle pass (its groups of one thread share pos, hence the twiddle)
    template <bool DIT>
    __device__ __forceinline__ void middle() {
        if constexpr (r2 > 0) {
            constexpr int h = 1 << r3;
#pragma unroll
            for (int g0 = 0; g0 < (S >> r2); g0 += T) {
                const int gi = tid + g0;
                if ((S >> r2) % T && gi >= (S >> r2)) break;
                const int base = (gi >> r3) * (h << r2) + (gi & (h - 1));
                double2 x[1 << r2];
#pragma unroll
                for (int k = 0; k < (1 << r2); k++) x[k] = buf[pidx(base + k * h)];
                if (DIT) dit_regs<r2, false, false>(x, w2);
                else dif_regs<r2, false, false>(x, w2);
#pragma unroll
                for (int k = 0; k < (1 << r2); k++) buf[pidx(base + k * h)] = x[k];
            }
            group_sync<T>();
        }
    }

    // Backward DFT of the natural-order input in buf (complete before the
    // call); on return x[k] of an active thread is output tid + k ST.
    __device__ __forceinline__ void backward(double2 (&x)[NO]) {
        if constexpr (r1 == 0) {
            if (inner()) {
#pragma unroll
                for (int k = 0; k < NO; k++) x[k] = buf[pidx(bitrev(k, r3))];
                dit_regs<r3, true, false>(x, w1);
            }
        } else {
            double2 v[1 << r3];
            if (inner()) {
#pragma unroll
                for (int k = 0; k < (1 << r3); k++) v[k] = buf[pidx((bitrev(k, r3) << (LG - r3)) | bitrev(tid, LG - r3))];
                dit_regs<r3, true, false>(v, w1);
            }
            group_sync<T>();  // every input is in registers
            if (inner()) {
#pragma unroll
                for (int k = 0; k < (1 << r3); k++) buf[pidx((tid << r3) + k)] = v[k];
            }
            group_sync<T>();
            middle<true>();
            if (active()) {
#pragma unroll
                for (int k = 0; k < NO; k++) x[k] = buf[pidx(tid + k * ST)];
                dit_regs<r1, false, false>(x, w1);
            }
        }
    }

    // Circular convolution with the spectrum V (laid out [k][group] of the
    // innermost pass): cur[k] of an active thread holds input tid + k ST, k <
    // NO / 2 (the upper half is zero), and on return the output of that index.
    // Writes only what the same thread read last, so calls can follow each
    // other; the buffer's earlier contents must have been read by all.
    // (No array lives across a pass: values merged under a condition would.)
    __device__ __forceinline__ void convolve(double2 (&cur)[NO / 2], const double2 *__restrict__ V) {
        if constexpr (r1 == 0) {
            double2 x[NO];
#pragma unroll
            for (int k = 0; k < NO / 2; k++) x[k] = cur[k];
            dif_regs<r3, true, true>(x, w1);
#pragma unroll
            for (int k = 0; k < NO; k++) x[k] = cmul(x[k], V[k]);
            dit_regs<r3, true, true>(x, w1);
#pragma unroll
            for (int k = 0; k < NO / 2; k++) cur[k] = x[k];
        } else {
            if (active()) {
                double2 x[NO];
#pragma unroll
                for (int k = 0; k < NO / 2; k++) x[k] = cur[k];
                dif_regs<r1, false, true>(x, w1);
#pragma unroll
                for (int k = 0; k < NO; k++) buf[pidx(tid + k * ST)] = x[k];
            }
            group_sync<T>();
            middle<false>();
            if (inner()) {
                constexpr int NG = S >> r3;
                double2 v[1 << r3];
#pragma unroll
                for (int k = 0; k < (1 << r3); k++) v[k] = buf[pidx((tid << r3) + k)];
                dif_regs<r3, true, false>(v, w1);
#pragma unroll
                for (int k0 = 0; k0 < (1 << r3); k0 += 4) {  // four loads at a time: registers
#pragma unroll
                    for (int k = k0; k < k0 + 4; k++) v[k] = cmul(v[k], V[k * NG + tid]);
                    asm volatile("" ::: "memory");
                }
                dit_regs<r3, true, false>(v, w1);
#pragma unroll
                for (int k = 0; k < (1 << r3); k++) buf[pidx((tid << r3) + k)] = v[k];
            }
            group_sync<T>();
            middle<true>();
            double2 x[NO];
#pragma unroll
            for (int k = 0; k < NO; k++) x[k] = buf[pidx(min(tid, ST - 1) + k * ST)];
            dit_regs<r1, false, true>(x, w1);
#pragma unroll
            for (int k = 0; k < NO / 2; k++) cur[k] = x[k];
        }
    }

    // Backward DFT of size n = 2h from the chirp-weighted halves even and odd
    // (input tid + k ST of each, zero past h), by Bluestein: for each of the
    // thread's p = tid + k ST < h, out(p, z_p, z_{p+h}).
    template <typename F>
    __device__ __forceinline__ void bluestein(double2 (&even)[NO / 2], double2 (&odd)[NO / 2], int n,
                                              const double2 *__restrict__ V, const double2 *__restrict__ W, F out) {
        const int h = n / 2;
        double2 A[NO / 2];
#pragma unroll 1
        for (int hh = 0; hh < 2; hh++) {
            convolve(even, V);
            if (hh == 0) {
#pragma unroll
                for (int k = 0; k < NO / 2; k++) {
                    A[k] = even[k];
                    even[k] = odd[k];
                }
            }
        }
        if (!active()) return;
        const double2 ws = expipi(2.0 * ST / n);
        double2 wp;
#pragma unroll
        for (int k0 = 0; k0 < NO / 2; k0 += 4) {
            double2 w[4];
#pragma unroll
            for (int k = 0; k < 4; k++) w[k] = W[min(tid + min(k0 + k, NO / 2 - 1) * ST, h - 1)];
#pragma unroll
            for (int k = k0; k < k0 + 4 && k < NO / 2; k++) {
                const int p = tid + k * ST;
                wp = k == k0 ? expipi(2.0 * p / n) : cmul(wp, ws);  // e^{2 pi i p/n}, stepped by products
                if (p < h) {
                    const double2 Ap = cmul(A[k], w[k - k0]), t = cmul(cmul(even[k], w[k - k0]), wp);
                    out(p, cadd(Ap, t), csub(Ap, t));
                }
            }
        }
    }
};

// f(RingFft) of the transform size 2^lg; a group of T threads has the sizes
// its class holds.
template <int T, typename F>
__device__ __forceinline__ void with_fft(int lg, int tid, double2 *buf, const RingArgs &a, F f) {
#define SHT_FFT(LG) f(RingFft<LG, T>(tid, buf, a.tw, a.tw_log))
    if constexpr (T == 64) {
        switch (lg) {
            case 1: SHT_FFT(1); break;
            case 2: SHT_FFT(2); break;
            case 3: SHT_FFT(3); break;
            case 4: SHT_FFT(4); break;
            case 5: SHT_FFT(5); break;
            case 6: SHT_FFT(6); break;
            case 7: SHT_FFT(7); break;
            case 8: SHT_FFT(8); break;
            case 9: SHT_FFT(9); break;
            default: SHT_FFT(10); break;
        }
    } else if constexpr (T == 128) {
        SHT_FFT(11);
    } else {
        SHT_FFT(12);
    }
#undef SHT_FFT
}

// Raw wrap sums (before the common phase) of the NBIN bins bin[p] of one
// thread (bins with on[p] false give 0) over every order, restricted to the
// terms j = g (mod G): class 1 m = b + jJ (j >= 0), then class 2 m = jJ - b
// (j >= 1), each in increasing j, read straight from the ring's q column
// (stride qs).  Loads go in rounds of U terms of every bin: all of a round's
// loads are issued before the first is added (loads past a bin's last term
// take order 0 and are dropped), so a thread waits for memory once per
// round rather than once per term.
template <int NBIN, int U>
__device__ __forceinline__ void bins_direct(const double2 *__restrict__ qr, size_t qs, int L, int J, int s,
                                            const int (&bin)[NBIN], const bool (&on)[NBIN], int g, int G,
                                            double2 (&acc)[NBIN]) {
    const int g2 = g == 0 ? G : g;  // first j of class 2
    int c1[NBIN], c2[NBIN];         // terms of each class (m <= L: j <= (L -+ b) / J)
    int r1 = 0, r2 = 0;
#pragma unroll
    for (int p = 0; p < NBIN; p++) {
        acc[p] = make_double2(0.0, 0.0);
        const int j1 = (L - bin[p]) / J, j2 = (L + bin[p]) / J;
        c1[p] = on[p] && j1 >= g ? (j1 - g) / G + 1 : 0;
        c2[p] = on[p] && j2 >= g2 ? (j2 - g2) / G + 1 : 0;
        r1 = max(r1, c1[p]);
        r2 = max(r2, c2[p]);
    }
    for (int i0 = 0; i0 < r1; i0 += U) {
        double2 v[NBIN][U];
#pragma unroll
        for (int p = 0; p < NBIN; p++)
#pragma unroll
            for (int u = 0; u < U; u++) {
                const int i = min(i0 + u, c1[p] - 1);
                v[p][u] = qr[(size_t)(i < 0 ? 0 : bin[p] + (g + i * G) * J) * qs];
            }
#pragma unroll
        for (int p = 0; p < NBIN; p++)
#pragma unroll
            for (int u = 0; u < U; u++) {
                const int j = g + (i0 + u) * G;
                if (i0 + u < c1[p]) {
                    double2 x = v[p][u];
                    if (bin[p] + j * J == 0) x.y = 0.0;  // real part of q_0 only
                    if (s & j & 1) x = make_double2(-x.x, -x.y);
                    acc[p] = cadd(acc[p], x);
                }
            }
    }
    for (int i0 = 0; i0 < r2; i0 += U) {
        double2 v[NBIN][U];
#pragma unroll
        for (int p = 0; p < NBIN; p++)
#pragma unroll
            for (int u = 0; u < U; u++) {
                const int i = min(i0 + u, c2[p] - 1);
                v[p][u] = qr[(size_t)(i < 0 ? 0 : (g2 + i * G) * J - bin[p]) * qs];
            }
#pragma unroll
        for (int p = 0; p < NBIN; p++)
#pragma unroll
            for (int u = 0; u < U; u++) {
                const int j = g2 + (i0 + u) * G;
                if (i0 + u < c2[p]) {
                    double2 x = cconj(v[p][u]);
                    if (s & j & 1) x = make_double2(-x.x, -x.y);
                    acc[p] = cadd(acc[p], x);
                }
            }
    }
}

// Synthesis of one ring of one map (item = ring position in the class's list
// times nmaps plus the map) by the T threads tid = 0..T-1 of a group owning
// the LDS block buf.
template <int T>
__device__ __forceinline__ void ring_synth_item(const RingArgs &a, const int item, const int tid, double2 *buf) {
    constexpr int CP = 4;  // bin pairs per thread and batch of loads
    const int pos = item / a.nmaps, b = item % a.nmaps;
    const int rho = a.rings[pos];
    const int J = a.ring_J[rho], s = a.ring_s[rho], M = a.ring_M[rho];
    const int n = J / 2, h = n / 2;
    const bool bs = M > 0;
    const double2 *__restrict__ W = a.chirp + (bs ? a.ring_chirp_off[rho] : 0);
    const int L = a.L;
    const int npair = n / 2 + 1;
    // ring-major q: the maps of one ring interleave in one contiguous block
    const size_t qs = (size_t)a.nmaps;
    const double2 *qr = a.q + (size_t)rho * (L + 1) * a.nmaps + b;

    // the raw sums Xk, Xnk of the pair of bins (k, n - k) (bin n for k = 0),
    // phase shifted, pre-twiddled and stored in the DFT's input: natural order,
    // or (Bluestein) even k at k/2 and odd k at h + (k-1)/2, chirp-weighted
    const double2 sJ = s ? expipi((double)T / J) : make_double2(1.0, 0.0), sn = expipi((double)T / n);
    auto put = [&](int k, double2 Xk, double2 Xnk, double2 pJ, double2 pn, double2 wk, double2 wnk) {
        if (s) {
            Xk = cmul(Xk, pJ);
            Xnk = cmul(Xnk, i_conj(pJ));  // e^{i pi (n - k)/J}, n = J/2
        }
        double2 Zk, Znk = make_double2(0.0, 0.0);
        const bool two = (k != 0) && (2 * k != n);
        if (k == 0) {
            const double2 e = cadd(Xk, cconj(Xnk)), o = csub(Xk, cconj(Xnk));
            Zk = make_double2(e.x - o.y, e.y + o.x);
        } else if (2 * k == n) {
            Zk = make_double2(2.0 * Xk.x, -2.0 * Xk.y);
        } else {
            const double2 e = cadd(Xk, cconj(Xnk));
            const double2 o = cmul(csub(Xk, cconj(Xnk)), pn);
            Zk = make_double2(e.x - o.y, e.y + o.x);
            Znk = make_double2(e.x + o.y, -e.y + o.x);  // conj(e) + i conj(o)
        }
        if (!bs) {
            buf[pidx(k)] = Zk;
            if (two) buf[pidx(n - k)] = Znk;
        } else {
            const int odd = k & 1;
            buf[pidx((k - odd) / 2 + odd * h)] = cmul(Zk, wk);
            if (two) buf[pidx((n - k - odd) / 2 + odd * h)] = cmul(Znk, wnk);
        }
    };
    auto chirp = [&](int k) { return W[max(0, min((k - (k & 1)) / 2, h - 1))]; };
    const double2 one = make_double2(1.0, 0.0);

    if (J <= L && npair <= T) {
        // few bins, several orders each: G groups of npair threads sum the
        // terms j = g mod G of their bins, then reduce
        const int G = T / npair, g = tid / npair, k = tid % npair;
        const int bn[2] = {k, k == 0 ? n : n - k};
        const bool on[2] = {g < G, g < G && 2 * k != n};
        double2 acc[2];
        bins_direct<2, 4>(qr, qs, L, J, s, bn, on, g, G, acc);
        if (G > 1) {
            if (g < G) {
                buf[2 * tid] = acc[0];
                buf[2 * tid + 1] = acc[1];
            }
            group_sync<T>();
            if (tid < npair) {
                acc[0] = acc[1] = make_double2(0.0, 0.0);
                for (int gg = 0; gg < G; gg++) {
                    acc[0] = cadd(acc[0], buf[2 * (gg * npair + tid)]);
                    acc[1] = cadd(acc[1], buf[2 * (gg * npair + tid) + 1]);
                }
            }
            group_sync<T>();
        }
        if (tid < npair)
            put(k, acc[0], acc[1], s ? expipi((double)k / J) : one, expipi((double)k / n), bs ? chirp(k) : one,
                bs ? chirp(n - k) : one);
    } else {
#pragma unroll 1
        for (int k0 = tid; k0 < npair; k0 += T * CP) {
            double2 xa[CP], xb[CP];
            if (J > L) {
                // bin b <= n collects m = b and, when J - b <= L, m = J - b
                // (conjugated, sign (-1)^s); bin n of pair 0 collects m = n
                // twice.  All loads go first, at valid orders.
                const double sg = (s & 1) ? -1.0 : 1.0;
                double2 v[CP][2];
#pragma unroll
                for (int c = 0; c < CP; c++) {
                    const int k = min(k0 + c * T, npair - 1), nk = n - k;
                    xa[c] = qr[(size_t)min(k, L) * qs];
                    xb[c] = qr[(size_t)min(nk, L) * qs];
                }
                if (n <= L) {
#pragma unroll
                    for (int c = 0; c < CP; c++) {
                        const int k = min(k0 + c * T, npair - 1), nk = n - k;
                        v[c][0] = qr[(size_t)(J - k <= L ? J - k : 0) * qs];
                        v[c][1] = qr[(size_t)(J - nk <= L ? J - nk : 0) * qs];
                    }
#pragma unroll
                    for (int c = 0; c < CP; c++) {
                        const int k = min(k0 + c * T, npair - 1), nk = n - k;
                        const double2 wa = keep(v[c][0], k != 0 && J - k <= L), wb = keep(v[c][1], J - nk <= L);
                        xa[c] = make_double2(xa[c].x + sg * wa.x, xa[c].y - sg * wa.y);
                        xb[c] = make_double2(xb[c].x + sg * wb.x, xb[c].y - sg * wb.y);
                        if (k == 0) xa[c].y = 0.0;
                    }
                } else {
#pragma unroll
                    for (int c = 0; c < CP; c++) {
                        const int k = min(k0 + c * T, npair - 1), nk = n - k;
                        xa[c] = keep(xa[c], k <= L);
                        xb[c] = keep(xb[c], nk <= L);
                        if (k == 0) xa[c].y = 0.0;
                    }
                }
            } else {
                // several pairs per thread: rounds of one term of each bin
                int bn[2 * CP];
                bool on[2 * CP];
#pragma unroll
                for (int c = 0; c < CP; c++) {
                    const int k = k0 + c * T;
                    bn[2 * c] = k;
                    bn[2 * c + 1] = k == 0 ? n : n - k;
                    on[2 * c] = k < npair;
                    on[2 * c + 1] = on[2 * c] && 2 * k != n;
                }
                double2 acc[2 * CP];
                bins_direct<2 * CP, 1>(qr, qs, L, J, s, bn, on, 0, 1, acc);
#pragma unroll
                for (int c = 0; c < CP; c++) {
                    xa[c] = acc[2 * c];
                    xb[c] = acc[2 * c + 1];
                }
            }
            double2 wv[CP][2];
            if (bs) {
#pragma unroll
                for (int c = 0; c < CP; c++) {
                    const int k = k0 + c * T;
                    wv[c][0] = chirp(k);
                    wv[c][1] = chirp(n - k);
                }
            }
            // e^{i pi k/J} and e^{i pi k/n}, exact at the batch's first k and
            // stepped by products (about an ulp per step)
            double2 pJ = s ? expipi((double)k0 / J) : one, pn = expipi((double)k0 / n);
#pragma unroll
            for (int c = 0; c < CP; c++) {
                const int k = k0 + c * T;
                if (k < npair) put(k, xa[c], xb[c], pJ, pn, wv[c][0], wv[c][1]);
                pJ = cmul(pJ, sJ);
                pn = cmul(pn, sn);
            }
        }
    }
    group_sync<T>();
    // pixel 2p = Re z_p, pixel 2p+1 = Im z_p
    double2 *out = reinterpret_cast<double2 *>(a.map + (size_t)b * a.npix + a.ring_off[rho]);
    if (!bs) {
        with_fft<T>(ilog2_dev(n), tid, buf, a, [&](auto fft) {
            using F = decltype(fft);
            double2 x[F::NO];
            fft.backward(x);
            if (fft.active()) {
#pragma unroll
                for (int k = 0; k < F::NO; k++) out[tid + k * F::ST] = x[k];
            }
        });
    } else {
        const double2 *__restrict__ V = a.bs_table + a.ring_bs_off[rho];
        with_fft<T>(ilog2_dev(M), tid, buf, a, [&](auto fft) {
            using F = decltype(fft);
            if constexpr (F::r3 >= 3) {  // a Bluestein transform has h >= 3
                double2 even[F::NO / 2], odd[F::NO / 2];
#pragma unroll
                for (int k = 0; k < F::NO / 2; k++) {
                    const int p = tid + k * F::ST, pc = min(p, h - 1);
                    even[k] = keep(buf[pidx(pc)], p < h);
                    odd[k] = keep(buf[pidx(h + pc)], p < h);
                }
                group_sync<T>();
                fft.bluestein(even, odd, n, V, W, [&](int p, double2 z0, double2 z1) {
                    out[p] = z0;
                    out[p + h] = z1;
                });
            }
        });
    }
}

// Groups of T threads; up to T = 64 a workgroup runs G maps of one ring (G
// divides nmaps), a wavefront and an LDS block each.  256 registers, two
// wavefronts a SIMD: the forms of two and four maps spill 6 of them (28 bytes of
// scratch a thread; the analysis 16, 68 bytes), its 128 and 256-thread forms 2
// and 4, the others none.
template <int T, int G>
__global__ __launch_bounds__(T * G, 2) void k_ring_synth(RingArgs a) {
    extern __shared__ double2 sm[];
    static_assert(G == 1 || T == 64, "wavefronts are independent, larger groups are not");
    const int sub = G == 1 ? 0 : __builtin_amdgcn_readfirstlane((int)threadIdx.x / T);
    const int item = xcd_item(blockIdx.x) * G + sub;
    if (item >= a.count * a.nmaps) return;
    ring_synth_item<T>(a, item, (int)threadIdx.x - sub * T, sm + (size_t)sub * a.fft_entries);
}

// Ring queue of a batch of requests: one launch per ring size class for all
// requests, item j = {argument block (request, class), item of that class};
// items are ordered request by request, ring by ring, map by map, so that
// the maps of one ring stay on one XCD as in k_ring_synth.
template <int T>
__global__ __launch_bounds__(T, 2) void k_ring_synth_queue(const RingArgs *__restrict__ args, const int2 *__restrict__ items,
                                                        int nitems) {
    const int j = xcd_item(blockIdx.x);
    if (j >= nitems) return;
    const int2 it = items[j];
    extern __shared__ double2 sm[];
    const RingArgs a = args[__builtin_amdgcn_readfirstlane(it.x)];
    ring_synth_item<T>(a, __builtin_amdgcn_readfirstlane(it.y), threadIdx.x, sm);
}

// Ring stage of the adjoint (the transpose of the above).  For ring k:
//   ybar_m = w_m sum_j y_j e^{-i m phi_j} = w_m e^{-i pi m s/J} F_{m mod J},
//   F_b = sum_j y_j e^{-2 pi i b j/J}  (F_{J-b} = conj F_b),
// with w_0 = 1 and w_m = wpos for m >= 1.  F_0..F_{J/2} come from one complex
// DFT of half length on z_p = y_{2p} + i y_{2p+1} (forward DFT taken as the
// conjugate of the backward one, so the synthesis FFT code is reused), and
// every m of bin b's two residue classes is written from G_b =
// e^{-i pi b s/J} F_b:  ybar_{b+jJ} = w (-1)^{js} G_b,
// ybar_{jJ-b} = w (-1)^{js} conj(G_b).
template <int T, int G>
__global__ __launch_bounds__(T * G, 2) void k_ring_analysis(RingArgs a) {
    extern __shared__ double2 sm[];
    static_assert(G == 1 || T == 64, "wavefronts are independent, larger groups are not");
    const int sub = G == 1 ? 0 : __builtin_amdgcn_readfirstlane((int)threadIdx.x / T);
    const int item = xcd_item(blockIdx.x) * G + sub;
    if (item >= a.count * a.nmaps) return;
    double2 *buf = sm + (size_t)sub * a.fft_entries;
    const int tid = (int)threadIdx.x - sub * T;
    const int pos = item / a.nmaps, b = item % a.nmaps;
    const int rho = a.rings[pos];
    const int J = a.ring_J[rho], s = a.ring_s[rho], M = a.ring_M[rho];
    const int n = J / 2, h = n / 2;
    const bool bs = M > 0;
    const double2 *__restrict__ W = a.chirp + (bs ? a.ring_chirp_off[rho] : 0);
    const int L = a.L;
    const size_t qstride = (size_t)a.nmaps;
    double2 *yr = a.ybar + (size_t)rho * (L + 1) * a.nmaps + b;

    const double2 *pix = reinterpret_cast<const double2 *>(a.map_in + (size_t)b * a.npix + a.ring_off[rho]);
    if (!bs) {
        constexpr int LD = 8;  // loads in flight per thread
#pragma unroll 1
        for (int p0 = tid; p0 < n; p0 += LD * T) {
            double2 x[LD];
#pragma unroll
            for (int j = 0; j < LD; j++) x[j] = pix[min(p0 + j * T, n - 1)];
#pragma unroll
            for (int j = 0; j < LD; j++)
                if (p0 + j * T < n) buf[pidx(p0 + j * T)] = cconj(x[j]);
        }
        group_sync<T>();
        with_fft<T>(ilog2_dev(n), tid, buf, a, [&](auto fft) {
            using F = decltype(fft);
            double2 x[F::NO];
            fft.backward(x);
            if (fft.active()) {  // where this thread read its last pass
#pragma unroll
                for (int k = 0; k < F::NO; k++) buf[pidx(tid + k * F::ST)] = x[k];
            }
        });
    } else {
        const double2 *__restrict__ V = a.bs_table + a.ring_bs_off[rho];
        with_fft<T>(ilog2_dev(M), tid, buf, a, [&](auto fft) {
            using F = decltype(fft);
            if constexpr (F::r3 >= 3) {
                double2 even[F::NO / 2], odd[F::NO / 2];
#pragma unroll
                for (int k0 = 0; k0 < F::NO / 2; k0 += 4) {
                    double2 x[4][2], w[4];
#pragma unroll
                    for (int k = 0; k < 4; k++) {
                        const int pc = min(tid + min(k0 + k, F::NO / 2 - 1) * F::ST, h - 1);
                        x[k][0] = pix[2 * pc];
                        x[k][1] = pix[2 * pc + 1];
                        w[k] = W[pc];
                    }
#pragma unroll
                    for (int k = k0; k < k0 + 4 && k < F::NO / 2; k++) {
                        const bool in = tid + k * F::ST < h;
                        even[k] = keep(cmul(cconj(x[k - k0][0]), w[k - k0]), in);
                        odd[k] = keep(cmul(cconj(x[k - k0][1]), w[k - k0]), in);
                    }
                }
                double2 z0[F::NO / 2], z1[F::NO / 2];
                fft.bluestein(even, odd, n, V, W, [&](int p, double2 zp, double2 zph) {
                    z0[(p - tid) / F::ST] = zp;
                    z1[(p - tid) / F::ST] = zph;
                });
                group_sync<T>();  // the last pass has been read
#pragma unroll
                for (int k = 0; k < F::NO / 2; k++) {
                    const int p = tid + k * F::ST;
                    if (fft.active() && p < h) {
                        buf[pidx(p)] = z0[k];
                        buf[pidx(p + h)] = z1[k];
                    }
                }
            }
        });
    }
    group_sync<T>();

    // bins b = 0..n, split over NG groups of the residue classes for small rings
    const int nb = n + 1;
    const int NG = nb >= T ? 1 : T / nb;
    // e^{-i pi bin/n} and e^{-i pi bin/J}: exact every fourth bin of a thread,
    // stepped by products between (with NG > 1 a thread has one bin)
    const double2 sn = expipi(-(double)T / n), sJ = s ? expipi(-(double)T / J) : make_double2(1.0, 0.0);
    double2 qn, qJ;
    int turn = 0;
    for (int u = tid; u < NG * nb; u += T, turn++) {
        const int g = u / nb, bin = u % nb;
        if ((turn & 3) == 0) {
            qn = expipi(-(double)bin / n);
            qJ = s ? expipi(-(double)bin / J) : make_double2(1.0, 0.0);
        }
        const double2 Zb = cconj(buf[pidx(bin == n ? 0 : bin)]);
        const double2 Znb = cconj(buf[pidx(bin == 0 ? 0 : n - bin)]);
        // F_b = (Z_b + conj Z_{n-b})/2 - (i/2) e^{-2 pi i b/J} (Z_b - conj Z_{n-b})
        const double2 e = cadd(Zb, cconj(Znb));
        const double2 d = cmul(csub(Zb, cconj(Znb)), qn);
        double2 F = make_double2(0.5 * (e.x + d.y), 0.5 * (e.y - d.x));
        double2 Gb = s ? cmul(F, qJ) : F;
        qn = cmul(qn, sn);
        qJ = cmul(qJ, sJ);
        // class 1: m = bin + jJ (j >= 0)
        for (long long j = g;; j += NG) {
            const long long m = bin + j * J;
            if (m > L) break;
            double2 v = (s & j & 1) ? make_double2(-Gb.x, -Gb.y) : Gb;
            if (m == 0) v = make_double2(v.x, 0.0);
            else v = make_double2(a.wpos * v.x, a.wpos * v.y);
            yr[(size_t)m * qstride] = v;
        }
        // class 2: m = jJ - bin (j >= 1); bins 0 and n are covered by class 1
        if (bin != 0 && bin != n) {
            for (long long j = (g == 0 ? NG : g);; j += NG) {
                const long long m = j * J - bin;
                if (m > L) break;
                double2 v = cconj(Gb);
                if (s & j & 1) v = make_double2(-v.x, -v.y);
                yr[(size_t)m * qstride] = make_double2(a.wpos * v.x, a.wpos * v.y);
            }
        }
    }
}

// Raises a kernel's dynamic LDS limit to `bytes`, once per (kernel, device):
// the attribute belongs to the device current at the call.
hipError_t allow_dynamic_lds(const void *fn, int bytes) {
    static std::mutex mu;
    static std::set<std::pair<const void *, int>> done;
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    std::lock_guard<std::mutex> lk(mu);
    if (done.count({fn, dev})) return hipSuccess;
    e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
    if (e == hipSuccess) done.insert({fn, dev});
    return e;
}

// LDS entries of a thread group of T for transforms of up to S points: the
// padded points, at least the 2 T partial bin sums of a short ring.
int ring_group_entries(int S, int T) { return std::max(S + S / 16, 2 * T); }

template <int T, int G>
static hipError_t launch_set(bool adj, const RingArgs &a, hipStream_t st) {
    const void *fn = adj ? (const void *)k_ring_analysis<T, G> : (const void *)k_ring_synth<T, G>;
    hipError_t e = allow_dynamic_lds(fn, 160 * 1024);
    if (e != hipSuccess) return e;
    const size_t lds = (size_t)G * a.fft_entries * sizeof(double2);
    const long long grid = ((long long)a.count * a.nmaps / G + 63) / 64 * 64;
    if (adj) hipLaunchKernelGGL((k_ring_analysis<T, G>), dim3((unsigned)grid), dim3(T * G), lds, st, a);
    else hipLaunchKernelGGL((k_ring_synth<T, G>), dim3((unsigned)grid), dim3(T * G), lds, st, a);
    return hipGetLastError();
}

// One launch per ring size class.
static hipError_t launch_sets(const sht_plan_s *p, bool adj, RingArgs a, hipStream_t st) {
    for (const auto &rs : p->ring_sets) {
        if (rs.rings.empty()) continue;
        a.rings = rs.d_rings;
        a.count = (int)rs.rings.size();
        a.fft_entries = ring_group_entries(rs.max_size, rs.threads);
        hipError_t e;
        switch (rs.threads) {
            case 64:
                e = a.nmaps % 4 == 0 ? launch_set<64, 4>(adj, a, st)
                                     : a.nmaps % 2 == 0 ? launch_set<64, 2>(adj, a, st) : launch_set<64, 1>(adj, a, st);
                break;
            case 128: e = launch_set<128, 1>(adj, a, st); break;
            default: e = launch_set<256, 1>(adj, a, st); break;
        }
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

static const void *ring_queue_kernel(int T) {
    return T == 64 ? (const void *)k_ring_synth_queue<64>
                   : T == 128 ? (const void *)k_ring_synth_queue<128> : (const void *)k_ring_synth_queue<256>;
}

// Raises the ring queue kernel's LDS limit on the current device (done at
// batch creation, so that runs make no runtime calls besides launches).
hipError_t ring_queue_prepare(int T) { return allow_dynamic_lds(ring_queue_kernel(T), 160 * 1024); }

hipError_t launch_ring_queue(int T, const RingArgs *args, const int2 *items, long long nitems, size_t lds,
                             hipStream_t st) {
    if (nitems < 0 || nitems > 0x7fffffffLL) return hipErrorInvalidValue;
    hipError_t e = ring_queue_prepare(T);
    if (e != hipSuccess || nitems == 0) return e;
    const dim3 grid((unsigned)((nitems + 63) / 64 * 64));
    switch (T) {
        case 64: hipLaunchKernelGGL(k_ring_synth_queue<64>, grid, dim3(T), lds, st, args, items, (int)nitems); break;
        case 128: hipLaunchKernelGGL(k_ring_synth_queue<128>, grid, dim3(T), lds, st, args, items, (int)nitems); break;
        default: hipLaunchKernelGGL(k_ring_synth_queue<256>, grid, dim3(T), lds, st, args, items, (int)nitems); break;
    }
    return hipGetLastError();
}

// Plan-wide fields of the ring argument block (synthesis direction); the
// caller sets the class fields (rings, count, fft_entries).
RingArgs ring_args(const sht_plan_s *p, int nmaps, const double *q, double *map) {
    RingArgs a;
    std::memset(&a, 0, sizeof(a));
    a.ring_J = p->d_ring_J;
    a.ring_s = p->d_ring_s;
    a.ring_M = p->d_ring_M;
    a.ring_off = p->d_ring_off;
    a.ring_bs_off = p->d_ring_bs_off;
    a.tw = reinterpret_cast<const double2 *>(p->d_tw);
    a.tw_log = p->tw_log;
    a.bs_table = reinterpret_cast<const double2 *>(p->d_bs_table);
    a.chirp = reinterpret_cast<const double2 *>(p->d_chirp);
    a.ring_chirp_off = p->d_ring_chirp_off;
    a.q = reinterpret_cast<const double2 *>(q);
    a.map = map;
    a.L = p->L;
    a.nrings = p->nrings;
    a.nmaps = nmaps;
    a.npix = 12LL * p->nside * p->nside;
    return a;
}

hipError_t launch_ring_synthesis(const sht_plan_s *p, int nmaps, const double *q, double *map,
                                 hipStream_t stream) {
    return launch_sets(p, false, ring_args(p, nmaps, q, map), stream);
}

hipError_t launch_ring_analysis(const sht_plan_s *p, int nmaps, const double *map, double *ybar,
                                double wpos, hipStream_t stream) {
    RingArgs a = ring_args(p, nmaps, nullptr, nullptr);
    a.map_in = map;
    a.ybar = reinterpret_cast<double2 *>(ybar);
    a.wpos = wpos;
    return launch_sets(p, true, a, stream);
}

}  // namespace sht
