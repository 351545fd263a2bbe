// Polarized (spin-2) synthesis as scalar transforms, for gfx950.
//
// The Discussion of the Wavemoth paper notes that the transform of a
// polarized map reduces to three scalar transforms (citing the reductions
// through spin-raising operators), which also amortises the streaming of
// the precomputed data.  With a_{+-2,lm} = -(E_lm +- i B_lm) and
// Q +- iU = sum a_{+-2,lm} _{+-2}Y_lm, the spin-2 functions follow from the
// scalar ones by two spin raisings; with N_l = sqrt((l-2)!/(l+2)!),
// c = cos(theta), s = sin(theta):
//   F1 = (_2 lambda + _-2 lambda)/2 = N_l [2 (m^2 lambda - c s lambda')/s^2 - l(l+1) lambda]
//   F2 = (_2 lambda - _-2 lambda)/2 = N_l 2 m (c lambda - s lambda')/s^2
// and s lambda'_lm = l e_{l+1} lambda_{l+1} - (l+1) e_l lambda_{l-1},
// e_l = sqrt((l^2 - m^2)/(4 l^2 - 1)).  So per mode (E, B) three scalar
// coefficient sets, of band limit L = L_pol + 1,
//   S0: N_l a_l,  S1: l(l+1) N_l a_l,
//   S2: (l-1) e_l N_{l-1} a_{l-1} - (l+2) e_{l+1} N_{l+1} a_{l+1},
// run through the scalar Legendre phase as six maps per polarized map (one
// pass over the plan's data for all of them), and per ring and order
//   F1 = 2 (m^2 S0 - c S2)/s^2 - S1,   F2 = 2 m (c S0 - S2)/s^2,
//   Q_m = -(F1[E] + i F2[B]),   U_m = -(F1[B] - i F2[E]),
// then the scalar ring stage on 2 maps per polarized map.
//
// The division by s^2 costs ~eps / s^2 of the map's scale near the poles;
// on the rings with s below the plan's threshold the spin-2 functions are
// evaluated directly instead: the Wigner-d three-term recurrence in l,
//   _s lambda_{l+1} = A_l (c + m s/(l(l+1))) _s lambda_l - (A_l / A_{l-1}) _s lambda_{l-1},
//   A_l = sqrt((2l+3)(2l+1)(l+1)^2 / (((l+1)^2 - m^2)((l+1)^2 - s^2))),
// from Goldberg's closed form at l0 = max(m, 2), with the plan's per-(m, s)
// start factors.  Evaluated as written it loses ~l eps / s in FP64, so it runs
// split about its solution at the pole, as the scalar one does there
// (legendre.hip): with r_l the ratio of _s lambda_{l+1} to _s lambda_l at
// theta -> 0 and v = 1 - c = 2 sin^2(theta/2),
//   _s lambda_{l+1} = r_l _s lambda_l + d_l,
//   d_l = A_l / (A_{l-1} r_{l-1}) d_{l-1} - A_l v _s lambda_l,
//   r_l^2 = (2l+3)/(2l+1) (l+1+M)(l+1-M') / ((l+1-M)(l+1+M')),
// {M, M'} = {m, -s}, the larger first.  One workgroup per (m, 64 polar rings),
// one wave per s; both hemispheres from one recurrence
// (_s lambda(pi - theta) = (-1)^(l+m) _{-s} lambda(theta)).
#include "ddmath.h"
#include "dpp.h"
#include "internal.h"

namespace sht {

namespace {

__device__ __forceinline__ double2 ld2(const double *p) { return *reinterpret_cast<const double2 *>(p); }

}  // namespace

// ---- coefficient sets -------------------------------------------------------
// E, B: [nalm(L-1)][n] complex; out: [nalm(L)][6n] complex, map 6b + {0, 1, 2}
// = S0, S1, S2 of E_b, 6b + {3, 4, 5} of B_b.  One thread per entry of an
// order (workgroup L + 1 apart: the next 256), the six loads unconditional, of
// degrees clamped to the order's (one workgroup per order and loads under their
// conditions, one after the other: 30 us at L = 1023, one map; so 25 us).
constexpr int kPolPrep = 256;
__global__ __launch_bounds__(kPolPrep) void k_pol_prep(const double *__restrict__ E, const double *__restrict__ B,
                                                       double *__restrict__ out, int L, int n) {
    const int m = blockIdx.x % (L + 1);
    const int Lp = L - 1;
    const size_t offo = (size_t)m * (2 * L + 3 - m) / 2;
    const size_t offi = (size_t)m * (2 * Lp + 3 - m) / 2;  // valid for m <= Lp
    const int e = blockIdx.x / (L + 1) * kPolPrep + threadIdx.x;
    if (e >= (L - m + 1) * n) return;
    const int l = m + e / n, b = e % n;
    double2 *o = reinterpret_cast<double2 *>(out) + (offo + l - m) * 6 * n + 6 * b;
    if (m > Lp) {  // the order L has no input
        for (int c = 0; c < 6; c++) o[c] = make_double2(0.0, 0.0);
        return;
    }
    double2 a[2][3];  // a_lm of E and B at l - 1, l, l + 1
#pragma unroll
    for (int d = 0; d < 3; d++) {
        const size_t at = (offi + (min(max(l - 1 + d, m), Lp) - m)) * n + b;
        a[0][d] = ld2(E + 2 * at);
        a[1][d] = ld2(B + 2 * at);
    }
#pragma unroll
    for (int d = 0; d < 3; d++) {
        // N_l a_lm for 2 <= l <= Lp, l >= m; Im a_l0 ignored
        const int ll = l - 1 + d;
        const bool none = ll < 2 || ll < m || ll > Lp;
        const double nl = 1.0 / sqrt((double)(ll - 1) * ll * (double)(ll + 1) * (ll + 2));
#pragma unroll
        for (int mode = 0; mode < 2; mode++) {
            double2 &x = a[mode][d];
            x.x = none ? 0.0 : x.x * nl;
            x.y = none || m == 0 ? 0.0 : x.y * nl;
        }
    }
    auto eps = [&](int l) -> double {
        return l > m ? sqrt(((double)l * l - (double)m * m) / (4.0 * l * l - 1.0)) : 0.0;
    };
    const double w = (double)l * (l + 1);
    const double f0 = (double)(l - 1) * eps(l), f1 = (double)(l + 2) * eps(l + 1);
#pragma unroll
    for (int mode = 0; mode < 2; mode++) {
        const double2 cm1 = a[mode][0], c = a[mode][1], cp1 = a[mode][2];
        o[3 * mode + 0] = c;
        o[3 * mode + 1] = make_double2(w * c.x, w * c.y);
        o[3 * mode + 2] = make_double2(f0 * cm1.x - f1 * cp1.x, f0 * cm1.y - f1 * cp1.y);
    }
}

struct PolArgs {
    const double *__restrict__ E;
    const double *__restrict__ B;
    const double *__restrict__ ring;  // [pol_n][6] z, sin(theta/2), cos(theta/2) (hi, lo)
    const double *__restrict__ K;     // [(L+1)*2][4]
    const int *__restrict__ grp_lo;   // scalar chain starts per (m, 64-ring group)
    double *__restrict__ q2;
    int L, nrings, pol_n, ng, ngp, n, map0;  // ng: the plan's 64-ring groups, ngp: polar groups
};

// ---- spin-2 combination -----------------------------------------------------
// One thread per (ring, m, polarized map): q6 [rings][L+1][6n] -> q2
// [rings][L+1][2n] (Q of map b at b, U at n + b), but for what the polar
// workgroups of the same launch write.
constexpr int kPolThreads = 128;
struct CombineArgs {
    const double *__restrict__ q6;
    const double *__restrict__ z2_hi;
    const double *__restrict__ z2_lo;
    int n_north;
    long long total;
};

__device__ __forceinline__ bool pol_dead(const PolArgs &a, int m, int g) {
    return a.grp_lo[(size_t)m * a.ng + g] >= (a.L - m) / 2 + 1;  // every chain stays below the cutoff
}

__device__ __forceinline__ void pol_combine(const CombineArgs &f, const PolArgs &a, long long t) {
    if (t >= f.total) return;
    const int L = a.L, n = a.n;
    const int b = (int)(t % n);
    const long long rm = t / n;
    const int m = (int)(rm % (L + 1)), r = (int)(rm / (L + 1));
    const int k = r < f.n_north ? r : a.nrings - 1 - r;
    if (k < a.pol_n && m < L && !pol_dead(a, m, k / 64)) return;
    const double *q6 = f.q6;
    const double zz = f.z2_hi[k];
    const double c = r < f.n_north ? sqrt(zz) : -sqrt(zz);
    const double s2 = (1.0 - zz) - f.z2_lo[k];
    const double2 *S = reinterpret_cast<const double2 *>(q6) + (size_t)rm * 6 * n + 6 * b;
    const double mm = (double)m * m, inv = 1.0 / s2;
    double2 F1[2], F2[2];
    for (int mode = 0; mode < 2; mode++) {
        const double2 S0 = S[3 * mode], S1 = S[3 * mode + 1], S2 = S[3 * mode + 2];
        F1[mode] = make_double2(2.0 * (mm * S0.x - c * S2.x) * inv - S1.x, 2.0 * (mm * S0.y - c * S2.y) * inv - S1.y);
        F2[mode] = make_double2(2.0 * m * (c * S0.x - S2.x) * inv, 2.0 * m * (c * S0.y - S2.y) * inv);
    }
    // Q = -(F1[E] + i F2[B]),  U = -(F1[B] - i F2[E])
    double2 Q = make_double2(-F1[0].x + F2[1].y, -F1[0].y - F2[1].x);
    double2 U = make_double2(-F1[1].x - F2[0].y, -F1[1].y + F2[0].x);
    if (m == 0) Q.y = U.y = 0.0;  // real fields
    double2 *o = reinterpret_cast<double2 *>(a.q2) + (size_t)rm * 2 * n;
    o[b] = Q;
    o[n + b] = U;
}

// ---- polar caps: the spin-2 recurrence itself -------------------------------
// mant * base^p with exponent tracking (mant kept in [0.5, 1) by powers of 2)
__device__ __forceinline__ void dd_pow_acc(dd &mant, int &e, dd base, int p) {
    int eb;
    const double bh = frexp(base.h, &eb);
    dd bm = {bh, ldexp(base.l, -eb)};
    int ex;
    for (; p > 0; p >>= 1) {
        if (p & 1) {
            mant = dd_mul(mant, bm);
            e += eb;
            const double h = frexp(mant.h, &ex);
            mant = {h, ldexp(mant.l, -ex)};
            e += ex;
        }
        bm = dd_mul(bm, bm);
        eb *= 2;
        const double h = frexp(bm.h, &ex);
        bm = {h, ldexp(bm.l, -ex)};
        eb += ex;
    }
}

// A_l and r_l of the file's head
__device__ __forceinline__ dd pol_A(double l, double mm) {
    const double q = l + 1.0;
    return dd_sqrt(dd_div(dd{(2.0 * l + 3.0) * (2.0 * l + 1.0) * q * q, 0.0}, dd{(q * q - mm) * (q * q - 4.0), 0.0}));
}
__device__ __forceinline__ dd pol_r(double l, double M, double M1) {
    const double q = l + 1.0;
    return dd_sqrt(dd_div(dd{(2.0 * l + 3.0) * (q + M) * (q - M1), 0.0}, dd{(2.0 * l + 1.0) * (q - M) * (q + M1), 0.0}));
}

// Rows of 64 degrees at a time are staged in the wave's LDS: E and B of NB
// maps (4 NB values) and the three coefficients, read by DPP row broadcasts.
// Values are held as p 2^(300 S), S <= 0, checked every 8 steps (a step grows
// them by less than 2^13); those with S < 0 are below 2^-180 and left out of
// the sums.  The recurrence is a serial chain of Lp - l0 steps of about four
// dependent operations; in double-double arithmetic (one wave for both s) it
// took 530 us at L = 1023 for one map.
constexpr int kPolRows = 64;

template <int NB>
__device__ __forceinline__ void pol_polar(const PolArgs &a, int m, int g, double (&lds)[2][kPolRows * 16]) {
    constexpr int NV = 4 * NB, CW = 16;
    static_assert(NV + 3 <= CW, "a row holds the values of NB maps and the coefficients");
    const int L = a.L, Lp = L - 1;
    const int si = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), lane = threadIdx.x & 63;
    if (pol_dead(a, m, g)) return;  // the combination writes 0
    const int k = g * 64 + lane;
    const bool act = k < a.pol_n;
    const int kk = act ? k : a.pol_n - 1;
    const dd sh = {a.ring[6 * kk + 2], a.ring[6 * kk + 3]};
    const dd chh = {a.ring[6 * kk + 4], a.ring[6 * kk + 5]};
    const double v = 2.0 * dd_mul(sh, sh).h;
    const int l0 = m > 2 ? m : 2;
    const int s = si == 0 ? 2 : -2;
    double *rows = lds[si];

    // start value and its power of two
    double P0;
    int S;
    {
        const int r = m - s > 0 ? m - s : 0;
        const int pc = 2 * r + s - m, ps = 2 * l0 - pc;
        const double *Kp = a.K + ((size_t)m * 2 + si) * 4;
        dd mant = {Kp[0], Kp[1]};
        int e = (int)Kp[2];
        dd_pow_acc(mant, e, chh, pc);
        dd_pow_acc(mant, e, sh, ps);
        S = e >= 0 ? 0 : -(-e / 300);
        P0 = ldexp(mant.h, e - 300 * S);
    }
    const double mm = (double)m * m, M = m > -s ? m : -s, M1 = m > -s ? -s : m;
    double P1 = -(pol_A((double)l0, mm).h * v) * P0;  // d at l0
    double live = S == 0 ? 1.0 : 0.0;
    bool dead = __any(S < 0);

    double acc[2][NV];  // by parity of l - l0: sums of E and B (re, im) of each map
#pragma unroll
    for (int q = 0; q < NV; q++) acc[0][q] = acc[1][q] = 0.0;
    const size_t offi = (size_t)m * (2 * Lp + 3 - m) / 2;
    double2 pe[NB], pb[NB];
    auto fetch = [&](int lb) {  // rows lb .. lb + 63, clamped to Lp (rows past it are staged as zeros)
        const size_t at = (offi + min(lb + lane, Lp) - m) * a.n + a.map0;
#pragma unroll
        for (int b = 0; b < NB; b++) {
            pe[b] = reinterpret_cast<const double2 *>(a.E)[at + b];
            pb[b] = reinterpret_cast<const double2 *>(a.B)[at + b];
        }
    };
    fetch(l0);
    for (int lb = l0; lb <= Lp; lb += kPolRows) {
        double2 *row = reinterpret_cast<double2 *>(rows + lane * CW);
#pragma unroll
        for (int b = 0; b < NB; b++) {
            row[2 * b] = pe[b];
            row[2 * b + 1] = pb[b];
        }
        if (lb + lane > Lp) {
#pragma unroll
            for (int q = 0; q < NV / 2; q++) row[q] = make_double2(0.0, 0.0);
        }
        {
            // step l: lambda_{l+1} = r_l lambda_l + d_l, then d_{l+1}
            const double l = lb + lane;
            const dd A = pol_A(l, mm), A1 = pol_A(l + 1.0, mm), r = pol_r(l, M, M1);
            double *c = rows + lane * CW + NV;
            c[0] = dd_div(A1, dd_mul(A, r)).h;
            c[1] = -A1.h;
            c[2] = r.h;
        }
        fetch(lb + kPolRows);
        const int steps = min(kPolRows, Lp - lb + 1);
        for (int j = 0; j < steps; j += 8) {
            double rv[8];
#pragma unroll
            for (int u = 0; u < 8; u++) rv[u] = rows[(j + u) * CW + (lane & 15)];
#pragma unroll
            for (int u = 0; u < 8; u++) {
                const double h = row_bcast<NV>(rv[u]), nA = row_bcast<NV + 1>(rv[u]), r = row_bcast<NV + 2>(rv[u]);
                fmac_row_bcast<NV>(acc[u & 1], rv[u], dead ? P0 * live : P0);
                const double nx = __builtin_fma(r, P0, P1);
                P1 = __builtin_fma(h, P1, (nA * v) * nx);
                P0 = nx;
            }
            if (dead) {
                if (S < 0 && fabs(P0) > 1.0) {
                    P0 = ldexp(P0, -300);
                    P1 = ldexp(P1, -300);
                    S++;
                }
                live = S == 0 ? 1.0 : 0.0;
                dead = __any(S < 0);
            }
        }
    }
    // Even and odd l - m: the north sum of this s, and the south sum of -s.
    // Wave 0 writes the north ring, wave 1 its mirror.
    const bool odd0 = (l0 - m) & 1;
    double north[NV], south[NV];
#pragma unroll
    for (int q = 0; q < NV; q++) {
        north[q] = acc[0][q] + acc[1][q];
        south[q] = odd0 ? acc[1][q] - acc[0][q] : acc[0][q] - acc[1][q];
        rows[q * 64 + lane] = si == 0 ? south[q] : north[q];
    }
    __syncthreads();
    if (!act) return;
    // sums over s = +2 (p) and -2 (q) at this wave's ring: F1 = (p + q)/2, F2 = (p - q)/2
    const double *other = lds[1 - si];
    const int ring = si == 0 ? k : a.nrings - 1 - k;
    double2 *o = reinterpret_cast<double2 *>(a.q2) + ((size_t)ring * (L + 1) + m) * 2 * a.n + a.map0;
#pragma unroll
    for (int b = 0; b < NB; b++) {
        double F1[4], F2[4];  // E re, im, B re, im
#pragma unroll
        for (int c = 0; c < 4; c++) {
            // north: own is s = +2; south: own (s = -2's sums) stands for +2
            const double p = si == 0 ? north[4 * b + c] : south[4 * b + c], q = other[(4 * b + c) * 64 + lane];
            F1[c] = 0.5 * (p + q);
            F2[c] = 0.5 * (p - q);
            if (m == 0 && (c & 1)) F1[c] = F2[c] = 0.0;  // real fields
        }
        // Q = -(sum E F1 + i sum B F2), U = -(sum B F1 - i sum E F2)
        double2 Q = make_double2(-F1[0] + F2[3], -F1[1] - F2[2]);
        double2 U = make_double2(-F1[2] - F2[1], -F1[3] + F2[0]);
        if (m == 0) Q.y = U.y = 0.0;
        o[b] = Q;
        o[a.n + b] = U;
    }
}

// The polar workgroups first: each is a long serial chain, which the
// combination's streaming fills (L = 1023, one map: 81 + 48 us as two launches,
// 84 us as one).
template <int NB>
__global__ __launch_bounds__(kPolThreads) void k_pol_finish(PolArgs a, CombineArgs f, int polar) {
    __shared__ __attribute__((aligned(16))) double lds[2][kPolRows * 16];
    if ((int)blockIdx.x < polar)
        pol_polar<NB>(a, blockIdx.x / a.ngp, blockIdx.x % a.ngp, lds);
    else
        pol_combine(f, a, ((long long)blockIdx.x - polar) * kPolThreads + threadIdx.x);
}

size_t pol_alm_bytes(const sht_plan_s *p, int nmaps) {
    return ((size_t)(p->L + 1) * (p->L + 2) / 2 * 6 * nmaps * 16 + 255) / 256 * 256;
}

hipError_t launch_pol_prep(const sht_plan_s *p, int nmaps, const double *E, const double *B, double *alm6,
                           hipStream_t st) {
    const long long per = ((long long)(p->L + 1) * nmaps + kPolPrep - 1) / kPolPrep;
    const dim3 grid((unsigned)((p->L + 1) * per));
    hipLaunchKernelGGL(k_pol_prep, grid, dim3(kPolPrep), 0, st, E, B, alm6, p->L, nmaps);
    return hipGetLastError();
}

hipError_t launch_pol_finish(const sht_plan_s *p, int nmaps, const double *E, const double *B, const double *q6,
                             double *q2, hipStream_t st) {
    const bool caps = p->pol_n > 0 && p->L >= 3;
    PolArgs a;
    a.E = E;
    a.B = B;
    a.ring = p->d_pol_ring;
    a.K = p->d_pol_K;
    a.grp_lo = p->d_grp_lo;
    a.q2 = q2;
    a.L = p->L;
    a.nrings = p->nrings;
    a.pol_n = caps ? p->pol_n : 0;
    a.n = nmaps;
    a.ng = p->n_north_pad / kLanes;
    a.ngp = caps ? (p->pol_n + 63) / 64 : 1;
    const int polar = caps ? p->L * a.ngp : 0;  // orders 0 .. L-1 x polar groups
    CombineArgs f;
    f.q6 = q6;
    f.z2_hi = p->d_z2_hi;
    f.z2_lo = p->d_z2_lo;
    f.n_north = p->n_north;
    f.total = (long long)p->nrings * (p->L + 1) * nmaps;  // in the first launch
    hipError_t e = hipSuccess;
    for (int b = 0; b < nmaps && e == hipSuccess;) {
        const int nb = nmaps - b == 4 ? 2 : std::min(nmaps - b, 3);
        a.map0 = b;
        const dim3 grid((unsigned)(polar + (f.total + kPolThreads - 1) / kPolThreads));
        if (nb == 3)
            hipLaunchKernelGGL(k_pol_finish<3>, grid, dim3(kPolThreads), 0, st, a, f, polar);
        else if (nb == 2)
            hipLaunchKernelGGL(k_pol_finish<2>, grid, dim3(kPolThreads), 0, st, a, f, polar);
        else
            hipLaunchKernelGGL(k_pol_finish<1>, grid, dim3(kPolThreads), 0, st, a, f, polar);
        e = hipGetLastError();
        b += nb;
        f.total = 0;
        if (!caps) break;
    }
    return e;
}

}  // namespace sht
