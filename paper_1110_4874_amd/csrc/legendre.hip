// Brute-force Legendre phase (Wavemoth paper, Sec. 2.4 Eqs. 12-14 and
// App. A.2 Eqs. A1-A2), for gfx950.
//
//   q_m(+-z_k) = q^even_m(z_k) +- q^odd_m(z_k),
//   q^t_m(z)   = sum_i P~_{m+t+2i}^m(z) a_{m+t+2i, m}
//
// One workgroup of two wavefronts handles one order m and a block of 64 x R
// north rings; wave t runs the two-step recurrence of parity t with R rings
// per lane, so the even and the odd chain advance side by side.  The
// recurrence coefficients and the a_lm of a chain step are the same for every
// lane: the wave fetches them a chunk of kChunk steps ahead with coalesced
// loads, stages them as rows of 16 (32) doubles in its own LDS slot, and the
// FP64 multiply-adds read them from one register per row through DPP row
// broadcasts.  P~ never leaves VGPRs (the GPU form of the paper's
// register-resident SSE kernel).  The even/odd fold of Eqs. 13-14 is fused
// into the store: the waves swap their sums through LDS and write ring k and
// its mirror 4N-2-k.
//
// Chains start at the plan's precomputed values (first l above the cutoff,
// rounded down to a multiple of kChunk chain steps), so a lane joins the
// wave-uniform loop only at chunk boundaries.
//
// The two-step recurrence runs in the scaling P~_l = f_l mu_l with f_{l+2} f_l
// = 1 / c_l, which makes its last coefficient -1:
//   mu_{l+2} = b_l (z^2 - d_l) mu_l - mu_{l-2},  b_l = f_l^2
// (c_l, d_l of App. A.2; f runs from about sqrt(m) to 2).
// Two FP64 operations a step instead of three; the f_l go into the staged
// a_lm.
//
// Near the poles a z-based FP64 recurrence loses ~l eps / sin(theta): z^2
// carries sin^2(theta) with an absolute error of eps.  The ring groups there
// run the recurrence split about its solution at the pole (the idea of
// Reinsch's modification of Clenshaw's recurrence): with r_l the ratio
// P~_{l+2}/P~_l at theta -> 0, P~_{l+2} = (r_l + h_l - sin^2 beta_l) P~_l -
// h_l r_{l-2} P~_{l-2} exactly, so
//   P~_{l+2} = r_l P~_l + d_l,   d_{l+2} = h_{l+2} d_l - sin^2 beta_{l+2} P~_{l+2}
// where sin^2(theta) enters with its own relative accuracy (in the scaled
// variables with the coefficients scaled likewise).  Four FP64 operations a
// step instead of two; phases on rings with sin(theta) <= 0.1 are off by 2e-15 to
// 8e-15 at L = 4095 (relative rms of a ring, white spectrum).
//
// Plans whose threshold the caller set, and polar groups that reach too far
// from the pole for the split recurrence, run those groups in double-double (31
// operations a step, one ring a lane, with priority over the other waves: the
// chain is serial).  Bound by the issue of those operations where most rings
// are such, else by the chain.  As launches of their own, with operands read
// step by step, they took 540 us at L = 1400, nside = 40, one map, and 2017 us
// at L = 4095, nside = 32 (whole syntheses); so 190 and 749 us.
#include <type_traits>

#include "ddmath.h"
#include "dpp.h"
#include "internal.h"

namespace sht {

// The recurrence of a ring group: scaled two-step, split about the pole, or
// two-step in double-double.
enum class Chain { PLAIN, SPLIT, DD };

// Staged row of a chain step: a_lm of NB maps (2 NB values), then the
// coefficients (two; split recurrence three; double-double three high and
// three low parts), in rows of 8, 16 or 32 doubles.  Two
// rows of 8 share one 16-lane read, and half as many values are fetched and
// staged (Legendre phase with rows of 16 and of 8: L = 1023, 1 map 121 and 113
// us, 3 maps 176 and 165; L = 2047, 1 map 780 and 750, 2 maps 961 and 919).
constexpr int leg_coefs(Chain K) { return K == Chain::DD ? 6 : K == Chain::SPLIT ? 3 : 2; }
template <int NB, Chain K>
constexpr int leg_row() {
    constexpr int v = 2 * NB + leg_coefs(K);
    return v <= 8 ? 8 : v <= 16 ? 16 : 32;
}
// LDS doubles of one wave: two staged chunks, and the chains' start values
// (R rings, or one in double-double) whose room holds one ring group's sums at
// the fold.  DD: of a kernel that has double-double blocks.
template <int NB, int R, bool DD>
constexpr int leg_wave_lds() {
    constexpr int sums = 128 * NB, starts = 128 * (DD && R < 2 ? 2 : R);
    return 2 * kChunk * leg_row<NB, DD ? Chain::DD : Chain::SPLIT>() + (starts > sums ? starts : sums);
}

// One workgroup: order m, rings of the 64-ring groups g0 .. min(g0 + R, gend) - 1
// (R per lane); wave t = threadIdx.x / 64 runs parity t.  W: LDS doubles of a wave.
template <int NB, int R, Chain K, int W>
__device__ __forceinline__ void leg_block(const LegArgs &a, const int m, const int g0, const int gend, double *lds) {
    constexpr bool SPLIT = K == Chain::SPLIT, DD = K == Chain::DD;
    constexpr int NC = 2 * NB;
    constexpr int CW = leg_row<NB, K>(), CS = kChunk * CW, E = CS / 64;
    constexpr int CB = CW == 32 ? 16 : NC;  // component of the first coefficient
    constexpr int CO = CB % 16;             // its lane within its 16-lane row
    static_assert(CO + leg_coefs(K) <= 16, "the coefficients share one 16-lane row");
    static_assert(2 * CS + 128 * NB <= W && 2 * CS + 128 * (DD ? 2 : R) <= W, "chunks, sums and starts fit");
    static_assert(!DD || R == 1, "one ring a lane in double-double");
    constexpr int KU = 4;                 // rows read from LDS at once
    constexpr int PK = CW < 16 ? 16 / CW : 1;  // rows within one 16-lane read
    const int t = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int L = a.L;
    const int n = L - m - t >= 0 ? (L - m - t) / 2 + 1 : 0;  // chain length
    double *room = lds + t * W;
    double *stg = room + (W - 2 * CS);
    const double4 *cf = reinterpret_cast<const double4 *>(a.coef_sc) + a.coef_off[m] + t;

    int sid[R], lo = kDead, hi = -1;
    double x[R], P0[R], P1[R], acc[R][NC];
    double xl = 0.0, P0l = 0.0, P1l = 0.0, s0l = 0.0, s1l = 0.0;  // low parts (double-double)
    const size_t row = (size_t)(2 * m + t);
    const double *v0p = a.start_val + row * 2 * a.np;
    const double *v1p = SPLIT ? a.start_d + row * a.n_pole_pad : v0p + a.np;
    double s0[R], s1[R];
#pragma unroll
    for (int r = 0; r < R; r++) {  // groups past the last repeat it and never start
        const int g = min(g0 + r, gend - 1), k = g * kLanes + lane;
        sid[r] = a.start_idx[row * a.np + k] | (g0 + r < gend ? 0 : kDead);
        x[r] = SPLIT ? a.s2[k] : a.z2_hi[k];
        s0[r] = v0p[k];
        s1[r] = v1p[k];
        if constexpr (DD) {
            xl = a.z2_lo[k];
            s0l = a.start_lo[row * 2 * a.n_dd_pad + k];
            s1l = a.start_lo[(row * 2 + 1) * a.n_dd_pad + k];
        }
        lo = min(lo, a.grp_lo[(size_t)m * a.ng + g]);
        hi = max(hi, a.grp_hi[(size_t)m * a.ng + g]);
        P0[r] = P1[r] = 0.0;
#pragma unroll
        for (int c = 0; c < NC; c++) acc[r][c] = 0.0;
    }

    if (lo < n) {
        // this lane's staged values: rows lane / CW (+ 64 / CW per e) of a
        // chunk, component lane % CW, of rows clamped to the last.  The loads are unconditional (a
        // select on them would become a branch that waits for memory); rows
        // past the last are overwritten with zeros in LDS.
        const int comp = lane % CW;
        const bool is_a = comp < NC;
        const double *base;
        unsigned stride;
        if (is_a) {
            base = a.alm + 2 * (((size_t)m * (2 * L + 3 - m) / 2 + t) * a.nmaps + a.map0) + comp;
            stride = 4u * (unsigned)a.nmaps;
        } else {
            const int ci = min(max(comp - CB, 0), leg_coefs(K) - 1);
            if constexpr (DD)
                base = ci < 3 ? a.coef_hi + ci : a.coef_lo + (ci - 3);
            else
                base = (SPLIT ? a.coef_pole : a.coef_sc) + ci;
            base += 4 * (a.coef_off[m] + t + 2);
            stride = 8u;
        }
        // factor of a staged value: f_l, or 1 for a coefficient and in double-double
        const double f1 = is_a ? 1.0 : 0.0, f0 = 1.0 - f1;
        const double *fb = reinterpret_cast<const double *>(cf) + 2;
        double pre[E], fac[E];
        auto fetch = [&](int c) {  // rows c .. c + kChunk - 1
#pragma unroll
            for (int e = 0; e < E; e++) {
                const unsigned i = (unsigned)min(c + (lane + 64 * e) / CW, n - 1);
                pre[e] = base[(size_t)i * stride];
                if constexpr (!DD) fac[e] = fb[8 * i];
            }
        };
        auto stage = [&](int sl, int c) {  // rows c .. c + kChunk - 1
#pragma unroll
            for (int e = 0; e < E; e++) {
                if constexpr (DD)
                    stg[sl * CS + lane + 64 * e] = pre[e];
                else
                    stg[sl * CS + lane + 64 * e] = pre[e] * __builtin_fma(fac[e], f1, f0);
            }
            if (c + kChunk > n) {
#pragma unroll
                for (int e = 0; e < E; e++)
                    if (c + (lane + 64 * e) / CW >= n) stg[sl * CS + lane + 64 * e] = 0.0;
            }
        };
        auto step = [&](auto first, double rv, double rc) {  // first: the row's first lane
            constexpr int C0 = decltype(first)::value;
            const double c0 = row_bcast<C0 + CO>(rc), c1 = row_bcast<C0 + CO + 1>(rc);
            const double c2 = leg_coefs(K) > 2 ? row_bcast<(C0 + CO + 2) % 16>(rc) : 0.0;
#pragma unroll
            for (int r = 0; r < R; r++) {
                fmac_row_bcast<NC, C0>(acc[r], rv, P0[r]);
                if constexpr (DD) {  // B, AB and G of App. A.2, high and low parts
                    const double l0 = row_bcast<(C0 + CO + 3) % 16>(rc), l1 = row_bcast<(C0 + CO + 4) % 16>(rc);
                    const double l2 = row_bcast<(C0 + CO + 5) % 16>(rc);
                    const dd A = dd_add_raw(dd_mul_raw({x[r], xl}, {c0, l0}), {c1, l1});
                    const dd y = dd_add_raw(dd_mul_raw(A, {P1[r], P1l}), dd_mul_raw({c2, l2}, {P0[r], P0l}));
                    const dd nx = fast_two_sum(y.h, y.l);
                    P0[r] = P1[r];
                    P0l = P1l;
                    P1[r] = nx.h;
                    P1l = nx.l;
                } else if constexpr (SPLIT) {  // c0 = h, c1 = -b (both of the next l), c2 = r
                    const double nx = __builtin_fma(c2, P0[r], P1[r]);
                    P1[r] = __builtin_fma(c0, P1[r], (c1 * x[r]) * nx);
                    P0[r] = nx;
                } else {
                    const double nx = __builtin_fma(__builtin_fma(x[r], c0, c1), P1[r], -P0[r]);
                    P0[r] = P1[r];
                    P1[r] = nx;
                }
            }
        };
        fetch(lo);
        // start values (in the scaled variables, or in two parts) wait in LDS until their chain joins
        double2 *starts = reinterpret_cast<double2 *>(room);
#pragma unroll
        for (int r = 0; r < R; r++) {
            if constexpr (DD) {
                starts[lane] = make_double2(s0[r], s1[r]);
                starts[64 + lane] = make_double2(s0l, s1l);
            } else {
                const int i = sid[r] >= kDead ? 0 : sid[r];
                starts[r * 64 + lane] = make_double2(s0[r] * cf[2 * i].w, SPLIT ? s1[r] : s1[r] * cf[2 * i + 2].w);
            }
        }
        stage(0, lo);
        fetch(lo + kChunk);
        if constexpr (DD) __builtin_amdgcn_s_setprio(3);  // a long serial chain among short ones
        int sl = 0;
        for (int c = lo; c < n; c += kChunk, sl ^= 1) {
            if (c <= hi) {
#pragma unroll
                for (int r = 0; r < R; r++)
                    if (sid[r] == c) {
                        const double2 s = starts[r * 64 + lane];
                        P0[r] = s.x;
                        P1[r] = s.y;
                        if constexpr (DD) {
                            const double2 sw = starts[64 + lane];
                            P0l = sw.x;
                            P1l = sw.y;
                        }
                    }
            }
            const double *cur = stg + sl * CS + (lane & 15);
#pragma unroll
            for (int u0 = 0; u0 < kChunk; u0 += KU) {
                double rv[KU / PK], rc[KU / PK];
#pragma unroll
                for (int u = 0; u < KU / PK; u++) {
                    rv[u] = cur[(u0 + PK * u) * CW];
                    rc[u] = CW <= 16 ? rv[u] : cur[(u0 + PK * u) * CW + 16];
                }
#pragma unroll
                for (int u = 0; u < KU / PK; u++) {
                    step(std::integral_constant<int, 0>{}, rv[u], rc[u]);
                    if constexpr (PK == 2) step(std::integral_constant<int, 8>{}, rv[u], rc[u]);
                }
            }
            stage(sl ^ 1, c + kChunk);
            fetch(c + 2 * kChunk);
        }
        if constexpr (DD) __builtin_amdgcn_s_setprio(0);
    }

    // fused even/odd fold and store (Eqs. 13-14), one ring group at a time:
    // wave 0 stores the north rings, wave 1 their mirrors
    const double *other = lds + (1 - t) * W;
#pragma unroll
    for (int r = 0; r < R; r++) {
        if (g0 + r >= gend) break;
        if (r) __syncthreads();  // the previous group has been read
#pragma unroll
        for (int c = 0; c < NC; c++) room[c * 64 + lane] = acc[r][c];
        __syncthreads();
        const int k = (g0 + r) * kLanes + lane, ks = a.nrings - 1 - k;
        if (k >= a.n_north || (t && ks == k)) continue;
        double2 *q = reinterpret_cast<double2 *>(a.q) + ((size_t)(t ? ks : k) * (L + 1) + m) * a.nmaps + a.map0;
#pragma unroll
        for (int b = 0; b < NB; b++) {
            const double ore = other[(2 * b) * 64 + lane], oim = other[(2 * b + 1) * 64 + lane];
            double2 v = t ? make_double2(ore - acc[r][2 * b], oim - acc[r][2 * b + 1])
                          : make_double2(acc[r][2 * b] + ore, acc[r][2 * b + 1] + oim);
            if (m == 0) v.y = 0.0;  // real field: Im a_l0 is ignored
            q[b] = v;
        }
    }
}

// The block of work rb of an order: double-double groups first (one each),
// then split ones (R groups each, the last block partial), then the plain ones.
template <int NB, int R, bool DD>
__device__ __forceinline__ void leg_item(const LegArgs &a, const int m, int rb, double *lds) {
    constexpr int W = leg_wave_lds<NB, R, DD>();
    if constexpr (DD) {
        if (rb < a.dd_groups) return leg_block<NB, 1, Chain::DD, W>(a, m, rb, rb + 1, lds);
        rb -= a.dd_groups;
    }
    if (rb < a.pole_blocks)
        leg_block<NB, R, Chain::SPLIT, W>(a, m, rb * R, a.pole_groups, lds);
    else
        leg_block<NB, R, Chain::PLAIN, W>(a, m, a.first_plain + (rb - a.pole_blocks) * R, a.ng, lds);
}

// One launch covers every (m, ring block), in the order of xcd_order().  DD: for
// plans with double-double groups (its registers and LDS would cost the one
// ring a lane kernels of the others a fifth of their wavefronts).
template <int NB, int R, bool DD>
__global__ __launch_bounds__(128, (R == 4 ? 4 : 1)) void k_legendre(LegArgs a) {
    __shared__ __attribute__((aligned(16))) double lds[2 * leg_wave_lds<NB, R, DD>()];
    const int nrb = a.dd_groups + a.pole_blocks + a.plain_blocks;
    const int slot = blockIdx.x >> 3, s = slot / nrb;
    const int m = xcd_order(blockIdx.x & 7, s);
    if (m > a.L) return;
    // an XCD deals its workgroups to its shader engines round robin: the
    // first block of each order moves on by one, so that no engine gets the
    // same (long or short) ring blocks of every order
    leg_item<NB, R, DD>(a, m, (slot + s) % nrb, lds);
}

// Rings per lane of a pass of nb maps: the plan's choice, or by the number
// of wavefronts at one ring per lane.  More rings per lane share a step's
// operand reads, but cut the number of wavefronts and run a lane's rings from
// the earliest of their chains.  Measured at 1, 2 and 4 rings, four maps:
// L = 255 (2048 wavefronts) 12.0, 14.6, 22.4 us; L = 511 (8192) 41, 39, 69 us;
// L = 767 (18432) 106, 97, 122 us; L = 1023 (32768) 223, 193, 220 us; L = 2047
// (131072) -, 1329, 1352 us; one map: L = 1023 132, 113, 124 us, L = 2047 -, 764,
// 750 us.  Above two maps the state of four rings leaves too few wavefronts.
static int leg_rings(const sht_plan_s *p, int nb) {
    int R = p->opts.rings_per_lane;
    if (R != 1 && R != 2 && R != 4) {
        const long long waves = 2LL * (p->L + 1) * (p->n_north_pad / kLanes);
        R = waves >= 65536 && nb <= 2 ? 4 : waves >= 8192 ? 2 : 1;
    }
    return nb > 4 ? std::min(R, 2) : R;
}

// Maps of the next pass with `left` maps to go.
int leg_pass_maps(int left) { return left >= 8 ? 8 : left == 7 ? 4 : left; }

template <int NB, int R>
static hipError_t launch_nbr(const sht_plan_s *p, LegArgs a, hipStream_t st) {
    const long long grid = (long long)((p->L + 64) / 64 * 64) * (a.dd_groups + a.pole_blocks + a.plain_blocks);
    if (grid <= 0) return hipSuccess;
    if (a.dd_groups > 0) hipLaunchKernelGGL((k_legendre<NB, R, true>), dim3((unsigned)grid), dim3(128), 0, st, a);
    else hipLaunchKernelGGL((k_legendre<NB, R, false>), dim3((unsigned)grid), dim3(128), 0, st, a);
    return hipGetLastError();
}

template <int NB>
static hipError_t launch_nb(const sht_plan_s *p, const LegArgs &a, int R, hipStream_t st) {
    if constexpr (NB <= 4) {
        if (R == 4) return launch_nbr<NB, 4>(p, a, st);
    }
    return R == 1 ? launch_nbr<NB, 1>(p, a, st) : launch_nbr<NB, 2>(p, a, st);
}

// Persistent form for batches of requests (the many-transform regime of
// Sec. 3.4): one launch per pass shape (workgroups of 8, 6, 5, 4, 3, 2 or 1
// maps) for every request of a batch, so that each launch runs one specialised
// body at its own occupancy.  Work items {pass, m, ring block, 0} of one shape come in eight lists,
// one per XCD (the items of one pass and order share a list, so that XCD's L2
// serves the order's coefficient and a_lm stream to all of them), each sorted
// longest first and cut into chunks that shrink along the list.  A workgroup
// takes chunks from its own XCD's list through a device counter (a
// vector-memory atomic) and, once that list is exhausted, from the others in
// turn; it leaves when every counter has passed the end of its list, so every
// workgroup reaches the exit.  The bodies are k_legendre's.
constexpr int kQueueLists = 8;
constexpr int kQueueStride = 16;  // counters 64 bytes apart

__global__ void k_queue_reset(unsigned *c) {
    if (blockIdx.x == 0)
        for (int i = threadIdx.x; i < kQueueShapes * kQueueLists; i += blockDim.x) c[i * kQueueStride] = 0u;
}

template <int NB, int R, bool DD>
__global__ __launch_bounds__(128) void k_legendre_queue(const LegArgs *__restrict__ passes,
                                                        const int4 *__restrict__ items,
                                                        const unsigned *__restrict__ chunk_off,
                                                        const unsigned *__restrict__ list_off,
                                                        unsigned *__restrict__ counter) {
    __shared__ __attribute__((aligned(16))) double lds[2 * leg_wave_lds<NB, R, DD>()];
    __shared__ unsigned taken;
    const int home = blockIdx.x & (kQueueLists - 1);  // workgroups are dealt to the XCDs round robin
    for (int s = 0; s < kQueueLists; s++) {
        const int x = (home + s) & (kQueueLists - 1);
        const unsigned lo = list_off[x], cnt = list_off[x + 1] - lo;
        for (;;) {
            __syncthreads();  // the previous item has left the LDS, and every thread has read `taken`
            if (threadIdx.x == 0) taken = atomicAdd(counter + x * kQueueStride, 1u);
            __syncthreads();
            const unsigned c = __builtin_amdgcn_readfirstlane(taken);
            if (c >= cnt) break;
            const unsigned i0 = chunk_off[lo + c], i1 = chunk_off[lo + c + 1];
            for (unsigned i = i0; i < i1; i++) {
                const int4 w = items[i];
                const int pi = __builtin_amdgcn_readfirstlane(w.x), m = __builtin_amdgcn_readfirstlane(w.y);
                const LegArgs a = passes[pi];
                if (i != i0) __syncthreads();  // the previous item has left the LDS
                leg_item<NB, R, DD>(a, m, __builtin_amdgcn_readfirstlane(w.z), lds);
            }
        }
    }
}

typedef void (*QueueKernel)(const LegArgs *, const int4 *, const unsigned *, const unsigned *, unsigned *);

template <int R, bool DD>
static QueueKernel queue_kernel_r(int shape) {
    constexpr int R2 = R < 2 ? R : 2;
    switch (shape) {
        case 0: return k_legendre_queue<8, R2, DD>;
        case 1: return k_legendre_queue<6, R2, DD>;
        case 2: return k_legendre_queue<5, R2, DD>;
        case 3: return k_legendre_queue<4, R, DD>;
        case 4: return k_legendre_queue<3, R, DD>;
        case 5: return k_legendre_queue<2, R, DD>;
        default: return k_legendre_queue<1, R, DD>;
    }
}

template <bool DD>
static QueueKernel queue_kernel_d(int shape, int R) {
    switch (R) {
        case 1: return queue_kernel_r<1, DD>(shape);
        case 4: return queue_kernel_r<4, DD>(shape);
        default: return queue_kernel_r<2, DD>(shape);
    }
}

static QueueKernel queue_kernel(int shape, int R, bool dd) {
    return dd ? queue_kernel_d<true>(shape, R) : queue_kernel_d<false>(shape, R);
}

int queue_shape(int nb) { return nb >= 8 ? 0 : 7 - nb; }
int queue_rings(int nb, int R) { return nb > 4 ? std::min(R, 2) : R; }

// Workgroups of the persistent launch of one shape: as many as the current
// device keeps resident at once.
hipError_t legendre_queue_grid(int shape, int rings_per_lane, bool dd, int *grid) {
    int dev = 0, cus = 0, per_cu = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e == hipSuccess) e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
    if (e == hipSuccess)
        e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, (const void *)queue_kernel(shape, rings_per_lane, dd),
                                                         kQueueThreads, 0);
    *grid = std::max(std::max(per_cu, 1) * std::max(cus, 1) / kQueueLists, 1) * kQueueLists;
    return e;
}

hipError_t launch_queue_reset(unsigned *counter, hipStream_t st) {
    hipLaunchKernelGGL(k_queue_reset, dim3(1), dim3(64), 0, st, counter);
    return hipGetLastError();
}

hipError_t launch_legendre_queue(int shape, const LegArgs *passes, const int4 *items, const unsigned *chunk_off,
                                 const unsigned *list_off, unsigned *counter, int rings_per_lane, bool dd, int grid,
                                 hipStream_t st) {
    if (shape < 0 || shape >= kQueueShapes || grid < 0) return hipErrorInvalidValue;
    if (grid == 0) return hipSuccess;  // no items of this shape
    hipLaunchKernelGGL(queue_kernel(shape, rings_per_lane, dd), dim3((unsigned)grid), dim3(kQueueThreads), 0, st,
                       passes, items, chunk_off, list_off + shape * (kQueueLists + 1),
                       counter + shape * kQueueLists * kQueueStride);
    return hipGetLastError();
}

// Argument block of one pass (maps map0 .. map0 + nb - 1 of nmaps) for
// R rings per lane.
LegArgs leg_args(const sht_plan_s *p, int nmaps, int map0, int R, const double *alm, double *q) {
    LegArgs a;
    a.z2_hi = p->d_z2_hi;
    a.z2_lo = p->d_z2_lo;
    a.s2 = p->d_s2;
    a.coef_off = p->d_coef_off;
    a.coef_hi = p->d_coef_hi;
    a.coef_lo = p->d_coef_lo;
    a.coef_pole = p->d_coef_pole;
    a.coef_sc = p->d_coef_sc;
    a.start_idx = p->d_start_idx;
    a.start_val = p->d_start_val;
    a.start_lo = p->d_start_lo;
    a.start_d = p->d_start_d;
    a.grp_lo = p->d_grp_lo;
    a.grp_hi = p->d_grp_hi;
    a.alm = alm;
    a.q = q;
    a.L = p->L;
    a.nrings = p->nrings;
    a.n_north = p->n_north;
    a.np = p->n_north_pad;
    a.n_dd_pad = std::max(p->n_dd_pad, 1);
    a.n_pole_pad = std::max(p->pole_groups, 1) * kLanes;
    a.ng = p->n_north_pad / kLanes;
    a.nmaps = nmaps;
    a.map0 = map0;
    a.pole_groups = p->pole_groups;
    a.dd_groups = p->pole_groups > 0 ? 0 : p->n_dd_groups;
    a.first_plain = a.pole_groups + a.dd_groups;
    a.pole_blocks = (a.pole_groups + R - 1) / R;
    a.plain_blocks = (a.ng - a.first_plain + R - 1) / R;
    return a;
}

hipError_t launch_legendre(const sht_plan_s *p, int nmaps, const double *alm, double *q,
                           hipStream_t stream) {
    hipError_t e = hipSuccess;
    for (int b = 0; b < nmaps && e == hipSuccess;) {
        const int nb = leg_pass_maps(nmaps - b), R = leg_rings(p, nb);
        const LegArgs a = leg_args(p, nmaps, b, R, alm, q);
        switch (nb) {
            case 8: e = launch_nb<8>(p, a, R, stream); break;
            case 6: e = launch_nb<6>(p, a, R, stream); break;
            case 5: e = launch_nb<5>(p, a, R, stream); break;
            case 4: e = launch_nb<4>(p, a, R, stream); break;
            case 3: e = launch_nb<3>(p, a, R, stream); break;
            case 2: e = launch_nb<2>(p, a, R, stream); break;
            default: e = launch_nb<1>(p, a, R, stream); break;
        }
        b += nb;
    }
    return e;
}

// ---- tables of the scaled and the split recurrence, made once per plan ------
// With D = ((l+1)^2 - m^2)((l+2)^2 - m^2) and Q_l = sqrt((2l+5) / ((2l+1) D)):
//   beta_l = 1 / c_l = (2l+3)(2l+1) Q_l,  r_l = (l+1+m)(l+2+m) Q_l,
//   h_l = (l-m)(l-1-m) (2l+3)/(2l-1) Q_l.
__device__ __forceinline__ dd pole_Q(double l, double m) {
    const dd D = dd_mul({(l + 1 - m) * (l + 1 + m), 0.0}, {(l + 2 - m) * (l + 2 + m), 0.0});
    return dd_sqrt(dd_div({2 * l + 5, 0.0}, dd_mul({2 * l + 1, 0.0}, D)));
}

// v rounded to double with the rounding error of the entries before it in the
// chain added, which it passes on: the errors of a table's entries sum to less
// than one rounding.  A coefficient's error shifts the chain's phase from there
// on, so independent errors add up like sqrt(l), these do not.
__device__ __forceinline__ double round_carry(dd v, double &carry) {
    const dd t = dd_add(v, {carry, 0.0});
    carry = t.l;
    return t.h;
}

// Scaled recurrence: entry e = l - m of order m holds {b_l, -b_l d_l, f_l,
// 1 / f_l}; one thread per order and parity follows the product of the c_l in
// double-double.  The product fixes f_{l+2} f_l = 1 / c_l only; the first value
// is chosen so that the last two are equal (a first pass finds the ratio), which
// lets f_l run smoothly towards 2 and b_l towards 4, as the carried rounding
// needs (f_m = 2 would make them alternate by a factor of m).  Near the equator,
// the recurrence's double root, these errors decide: the phases of rings there
// were off by 1.62e-14 (L = 1023, relative rms, red spectrum) and 2.99e-14 (L =
// 2047) with f_m = 2 and plain rounding, 1.34e-14 and 2.55e-14 by the unscaled
// recurrence.
__device__ __forceinline__ dd scaled_next(double l, double m, dd f) {
    // 1 / c_l = (2l+3) sqrt((2l+1)(2l+5) / D) = (2l+3)(2l+1) Q_l
    return dd_div(dd_mul({(2 * l + 3) * (2 * l + 1), 0.0}, pole_Q(l, m)), f);
}
__global__ __launch_bounds__(64) void k_scaled_coef(const long long *__restrict__ coef_off, double4 *__restrict__ out,
                                                    int rows) {
    const int row = blockIdx.x * 64 + threadIdx.x;
    if (row >= rows) return;
    const int m = row >> 1, t = row & 1;
    const long long base = coef_off[m], cnt = coef_off[m + 1] - base;
    const double mm = m;
    const int n = (int)((cnt - t + 1) / 2);  // entries of this parity (a dozen past L at least)
    dd f = {2.0, 0.0};
    double ratio = 1.0;
    for (int k = 0; k < n - 1; k++) {
        const dd nx = scaled_next(mm + t + 2.0 * k, mm, f);
        ratio = nx.h / f.h;
        f = nx;
    }
    f = {(n & 1) ? 2.0 / sqrt(ratio) : 2.0 * sqrt(ratio), 0.0};
    double cb = 0.0, ca = 0.0;
    for (int k = 0; k < n; k++) {
        const double l = mm + t + 2.0 * k;
        const dd b = dd_mul(f, f);
        const dd d = dd_div({2 * l * (l + 1) - 2 * mm * mm - 1, 0.0}, {(2 * l - 1) * (2 * l + 3), 0.0});
        out[base + t + 2 * k] =
            make_double4(round_carry(b, cb), round_carry(dd_neg(dd_mul(b, d)), ca), f.h, 1.0 / f.h);
        f = scaled_next(l, mm, f);
    }
}

hipError_t fill_scaled_coef(const sht_plan_s *p) {
    const int rows = 2 * (p->L + 1);
    hipLaunchKernelGGL(k_scaled_coef, dim3((unsigned)((rows + 63) / 64)), dim3(64), 0, nullptr, p->d_coef_off,
                       reinterpret_cast<double4 *>(p->d_coef_sc), rows);
    hipError_t e = hipGetLastError();
    return e != hipSuccess ? e : hipStreamSynchronize(nullptr);
}

// Split recurrence in the scaled variables (P~_l = f_l mu_l, d_l of the pair
// (l, l+2) scaled like P~_{l+2}): entry e holds {h_l f_l / f_{l+2},
// -beta_l f_l / f_{l+2}, r_{l-2} f_{l-2} / f_l, 0}, with carried rounding; entries
// 0 and 1 are not used.
__global__ __launch_bounds__(64) void k_pole_coef(const long long *__restrict__ coef_off,
                                                  const double4 *__restrict__ sc, double4 *__restrict__ out, int rows) {
    const int row = blockIdx.x * 64 + threadIdx.x;
    if (row >= rows) return;
    const int m = row >> 1;
    const long long base = coef_off[m], cnt = coef_off[m + 1] - base;
    double ch = 0.0, cb = 0.0, cr = 0.0;
    for (long long e = row & 1; e < cnt; e += 2) {
        double4 v = make_double4(0.0, 0.0, 0.0, 0.0);
        if (e >= 2 && e + 2 < cnt) {
            const double l = (double)(m + e), mm = m;
            const dd Qf = dd_mul(pole_Q(l, mm), dd_div({sc[base + e].z, 0.0}, {sc[base + e + 2].z, 0.0}));
            v.x = round_carry(dd_mul(dd_div(dd_mul({(l - mm) * (l - 1 - mm), 0.0}, {2 * l + 3, 0.0}), {2 * l - 1, 0.0}), Qf), ch);
            v.y = round_carry(dd_neg(dd_mul({(2 * l + 3) * (2 * l + 1), 0.0}, Qf)), cb);
            v.z = round_carry(dd_mul(dd_mul({(l - 1 + mm) * (l + mm), 0.0}, pole_Q(l - 2, mm)),
                                     dd_div({sc[base + e - 2].z, 0.0}, {sc[base + e].z, 0.0})), cr);
        }
        out[base + e] = v;
    }
}

// (P~_{l+2} - r_l P~_l) / f_{l+2} at each chain's start, l = m + t + 2 start_idx,
// from the stored start values (with their low parts on the first n_dd_pad
// rings; farther from the pole the difference no longer cancels).
__global__ __launch_bounds__(256) void k_pole_start(LegArgs a, double *__restrict__ out) {
    const int row = blockIdx.x, m = row >> 1, t = row & 1;
    const double4 *sc = reinterpret_cast<const double4 *>(a.coef_sc) + a.coef_off[m] + t;
    for (int k = threadIdx.x; k < a.n_pole_pad; k += 256) {
        const int i = a.start_idx[(size_t)row * a.np + k];
        double d = 0.0;
        if (i < kDead) {
            const size_t r2 = (size_t)row * 2;
            dd p0 = {a.start_val[r2 * a.np + k], 0.0}, p1 = {a.start_val[(r2 + 1) * a.np + k], 0.0};
            if (k < a.n_dd_pad) {
                p0.l = a.start_lo[r2 * a.n_dd_pad + k];
                p1.l = a.start_lo[(r2 + 1) * a.n_dd_pad + k];
            }
            const double l = m + t + 2.0 * i;
            const dd r = dd_mul({(l + 1 + m) * (l + 2 + m), 0.0}, pole_Q(l, m));
            d = dd_div(dd_sub(p1, dd_mul(r, p0)), {sc[2 * i + 2].z, 0.0}).h;
        }
        out[(size_t)row * a.n_pole_pad + k] = d;
    }
}

hipError_t fill_pole_tables(const sht_plan_s *p) {
    const int rows = 2 * (p->L + 1);
    hipLaunchKernelGGL(k_pole_coef, dim3((unsigned)((rows + 63) / 64)), dim3(64), 0, nullptr, p->d_coef_off,
                       reinterpret_cast<const double4 *>(p->d_coef_sc), reinterpret_cast<double4 *>(p->d_coef_pole), rows);
    const LegArgs a = leg_args(p, 1, 0, 1, nullptr, nullptr);
    hipLaunchKernelGGL(k_pole_start, dim3((unsigned)(2 * (p->L + 1))), dim3(256), 0, nullptr, a, p->d_start_d);
    hipError_t e = hipGetLastError();
    return e != hipSuccess ? e : hipStreamSynchronize(nullptr);
}

}  // namespace sht
