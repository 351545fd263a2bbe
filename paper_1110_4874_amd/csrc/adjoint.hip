// Adjoint Legendre transform, for gfx950: the transpose of the Legendre
// phase of Sec. 2.4 Eq. 12 (the paper's backward Legendre transform of
// Sec. 3 Eq. 18 without quadrature weights), with the even/odd ring
// symmetry of Eqs. 13-14 applied in reverse:
//
//   g_lm = sum_{north k} P~_l^m(z_k) ybar^t_m(z_k),   t = (l - m) mod 2,
//   ybar^even(z) = ybar(z) + ybar(-z),  ybar^odd(z) = ybar(z) - ybar(-z)
//
// (the equator ring counts once).  The recurrence runs along l for every
// ring, but the outputs are indexed by l and summed over rings.  One
// workgroup owns one order m and parity t and all rings; each wave runs the
// scaled (near the poles: split) two-step recurrence of legendre.hip for
// 64 R rings and the sum over rings is a matrix product on the matrix cores
// (k_legendre_adj).  Rings that run in double-double (plans that set dd_sin)
// have their own launch, which writes g before the others add to it
// (k_legendre_adj_dd).  Every sum runs in a fixed order: deterministic, no
// atomics, no partial-sum workspace.
#include "ddmath.h"
#include "dpp.h"
#include "internal.h"

namespace sht {

struct AdjArgs {
    const double *__restrict__ z2_hi;
    const double *__restrict__ z2_lo;
    const double *__restrict__ s2;
    const long long *__restrict__ coef_off;
    const double *__restrict__ coef_hi;
    const double *__restrict__ coef_lo;
    const double *__restrict__ coef_sc;
    const double *__restrict__ coef_pole;
    const int *__restrict__ start_idx;
    const double *__restrict__ start_val;
    const double *__restrict__ start_lo;
    const double *__restrict__ start_d;
    const int *__restrict__ grp_lo;
    const int *__restrict__ grp_hi;
    const double2 *__restrict__ ybar;  // [ring][m][nmaps]
    double *__restrict__ g;            // [nalm][nmaps] complex
    int L, nrings, n_north, np, n_dd_pad, n_pole_pad, ng;
    int nmaps, map0, nb;  // maps map0 .. map0 + nb - 1 of nmaps
    int pole_groups;      // groups run by the split recurrence
    int first_group, end_group;  // 64-ring groups summed by a k_legendre_adj launch
    int k0, k1;           // double-double rings [k0, k1) of a k_legendre_adj_dd launch
    int accumulate;       // 0: write g, 1: add to g
};

// Lane shuffle of a double within a row of 16 lanes (DPP control CTRL).
template <int CTRL>
__device__ __forceinline__ double dpp_d(double v) {
    const long long x = __builtin_bit_cast(long long, v);
    const int lo = __builtin_amdgcn_update_dpp(0, (int)x, CTRL, 0xF, 0xF, false);
    const int hi = __builtin_amdgcn_update_dpp(0, (int)(x >> 32), CTRL, 0xF, 0xF, false);
    return __builtin_bit_cast(double, ((long long)hi << 32) | (long long)(unsigned)lo);
}

// Sum over each row of 16 lanes, every lane of the row receiving the total:
// pairs, quads, mirrored quads, mirrored halves.  Partners add the same two
// numbers, so the result is the same in every lane.
__device__ __forceinline__ double row16_sum(double v) {
    v += dpp_d<0xB1>(v);   // quad_perm [1,0,3,2]
    v += dpp_d<0x4E>(v);   // quad_perm [2,3,0,1]
    v += dpp_d<0x141>(v);  // row_half_mirror
    v += dpp_d<0x140>(v);  // row_mirror
    return v;
}

__device__ __forceinline__ int wave_min(int v) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v = min(v, __shfl_xor(v, off, 64));
    return v;
}

// Double-double rings: one workgroup per order, 256 threads with one ring
// each, both parities, NB maps per pass.  A group of G chain
// steps (G * 4 * NB = 16 outputs) is written to one of two LDS buffers as
// per-thread partial sums red[G][4*NB][T]; after one barrier, 16 lanes per
// output add 16 partials each and finish with a 16-lane DPP tree, while the
// next group fills the other buffer.  Outputs already in g (accumulating
// launches) are fetched one group ahead.  The recurrence coefficients of the
// order stream through LDS in blocks of kAdjCB steps, each block fetched from
// memory two blocks ahead of its use, so that the chain never waits on HBM.
constexpr int kAdjCB = 32;  // chain steps per LDS coefficient block

template <int NB>
__global__ __launch_bounds__(256) void k_legendre_adj_dd(AdjArgs a) {
    constexpr int T = 256, R = 1;  // the reduction maps 16 outputs x 16 slices onto 256 threads
    constexpr int NV = 4 * NB;     // (parity, map, re/im) components per step
    constexpr int G = 16 / NV;     // chain steps per LDS group
    constexpr int SL = T / 16;     // partial-sum slices per output
    constexpr int PS = T / SL;     // partials added by one slice
    constexpr int CW = 8;          // doubles per step and table: even B, AB, G, pad, odd B, AB, G, pad
    constexpr int CE = kAdjCB * CW / T;  // table entries per thread and block
    static_assert(kAdjCB % G == 0 && kAdjCB > G && CE >= 1, "coefficient block shape");
    extern __shared__ double red[];
    constexpr int GO = kAdjCB / G * 16;  // outputs per coefficient block
    static_assert(GO <= T, "one staged output per thread");
    __shared__ double cbuf[2][2 * kAdjCB * CW];
    __shared__ double gbuf_acc[2][GO];  // outputs already in g, for accumulating launches
    const int m = blockIdx.x;
    const int tid = threadIdx.x, lane = tid & 63;
    const int L = a.L;
    const int n0 = (L - m) / 2 + 1;
    const int n1 = (L - m >= 1) ? (L - m - 1) / 2 + 1 : 0;
    const size_t aoff = (size_t)m * (2 * L + 3 - m) / 2;

    // chain range over the groups of this launch's rings
    __shared__ int s_lo, s_hi;
    if (tid == 0) {
        int lo = kDead, hi = -1;
        for (int gr = a.k0 / kLanes; gr < (a.k1 + kLanes - 1) / kLanes; gr++) {
            lo = min(lo, a.grp_lo[(size_t)m * a.ng + gr]);
            hi = max(hi, a.grp_hi[(size_t)m * a.ng + gr]);
        }
        s_lo = lo;
        s_hi = hi;
    }
    __syncthreads();
    const int lo = s_lo, hi = s_hi;

    auto gaddr = [&](int l, int b, int ri) { return a.g + 2 * ((aoff + l - m) * a.nmaps + a.map0 + b) + ri; };

    if (lo >= n0) {  // every chain of these rings stays below the cutoff
        if (!a.accumulate)
            for (int e = tid; e < (L - m + 1) * NB * 2; e += T) *gaddr(m + e / (NB * 2), (e / 2) % NB, e % 2) = 0.0;
        return;
    }

    int k[R];
    bool val[R];
    double z2h[R], z2l[R];
    int sid[R][2];
    dd st0[R][2], st1[R][2], p0[R][2], p1[R][2];
    double yer[R][NB], yei[R][NB], yor[R][NB], yoi[R][NB];
    int wlo = kDead;
#pragma unroll
    for (int r = 0; r < R; r++) {
        k[r] = a.k0 + tid * R + r;
        val[r] = k[r] < a.k1 && k[r] < a.n_north;
        const int kk = val[r] ? k[r] : a.k0;
        z2h[r] = a.z2_hi[kk];
        z2l[r] = a.z2_lo[kk];
#pragma unroll
        for (int t = 0; t < 2; t++) {
            const size_t row = (size_t)(2 * m + t);
            sid[r][t] = val[r] ? a.start_idx[row * a.np + kk] : kDead;
            wlo = min(wlo, sid[r][t]);
            st0[r][t].h = a.start_val[(row * 2 + 0) * a.np + kk];
            st1[r][t].h = a.start_val[(row * 2 + 1) * a.np + kk];
            st0[r][t].l = a.start_lo[(row * 2 + 0) * a.n_dd_pad + kk];
            st1[r][t].l = a.start_lo[(row * 2 + 1) * a.n_dd_pad + kk];
            p0[r][t] = {0.0, 0.0};
            p1[r][t] = {0.0, 0.0};
        }
        // unfold the ring and its mirror into even/odd parts
        const int ks = a.nrings - 1 - kk;
        const double2 *yn = a.ybar + ((size_t)kk * (a.L + 1) + m) * a.nmaps + a.map0;
        const double2 *ys = a.ybar + ((size_t)ks * (a.L + 1) + m) * a.nmaps + a.map0;
#pragma unroll
        for (int b = 0; b < NB; b++) {
            double2 vn = val[r] ? yn[b] : make_double2(0.0, 0.0);
            double2 vs = (val[r] && ks != kk) ? ys[b] : make_double2(0.0, 0.0);
            yer[r][b] = vn.x + vs.x;
            yei[r][b] = vn.y + vs.y;
            yor[r][b] = vn.x - vs.x;
            yoi[r][b] = vn.y - vs.y;
        }
    }
    // first chain step at which any ring of this wave is alive
    wlo = __builtin_amdgcn_readfirstlane(wave_min(wlo));

    // coefficient blocks: block j holds chain steps lo + j*kAdjCB + s, s < kAdjCB,
    // as the table entries 2*step + 2 (even chain) and 2*step + 3 (odd chain);
    // steps past n0 are not fetched (the table is padded only a few steps)
    const long long cbase = a.coef_off[m];
    const double *__restrict__ chd = a.coef_hi + 4 * cbase;
    const double *__restrict__ cld = a.coef_lo + 4 * cbase;
    // staged outputs: thread tid < GO holds output tid % 16 of group tid / 16
    const int so = tid % 16, sv = so % NV, sg = so / NV;
    const int sb = sv / 4, st_ = (sv % 4) / 2, sri = sv % 2;
    const int snt = st_ == 0 ? n0 : n1;
    double creg[2][CE], greg = 0.0;
    auto fetch_block = [&](int j) {
        if (a.accumulate && tid < GO) {
            const int step = lo + j * kAdjCB + (tid / 16) * G + sg;
            greg = step < snt ? *gaddr(m + st_ + 2 * step, sb, sri) : 0.0;
        }
#pragma unroll
        for (int e = 0; e < CE; e++) {
            const int el = tid + e * T;
            const int step = lo + j * kAdjCB + el / CW;
            const size_t idx = (size_t)(2 * step + 2) * 4 + el % CW;
            creg[0][e] = step <= n0 ? chd[idx] : 0.0;
            creg[1][e] = step <= n0 ? cld[idx] : 0.0;
        }
    };
    auto stage_block = [&](int slot) {
#pragma unroll
        for (int e = 0; e < CE; e++) {
            cbuf[slot][tid + e * T] = creg[0][e];
            cbuf[slot][kAdjCB * CW + tid + e * T] = creg[1][e];
        }
        if (a.accumulate && tid < GO) gbuf_acc[slot][tid] = greg;
    };
    auto coef = [&](int i, double4 &e4, double4 &o4, double4 &el, double4 &ol) {
        const int j = (i - lo) / kAdjCB, s = (i - lo) % kAdjCB;
        const double4 *cb = reinterpret_cast<const double4 *>(&cbuf[j & 1][s * CW]);
        e4 = cb[0];
        o4 = cb[1];
        {
            const double4 *cbl = reinterpret_cast<const double4 *>(&cbuf[j & 1][kAdjCB * CW + s * CW]);
            el = cbl[0];
            ol = cbl[1];
        }
    };
    fetch_block(0);
    stage_block(0);
    fetch_block(1);
    __syncthreads();

    // reduction role of this thread: output (rg, rv) of a group, slice rs
    const int ro = tid / SL, rs = tid % SL;
    const int rg = ro / NV, rv = ro % NV;               // step in group, component
    const int rb = rv / 4, rt = (rv % 4) / 2, rri = rv % 2;
    const int nt = rt == 0 ? n0 : n1;


    double4 e4, o4, el = {0, 0, 0, 0}, ol = {0, 0, 0, 0};
    coef(lo, e4, o4, el, ol);

    // Steps run in groups of G without a break: the last group may run past
    // n0 (its extra partials are never stored, its coefficients are stale
    // but finite table or LDS values).  A group whose steps all precede the
    // first live chain of the wave (wlo and lo are multiples of kChunk, and
    // G divides kChunk) only writes zero partials; chains join at the first
    // step of a group.
    int buf = 0;
    for (int g0 = lo; g0 < n0; g0 += G, buf ^= 1) {
        double *gbuf = red + (size_t)buf * G * NV * T;
        double *rbuf = gbuf + tid;
        if (g0 + G <= wlo) {
#pragma unroll
            for (int v = 0; v < G * NV; v++) rbuf[v * T] = 0.0;
            coef(g0 + G, e4, o4, el, ol);
        } else {
            if ((g0 % kChunk) == 0 && g0 <= hi) {
#pragma unroll
                for (int r = 0; r < R; r++)
#pragma unroll
                    for (int t = 0; t < 2; t++)
                        if (sid[r][t] == g0) {
                            p0[r][t] = st0[r][t];
                            p1[r][t] = st1[r][t];
                        }
            }
#pragma unroll
            for (int u = 0; u < G; u++) {
                const int i = g0 + u;
                // coefficients of the next step
                double4 e4n, o4n, eln = el, oln = ol;
                coef(i + 1, e4n, o4n, eln, oln);
                // partial sums of this thread's rings: P(i) * ybar^t
                double pe_r[NB], pe_i[NB], po_r[NB], po_i[NB];
#pragma unroll
                for (int b = 0; b < NB; b++) pe_r[b] = pe_i[b] = po_r[b] = po_i[b] = 0.0;
#pragma unroll
                for (int r = 0; r < R; r++) {
                    const double pe = p0[r][0].h, po = p0[r][1].h;
#pragma unroll
                    for (int b = 0; b < NB; b++) {
                        pe_r[b] = __builtin_fma(pe, yer[r][b], pe_r[b]);
                        pe_i[b] = __builtin_fma(pe, yei[r][b], pe_i[b]);
                        po_r[b] = __builtin_fma(po, yor[r][b], po_r[b]);
                        po_i[b] = __builtin_fma(po, yoi[r][b], po_i[b]);
                    }
                }
                double *rs_ = rbuf + (size_t)u * NV * T;
#pragma unroll
                for (int b = 0; b < NB; b++) {
                    rs_[(4 * b + 0) * T] = pe_r[b];
                    rs_[(4 * b + 1) * T] = pe_i[b];
                    rs_[(4 * b + 2) * T] = po_r[b];
                    rs_[(4 * b + 3) * T] = po_i[b];
                }
                // advance the recurrence
                {
                    const dd Be = {e4.x, el.x}, ABe = {e4.y, el.y}, Ge = {e4.z, el.z};
                    const dd Bo = {o4.x, ol.x}, ABo = {o4.y, ol.y}, Go = {o4.z, ol.z};
#pragma unroll
                    for (int r = 0; r < R; r++) {
                        const dd z2 = {z2h[r], z2l[r]};
                        const dd Ae = dd_add(dd_mul(z2, Be), ABe);
                        const dd Ao = dd_add(dd_mul(z2, Bo), ABo);
                        const dd ne = dd_add(dd_mul(Ae, p1[r][0]), dd_mul(Ge, p0[r][0]));
                        const dd no = dd_add(dd_mul(Ao, p1[r][1]), dd_mul(Go, p0[r][1]));
                        p0[r][0] = p1[r][0];
                        p1[r][0] = ne;
                        p0[r][1] = p1[r][1];
                        p1[r][1] = no;
                    }
                }
                e4 = e4n;
                o4 = o4n;
                el = eln;
                ol = oln;
            }
        }
        __syncthreads();
        // after the first group of block j, block j + 1 goes to LDS (its slot
        // was last read before this barrier) and block j + 2 is fetched
        if ((g0 - lo) % kAdjCB == 0) {
            const int j = (g0 - lo) / kAdjCB;
            stage_block((j + 1) & 1);
            fetch_block(j + 2);
        }
        // reduce the group: slice rs of output (rg, rv) adds partials rs + SL*j
        const double *rp = gbuf + ((size_t)rg * NV + rv) * T + rs;
        double acc0 = 0.0, acc1 = 0.0;
#pragma unroll
        for (int j = 0; j < PS; j += 2) {
            acc0 += rp[SL * j];
            acc1 += rp[SL * (j + 1)];
        }
        double acc = row16_sum(acc0 + acc1);
        const int is = g0 + rg;  // chain step of this output
        if (rs == 0 && is < nt) {
            if (a.accumulate) {
                const int j = (g0 - lo) / kAdjCB, q = ((g0 - lo) % kAdjCB) / G;
                acc += gbuf_acc[j & 1][q * 16 + ro];
            }
            if (m == 0 && rri == 1) acc = 0.0;
            *gaddr(m + rt + 2 * is, rb, rri) = acc;
        }
    }
    // entries before lo are zero
    if (!a.accumulate) {
        for (int e = tid; e < 2 * lo * NB * 2 && e < (L - m + 1) * NB * 2; e += T) {
            const int l = m + e / (NB * 2);
            if (l - m < 2 * lo) *gaddr(l, (e / 2) % NB, e % 2) = 0.0;
        }
    }
}

// The sum over rings of each output on the matrix cores: per four chain steps
// a wave writes its rings' Legendre values to LDS and multiplies them, 16
// rings at a time, by the unfolded ring phases Y in FP64 MFMA 4x4x4 products
// of four blocks (block b of lane l: (l / 4) % 4; operand A: step l % 4, ring
// l / 4 of the 16; operand B: ring l / 4, value l % 4 = re/im of two maps;
// result: step l / 16, value l % 4, the rings' sum still split over b).  The
// four-block form wastes no column at two maps and above: it runs at the FP64
// peak (72 TFLOP/s measured), where the 16x16x4 form needs eight maps to fill
// its 16 columns.  The four blocks are added by DPP, the waves' sums through
// LDS, one barrier per 16 chain steps (the sums double-buffered), and the
// first waves add them in a fixed order, scale by f_l and store.
//
// A workgroup covers up to 16 R ring groups of its order and parity (W waves
// of R groups each): every ring up to nside = 512 R, else launches over the
// following groups add to g.
constexpr int kAdjMaxWaves = 16;
constexpr int kAdjSteps = 16;     // chain steps per barrier
constexpr int kAdjTileRow = 68;   // doubles per row of 64 rings: 16-lane reads of 4 rows hit distinct banks
// The chains' start values wait in registers where those reach, else in LDS.
constexpr bool adj_start_regs(int NS, int R) { return NS * R <= 4 && R <= 2; }
// LDS doubles of one wave (a tile of 4 steps, a block of coefficients, start
// values), and of a wave's sums of one block of steps
constexpr int adj_wave_lds(int NS, int R) {
    return 4 * kAdjTileRow + 4 * kAdjSteps + (adj_start_regs(NS, R) ? 0 : 128 * R);
}
constexpr int adj_sums(int NS) { return 4 * kAdjSteps * NS; }

// One wave's share of the kAdjSteps steps from c on: the recurrence of its R
// ring groups, the products with their phases Y, and the sums of its rings.
template <int NS, int R, bool POLE>
__device__ __forceinline__ void adj_steps(int c, int whi, int lane, const int (&sid)[R], const double (&x)[R],
                                          const double (&Y)[R][4][NS], const double (&s0)[R], const double (&s1)[R],
                                          double (&P0)[R], double (&P1)[R], const double *cst, double *tile,
                                          const double *room, double *mysum) {
    constexpr bool REGS = adj_start_regs(NS, R);
    const int blk = (lane >> 2) & 3;
#pragma unroll
    for (int q = 0; q < kAdjSteps / 4; q++) {
        const double cv = cst[16 * q + (lane & 15)];
        if (q % 2 == 0 && c + 4 * q <= whi) {
#pragma unroll
            for (int r = 0; r < R; r++)
                if (sid[r] == c + 4 * q) {
                    const double2 v = REGS ? make_double2(s0[r], s1[r])
                                           : *reinterpret_cast<const double2 *>(room + 2 * (r * 64 + lane));
                    P0[r] = v.x;
                    P1[r] = v.y;
                }
        }
        const double cB[4] = {row_bcast<0>(cv), row_bcast<4>(cv), row_bcast<8>(cv), row_bcast<12>(cv)};
        const double cA[4] = {row_bcast<1>(cv), row_bcast<5>(cv), row_bcast<9>(cv), row_bcast<13>(cv)};
        const double cH[4] = {row_bcast<2>(cv), row_bcast<6>(cv), row_bcast<10>(cv), row_bcast<14>(cv)};
        double D[NS];
#pragma unroll
        for (int s = 0; s < NS; s++) D[s] = 0.0;
#pragma unroll
        for (int r = 0; r < R; r++) {
#pragma unroll
            for (int u = 0; u < 4; u++) {
                tile[u * kAdjTileRow + lane] = P0[r];
                if constexpr (POLE) {  // cB = b, cA = r, cH = h
                    const double nx = __builtin_fma(cA[u], P0[r], P1[r]);
                    P1[r] = __builtin_fma(cH[u], P1[r], -(cB[u] * x[r]) * nx);
                    P0[r] = nx;
                } else {
                    const double nx = __builtin_fma(__builtin_fma(x[r], cB[u], cA[u]), P1[r], -P0[r]);
                    P0[r] = P1[r];
                    P1[r] = nx;
                }
            }
            // the wave's own tile: its LDS writes and reads complete in order
            double av[4];
#pragma unroll
            for (int k = 0; k < 4; k++) av[k] = tile[(lane & 3) * kAdjTileRow + 16 * k + (lane >> 2)];
#pragma unroll
            for (int k = 0; k < 4; k++)
#pragma unroll
                for (int s = 0; s < NS; s++)
                    D[s] = __builtin_amdgcn_mfma_f64_4x4x4f64(av[k], Y[r][k][s], D[s], 0, 0, 0);
        }
        // the four blocks' sums, in every block; block s stores value set s
        double v = row_ror_add<4>(row_ror_add<8>(D[0]));
#pragma unroll
        for (int s = 1; s < NS; s++) {
            const double d = row_ror_add<4>(row_ror_add<8>(D[s]));
            v = blk == s ? d : v;
        }
        if (blk < NS) mysum[16 * NS * q + 16 * blk + 4 * (lane >> 4) + (lane & 3)] = v;
    }
}

template <int NS, int R>
__global__ __launch_bounds__(64 * kAdjMaxWaves) void k_legendre_adj(AdjArgs a) {
    extern __shared__ double lds[];
    constexpr int SB = kAdjSteps, NO = adj_sums(NS);
    const int W = blockDim.x >> 6, w = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int slot = blockIdx.x >> 3;
    const int m = xcd_order(blockIdx.x & 7, slot >> 1), t = slot & 1;
    if (m > a.L) return;
    const int L = a.L;
    const int n = L - m - t >= 0 ? (L - m - t) / 2 + 1 : 0;  // chain length
    double *tile = lds + (size_t)w * adj_wave_lds(NS, R), *cst = tile + 4 * kAdjTileRow, *room = cst + 4 * SB;
    double *sums = lds + (size_t)W * adj_wave_lds(NS, R);  // [2][W][NO]
    const size_t arow = (size_t)m * (2 * L + 3 - m) / 2 + t;
    double *gm = a.g + 2 * (arow * a.nmaps + a.map0);

    // this wave's groups: the launch's polar groups fill the first waves, the
    // others the rest, so that a wave runs one recurrence
    const int pole_end = min(max(a.pole_groups, a.first_group), a.end_group);
    const int wp = (pole_end - a.first_group + R - 1) / R;
    const bool pole = w < wp;
    const int g0 = pole ? a.first_group + w * R : pole_end + (w - wp) * R, g1 = pole ? pole_end : a.end_group;
    // chain ranges: of all groups (one per lane), and of this wave's
    int glo = kDead, ghi = -1;
    if (lane >= a.first_group && lane < a.end_group) {
        glo = a.grp_lo[(size_t)m * a.ng + lane];
        ghi = a.grp_hi[(size_t)m * a.ng + lane];
    }
    // rings: chain starts and positions, all loads issued before their first
    // use (groups past the wave's last repeat it and never start)
    const double4 *sc = reinterpret_cast<const double4 *>(a.coef_sc) + a.coef_off[m] + t;
    const size_t row = (size_t)(2 * m + t);
    const double *xp = pole ? a.s2 : a.z2_hi;
    const double *v0p = a.start_val + row * 2 * a.np;
    const double *v1p = pole ? a.start_d + row * a.n_pole_pad : v0p + a.np;
    int sid[R];
    double x[R], P0[R], P1[R], Y[R][4][NS], s0[R], s1[R];
#pragma unroll
    for (int r = 0; r < R; r++) {
        const int k = min(g0 + r, g1 - 1) * kLanes + lane;
        sid[r] = a.start_idx[row * a.np + k] | (g0 + r < g1 ? 0 : kDead);
        x[r] = xp[k];
        s0[r] = v0p[k];
        s1[r] = v1p[k];
        P0[r] = P1[r] = 0.0;
    }
    // phases of 16 rings by two maps an operand, north and mirror unfolded
    const unsigned qrow = (unsigned)(L + 1) * (unsigned)a.nmaps;
    const double *y0 = reinterpret_cast<const double *>(a.ybar + (size_t)m * a.nmaps + a.map0);
    int yc[NS];
#pragma unroll
    for (int s = 0; s < NS; s++) yc[s] = min(4 * s + (lane & 3), 2 * a.nb - 1);  // past the last map: not stored
#pragma unroll
    for (int r = 0; r < R; r++)
#pragma unroll
        for (int q = 0; q < 4; q++) {
            const int kr = min(min(g0 + r, g1 - 1) * kLanes + 16 * q + (lane >> 2), a.n_north - 1);
            const int ks = a.nrings - 1 - kr;
            const double sg = ks == kr ? 0.0 : t ? -1.0 : 1.0;  // the equator counts once
            const double *yn = y0 + 2 * ((size_t)(unsigned)kr * qrow), *ys = y0 + 2 * ((size_t)(unsigned)ks * qrow);
#pragma unroll
            for (int s = 0; s < NS; s++) Y[r][q][s] = __builtin_fma(sg, ys[yc[s]], yn[yc[s]]);
        }
    const bool mine = lane >= g0 && lane < min(g0 + R, g1);
    const int lo = __builtin_amdgcn_readfirstlane(wave_min(glo));
    const int wlo = __builtin_amdgcn_readfirstlane(wave_min(mine ? glo : kDead));
    const int whi = -__builtin_amdgcn_readfirstlane(wave_min(mine ? -ghi : 1));
    if (!a.accumulate)  // below the cutoff on every ring
        for (int e = threadIdx.x; e < min(lo, n) * 2 * a.nb; e += blockDim.x)
            gm[(size_t)(e / (2 * a.nb)) * 4 * a.nmaps + e % (2 * a.nb)] = 0.0;
    if (lo >= n) return;
    // start values in the scaled variables (they wait in LDS where registers
    // do not reach)
#pragma unroll
    for (int r = 0; r < R; r++) {
        const int i = sid[r] >= kDead ? 0 : sid[r];
        s0[r] *= sc[2 * i].w;
        s1[r] *= pole ? 1.0 : sc[2 * i + 2].w;
        if (!adj_start_regs(NS, R))
            *reinterpret_cast<double2 *>(room + 2 * (r * 64 + lane)) = make_double2(s0[r], s1[r]);
    }

    // coefficients of the block's steps: lane 4 u + c holds value c of step u
    // (b, -b d of the scaled recurrence; b, r, h of the split one)
    const int cc = lane & 3;
    const double *cb = (pole && cc ? a.coef_pole + (cc == 1 ? 2 : 0) : a.coef_sc + (cc & 1)) +
                       4 * (a.coef_off[m] + t + 2);
    auto coef = [&](int c) { return cb[8 * (size_t)min(c + (lane >> 2), n - 1)]; };
    double cnext = coef(lo);

    // output o of a block: steps of four, value set, step, value
    auto out_step = [](int o) { return 4 * (o / (16 * NS)) + (o / 4) % 4; };
    auto out_col = [](int o) { return 4 * ((o / 16) % NS) + o % 4; };
    int buf = 0;
    for (int c = lo; c < n; c += SB, buf ^= 1) {
        // what the reduction of this block needs from memory
        double f = 0.0, old = 0.0;
        if (w < NS) {
            const int o = 64 * w + lane, step = min(c + out_step(o), n - 1);
            f = sc[2 * step].z;
            if (a.accumulate) old = gm[(size_t)step * 4 * a.nmaps + min(out_col(o), 2 * a.nb - 1)];
        }
        double *mysum = sums + ((size_t)buf * W + w) * NO;
        cst[lane] = cnext;
        cnext = coef(c + SB);
        if (c + SB <= wlo) {
#pragma unroll
            for (int e = 0; e < NO / 64; e++) mysum[64 * e + lane] = 0.0;
        } else if (pole) {
            adj_steps<NS, R, true>(c, whi, lane, sid, x, Y, s0, s1, P0, P1, cst, tile, room, mysum);
        } else {
            adj_steps<NS, R, false>(c, whi, lane, sid, x, Y, s0, s1, P0, P1, cst, tile, room, mysum);
        }
        __syncthreads();
        // the first waves add the waves' sums, 64 outputs each
        for (int e = w; e < NS; e += W) {
            const int o = 64 * e + lane, step = c + out_step(o), col = out_col(o);
            if (step < n && col < 2 * a.nb) {
                double *out = gm + (size_t)step * 4 * a.nmaps + col;
                if (e != w) {
                    f = sc[2 * step].z;
                    old = a.accumulate ? *out : 0.0;
                }
                const double *p = sums + (size_t)buf * W * NO + o;
                double sum = 0.0;
                int v = 0;
                for (; v + 4 <= W; v += 4, p += 4 * NO) {
                    const double p0 = p[0], p1 = p[NO], p2 = p[2 * NO], p3 = p[3 * NO];
                    sum += (p0 + p1) + (p2 + p3);
                }
                for (; v < W; v++, p += NO) sum += p[0];
                *out = m == 0 && (col & 1) ? 0.0 : __builtin_fma(f, sum, old);
            }
        }
    }
}

// Defined with the ring kernels: raises a kernel's dynamic LDS limit once
// per (kernel, device).
hipError_t allow_dynamic_lds(const void *fn, int bytes);

template <int NS, int R>
static hipError_t launch_adj_cfg(AdjArgs a, hipStream_t st) {
    const int pole_end = std::min(std::max(a.pole_groups, a.first_group), a.end_group);
    const int W = (pole_end - a.first_group + R - 1) / R + (a.end_group - pole_end + R - 1) / R;
    const size_t lds = ((size_t)W * adj_wave_lds(NS, R) + 2 * (size_t)W * adj_sums(NS)) * sizeof(double);
    if (W < 1 || W > kAdjMaxWaves || a.ng > 64 || lds > 160 * 1024) return hipErrorInvalidValue;
    const void *fn = (const void *)k_legendre_adj<NS, R>;
    hipError_t e = allow_dynamic_lds(fn, 160 * 1024);
    if (e != hipSuccess) return e;
    const dim3 grid((unsigned)((a.L + 64) / 64 * 64 * 2));
    hipLaunchKernelGGL((k_legendre_adj<NS, R>), grid, dim3(64 * W), lds, st, a);
    return hipGetLastError();
}

// R ring groups per wave (eight maps: 1; the phases take 8 R NS registers of
// the 128 that 16 waves leave; six maps at two groups spill 20)
static hipError_t launch_adj(const AdjArgs &a, int NS, int R, hipStream_t st) {
    switch (NS) {
        case 4: return launch_adj_cfg<4, 1>(a, st);
        case 3: return R == 1 ? launch_adj_cfg<3, 1>(a, st) : launch_adj_cfg<3, 2>(a, st);
        case 2: return R == 1 ? launch_adj_cfg<2, 1>(a, st) : launch_adj_cfg<2, 2>(a, st);
        default: return R == 1 ? launch_adj_cfg<1, 1>(a, st) : launch_adj_cfg<1, 2>(a, st);
    }
}

template <int NB>
static hipError_t launch_adj_dd(const sht_plan_s *p, AdjArgs a, hipStream_t st) {
    const size_t lds = (size_t)2 * 16 * 256 * sizeof(double);
    hipError_t ea = allow_dynamic_lds((const void *)k_legendre_adj_dd<NB>, (int)lds);
    if (ea != hipSuccess) return ea;
    hipLaunchKernelGGL((k_legendre_adj_dd<NB>), dim3((unsigned)(p->L + 1)), dim3(256), lds, st, a);
    return hipGetLastError();
}

hipError_t launch_legendre_adjoint(const sht_plan_s *p, int nmaps, const double *ybar, double *g,
                                   hipStream_t stream) {
    AdjArgs a;
    a.z2_hi = p->d_z2_hi;
    a.z2_lo = p->d_z2_lo;
    a.s2 = p->d_s2;
    a.coef_off = p->d_coef_off;
    a.coef_hi = p->d_coef_hi;
    a.coef_lo = p->d_coef_lo;
    a.coef_sc = p->d_coef_sc;
    a.coef_pole = p->d_coef_pole;
    a.start_idx = p->d_start_idx;
    a.start_val = p->d_start_val;
    a.start_lo = p->d_start_lo;
    a.start_d = p->d_start_d;
    a.grp_lo = p->d_grp_lo;
    a.grp_hi = p->d_grp_hi;
    a.ybar = reinterpret_cast<const double2 *>(ybar);
    a.g = g;
    a.L = p->L;
    a.nrings = p->nrings;
    a.n_north = p->n_north;
    a.np = p->n_north_pad;
    a.n_dd_pad = std::max(p->n_dd_pad, 1);
    a.n_pole_pad = std::max(p->pole_groups, 1) * kLanes;
    a.ng = p->n_north_pad / kLanes;
    a.nmaps = nmaps;
    a.pole_groups = p->pole_groups;
    a.k0 = a.k1 = 0;
    hipError_t e = hipSuccess;
    // double-double rings first, two maps per pass, in chunks of 256 rings;
    // the first chunk writes g
    const int kdd = p->pole_groups > 0 ? 0 : std::min(p->n_dd_pad, p->n_north);
    for (int b = 0; kdd > 0 && b < nmaps && e == hipSuccess;) {
        a.nb = (nmaps - b) >= 2 ? 2 : 1;
        a.map0 = b;
        for (int k0 = 0; k0 < kdd && e == hipSuccess; k0 += 256) {
            a.k0 = k0;
            a.k1 = std::min(kdd, k0 + 256);
            a.accumulate = k0 > 0 ? 1 : 0;
            e = a.nb == 2 ? launch_adj_dd<2>(p, a, stream) : launch_adj_dd<1>(p, a, stream);
        }
        b += a.nb;
    }
    // the other rings, up to 16 R groups per launch.  Measured with one and two
    // groups a wave, four maps: 4 groups (L = 255) 15.0 and 18.9 us, 8 (L = 511)
    // 49 and 48, 12 (L = 767) 130 and 146, 16 (L = 1023) 348 and 245.  Eight maps
    // a pass take 69 us at 8 groups (two passes of four: 98) and 523 at 16 (489).
    // (opts.rings_per_lane is the synthesis kernel's and has no say here: one
    // group a wave at 16 groups would take 348 us for 245.)
    const int first = kdd > 0 ? p->n_dd_groups : 0, ng = a.ng - first;
    for (int b = 0; b < nmaps && e == hipSuccess;) {
        const int left = nmaps - b;
        a.map0 = b;
        a.nb = left >= 7 ? (ng <= 8 ? std::min(left, 8) : 4) : left;
        const int NS = (a.nb + 1) / 2;
        const int R = NS == 4 || ng <= 12 ? 1 : 2;
        for (int g = first; g < a.ng && e == hipSuccess; g = a.end_group) {
            a.accumulate = kdd > 0 || g > first ? 1 : 0;
            a.first_group = g;
            a.end_group = std::min(a.ng, g + R * kAdjMaxWaves);
            // polar and other groups do not share a wave
            if (g < a.pole_groups && a.pole_groups < a.end_group && (a.pole_groups - g) % R != 0)
                a.end_group = std::min(a.ng, a.pole_groups + R * (kAdjMaxWaves - (a.pole_groups - g + R - 1) / R));
            e = launch_adj(a, NS, R, stream);
        }
        b += a.nb;
    }
    return e;
}

}  // namespace sht
