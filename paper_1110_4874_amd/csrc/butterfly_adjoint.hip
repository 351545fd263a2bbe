// Adjoint of the butterfly-compressed Legendre phase (Sec. 3.2 and App. A.1
// of the Wavemoth paper): g^t = Lambda ybar^t (Sec. 2.4 Eq. 12 transposed)
// runs the factorization backwards, per batch of orders:
//  1. level 1 takes ybar^even = ybar(z) + ybar(-z) and ybar^odd =
//     ybar(z) - ybar(-z) per north ring (Eqs. 13-14 transposed):
//     k_bf_unfold_level1 builds both for the two level-1 nodes of one order
//     and ring range in LDS and splits them at once; orders whose parities
//     split differently get their level-1 vectors from k_bf_unfold and run
//     k_bf_level_t over the listed level-1 nodes;
//  2. k_bf_level_t, level 2 and down: each pair node splits u into its
//     children, v_ch = A~_ch u (identity rows gather u, the dense part T U
//     runs on the matrix cores), so no two waves write one entry;
//  3. k_bf_residual_t: one wave per residual task regenerates the Legendre
//     values of its skeleton rings, four rows at a time, multiplies them by
//     v in FP64 matrix products (sum_z P~(z) v(z)), and adds each row's
//     result to g with one atomic per component (several tasks share a row
//     block's rows, so the order of those few addends, and the last bits of
//     g, may vary from run to run).
#include "butterfly_common.h"
#include "dpp.h"

namespace sht {

// Unfold of the listed slots of one batch: slot j (order m = batch + j
// nbatch) gets ybar^even and ybar^odd of every north ring in its level-1
// vectors (the equator once).
template <typename S>
__global__ __launch_bounds__(kBfThreads) void k_bf_unfold(BfArgs<S> a, int batch, int nbatch,
                                                          const int *__restrict__ slots, int count) {
    const int K = a.K, NP = a.ES / 2;  // maps of the pass
    const long long e = (long long)blockIdx.x * kBfThreads + threadIdx.x;
    if (e >= (long long)count * K * NP) return;
    const int b = (int)(e % NP);
    const long long jk = e / NP;
    const int k = (int)(jk % K), j = slots[jk / K];
    const int m = batch + j * nbatch;
    const int ks = a.nrings - 1 - k;
    const double2 yn = a.ybar[((size_t)k * (a.L + 1) + m) * a.nmaps + a.map0 + b];
    const double2 ys =
        ks != k ? a.ybar[((size_t)ks * (a.L + 1) + m) * a.nmaps + a.map0 + b] : make_double2(0.0, 0.0);
    S *qe = a.ws + ((size_t)(2 * j) * K + k) * a.ES + 2 * b;
    S *qo = a.ws + ((size_t)(2 * j + 1) * K + k) * a.ES + 2 * b;
    qe[0] = (S)(yn.x + ys.x);
    qe[1] = (S)(yn.y + ys.y);
    qo[0] = (S)(yn.x - ys.x);
    qo[1] = (S)(yn.y - ys.y);
}

// One ID block transposed (child ch of a pair node) on one wave:
//   v_ch = A~_ch u:  v[s] = u[perm s] + sum_d T[s][d] u[perm (k + d)].
// The dense part runs on the matrix cores with the skeleton rows s as the
// output rows (four 16-row tiles sharing each U operand) and the dense
// columns d as the reduction, kBfTJ K-steps per batch of loads.  With the
// transposed copy (TT, T^T row-major) lane (i, kq) of K-step j reads
// T^T[d0 + 4 j + kq][s0 + i], 16 consecutive entries per row as in the
// synthesis; otherwise it reads T[s0 + i][d0 + kBfTJ kq + j], kBfTJ
// contiguous entries of 16 different rows.
constexpr int kBfTJ = 2;  // K-steps per batch of loads in the transposed level

// NT 16-row tiles of skeleton rows s0 .. s0 + 16 NT - 1 of one transposed ID
// block (the tile count is a template parameter so that the products run
// back to back).  Columns d past nd get U = 0; rows past k hold clamped rows
// that are not stored.
template <int NT, int NB, bool TT, typename S>
__device__ __forceinline__ void split_tiles(const S *__restrict__ Tb, S *__restrict__ v, int ES, const S *u,
                                            const int16_t *pl, int kk, int nd, int s0, int lane) {
    constexpr int NC = 2 * NB;
    constexpr int DB = 4 * kBfTJ;  // dense columns per batch
    typedef typename Acc<S>::type acc_t;
    const int i16 = lane & 15, k4 = lane >> 4;
    const int ic = min(i16, NC - 1);
    acc_t acc[NT];
#pragma unroll
    for (int tt = 0; tt < NT; tt++) acc[tt] = acc_t{0, 0, 0, 0};
    for (int d0 = 0; d0 < nd; d0 += DB) {
        S av[NT][kBfTJ], bv[kBfTJ];
#pragma unroll
        for (int j = 0; j < kBfTJ; j++) {
            const int d = TT ? d0 + 4 * j + k4 : d0 + kBfTJ * k4 + j, dc = min(d, nd - 1);
            bv[j] = u[pl[kk + dc] * NC + ic] * (S)(d < nd);
#pragma unroll
            for (int tt = 0; tt < NT; tt++) {
                const int sr = min(s0 + 16 * tt + i16, kk - 1);
                av[tt][j] = Tb[TT ? (unsigned)(dc * kk + sr) : (unsigned)(sr * nd + dc)];
            }
        }
#pragma unroll
        for (int j = 0; j < kBfTJ; j++)
#pragma unroll
            for (int tt = 0; tt < NT; tt++) acc[tt] = mfma_16x16x4(av[tt][j], bv[j], acc[tt]);
    }
#pragma unroll
    for (int tt = 0; tt < NT; tt++)
#pragma unroll
        for (int r = 0; r < 4; r++) {
            const int sr = s0 + 16 * tt + acc_row<S>(k4, r);
            if (sr < kk && i16 < NC) v[sr * ES + i16] = acc[tt][r] + u[pl[sr] * NC + i16];
        }
}

template <int NB, bool TT, typename S, bool ONE>
__device__ __forceinline__ void id_block_t(const BfArgs<S> &a, int node, int ch, int half, int lane, const S *u,
                                           const int16_t *pl, int col) {
    constexpr int TPW = 4 / kBfHalves;  // 16-row tiles per wave
    const int *ni = a.node_i + (size_t)node * kBfNodeInts;
    const int kk = ni[2 + ch], nd = ni[4 + ch];
    const int ES = ONE ? 2 * NB : a.ES;  // one group per pass: the stride is a constant
    S *__restrict__ v = a.ws + (size_t)ni[ch] * ES + col;
    const long long toff = (long long)(unsigned)ni[12 + 2 * ch] | ((long long)ni[13 + 2 * ch] << 32);
    const S *__restrict__ Tb = a.T + toff;
    for (int s00 = 0; s00 < kk; s00 += 64) {
        const int ntile = min(TPW, min(4, (kk - s00 + 15) >> 4) - half * TPW);  // tiles of this wave
        const int s0 = s00 + 16 * TPW * half;
        switch (ntile) {
            case 1: split_tiles<1, NB, TT, S>(Tb, v, ES, u, pl, kk, nd, s0, lane); break;
            case 2: split_tiles<2, NB, TT, S>(Tb, v, ES, u, pl, kk, nd, s0, lane); break;
            case 3: split_tiles<3, NB, TT, S>(Tb, v, ES, u, pl, kk, nd, s0, lane); break;
            case 4: split_tiles<4, NB, TT, S>(Tb, v, ES, u, pl, kk, nd, s0, lane); break;
            default: break;
        }
    }
}

// LDS of one transposed pair node with n columns: u (n entries of 2 NB
// values) and both children's column permutations (2 n int16).
template <int NB, typename S>
inline size_t bf_level_t_lds(int n) {
    return (size_t)n * (2 * NB * sizeof(S) + 2 * sizeof(int16_t));
}

// One workgroup of 2 kBfHalves waves per pair node: per group of NB maps,
// u is staged in LDS, then wave w writes half w / 2 of the rows of child
// w % 2's vector.
template <int NB, bool TT, typename S, bool ONE>
__device__ __forceinline__ void level_node_tg(const BfArgs<S> &a, int node) {
    constexpr int NC = 2 * NB;
    extern __shared__ char lds_raw[];
    S *u = reinterpret_cast<S *>(lds_raw);
    const int *ni = a.node_i + (size_t)node * kBfNodeInts;
    const int n = ni[2] + ni[4];
    int16_t *pl = reinterpret_cast<int16_t *>(u + (size_t)n * NC);
    const int ES = ONE ? NC : a.ES, G = ONE ? 1 : a.G;
    const S *__restrict__ in = a.ws + (size_t)ni[6] * ES;
    const int16_t *__restrict__ pg = a.perm + ni[7];
    for (int e = threadIdx.x; e < 2 * n; e += kBfLevelThreads) pl[e] = pg[e];
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    for (int g = 0; g < G; g++) {
        if (g) __syncthreads();  // the previous group's splits have read u
        if (ONE) {
            for (int e = threadIdx.x; e < n * NC; e += kBfLevelThreads) u[e] = in[e];
        } else {
            for (int e = threadIdx.x; e < n * NC; e += kBfLevelThreads) u[e] = in[(size_t)(e / NC) * ES + g * NC + e % NC];
        }
        __syncthreads();
        id_block_t<NB, TT, S, ONE>(a, node, w & 1, w >> 1, threadIdx.x & 63, u, pl + (w & 1) * n, g * NC);
    }
}



// ONE: the pass has a single group of maps (separate instantiations, so the
// common case keeps its constant strides and its register count).
template <int NB, bool TT, typename S, bool ONE>
__global__ __launch_bounds__(kBfLevelThreads) void k_bf_level_t(BfArgs<S> a, long long n0) {
    level_node_tg<NB, TT, S, ONE>(a, (int)(n0 + blockIdx.x));
}

// Level-1 nodes that run alone (their order was unfolded beforehand).
template <int NB, bool TT, typename S, bool ONE>
__global__ __launch_bounds__(kBfLevelThreads) void k_bf_level_t_list(BfArgs<S> a, const int *__restrict__ list,
                                                                     long long n0) {
    level_node_tg<NB, TT, S, ONE>(a, list[n0 + blockIdx.x]);
}

// Unfold fused with level 1 (Eqs. 13-14 transposed): one workgroup per unit
// {even node, odd node, first ring k0, slot}; both nodes cover the rings
// k0 .. k0+n-1 of one order, so ybar^even and ybar^odd of those rings are
// built in LDS from the two hemispheres' ybar and split by both nodes at once.
constexpr int kBfUnfoldThreads = 2 * kBfLevelThreads;

template <int NB, bool TT, typename S, bool ONE>
__global__ __launch_bounds__(kBfUnfoldThreads) void k_bf_unfold_level1(BfArgs<S> a, const int4 *__restrict__ units,
                                                                       long long u0, int batch, int nbatch) {
    constexpr int NC = 2 * NB;
    extern __shared__ char lds_raw[];
    const int4 un = units[u0 + blockIdx.x];
    const int *nie = a.node_i + (size_t)un.x * kBfNodeInts;
    const int n = nie[2] + nie[4];
    S *uE = reinterpret_cast<S *>(lds_raw);
    S *uO = uE + (size_t)n * NC;
    int16_t *pl = reinterpret_cast<int16_t *>(uO + (size_t)n * NC);  // even node's 2n entries, then odd's
    const int16_t *__restrict__ pe = a.perm + nie[7];
    const int16_t *__restrict__ po = a.perm + a.node_i[(size_t)un.y * kBfNodeInts + 7];
    for (int e = threadIdx.x; e < 4 * n; e += kBfUnfoldThreads) pl[e] = e < 2 * n ? pe[e] : po[e - 2 * n];
    const int m = batch + un.w * nbatch, k0 = un.z;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int par = w / (2 * kBfHalves), wc = w % (2 * kBfHalves);
    const int G = ONE ? 1 : a.G;
    for (int g = 0; g < G; g++) {
        if (g) __syncthreads();  // the previous group's splits have read uE and uO
        const int mb = a.map0 + g * NB;
        for (int e = threadIdx.x; e < n * NB; e += kBfUnfoldThreads) {
            const int c = e / NB, b = e % NB;
            const int k = k0 + c, ks = a.nrings - 1 - k;
            const double2 yn = a.ybar[((size_t)k * (a.L + 1) + m) * a.nmaps + mb + b];
            const double2 ys =
                ks != k ? a.ybar[((size_t)ks * (a.L + 1) + m) * a.nmaps + mb + b] : make_double2(0.0, 0.0);
            uE[c * NC + 2 * b] = (S)(yn.x + ys.x);
            uE[c * NC + 2 * b + 1] = (S)(yn.y + ys.y);
            uO[c * NC + 2 * b] = (S)(yn.x - ys.x);
            uO[c * NC + 2 * b + 1] = (S)(yn.y - ys.y);
        }
        __syncthreads();
        id_block_t<NB, TT, S, ONE>(a, par ? un.y : un.x, wc & 1, wc >> 1, threadIdx.x & 63, par ? uO : uE,
                                   pl + (2 * par + (wc & 1)) * n, g * NC);
    }
}

// One transposed residual task on one wave: R rings per lane, rows
// [imin, iend) of parity t; each row's sum over the task's rings goes to g.
// As in the brute-force adjoint (adjoint.hip): four rows at a time the wave
// writes its rings' values of the scaled recurrence to LDS and multiplies
// them, 16 rings at a time, by the vector in FP64 MFMA 4x4x4 products of four
// blocks (operand A: row l % 4, ring l / 4; B: ring l / 4, value l % 4; result:
// row l / 16, value l % 4, split over the blocks (l / 4) % 4), which are added by
// DPP.  Rows are taken at multiples of four; those outside [imin, iend) add
// nothing.  (With the sums of 64 lanes by lane swaps, row by row, and
// coefficients by uniform loads, the launch took 1238 us at L = 2047, 4 maps;
// so 943 us.)
constexpr int kBfTileRow = 68;  // doubles per row of 64 rings: 16-lane reads of 4 rows hit distinct banks
constexpr int kBfTLds = 4 * kBfTileRow + 64;  // a tile of four rows, coefficients of 16

template <int NB, int R, typename S>
__device__ __forceinline__ void residual_task_t(const BfArgs<S> &a, long long tk, int lane, int t, int imin,
                                                int iend, int nl, int outb, int m, double *lds, int col0) {
    constexpr int NC = 2 * NB, NS = (NC + 3) / 4;
    double *tile = lds, *cst = lds + 4 * kBfTileRow;
    if (imin >= iend) return;
    const double4 *sc = reinterpret_cast<const double4 *>(a.coef_sc) + a.coef_off[m] + t;
    int i0[R];
    double z2[R], v0[R], v1[R], P0[R], P1[R], Y[R][4][NS];
#pragma unroll
    for (int r = 0; r < R; r++) {
        const size_t li = (size_t)tk * kBfTaskRings + r * 64 + lane;
        const int2 ln = a.res_lane[li];
        const double2 sv = a.res_val[li];
        i0[r] = ln.y;
        z2[r] = a.z2[ln.x];
        v0[r] = sv.x;
        v1[r] = sv.y;
        P0[r] = P1[r] = 0.0;
        // (lanes past the task's last ring never start)
#pragma unroll
        for (int q = 0; q < 4; q++)
#pragma unroll
            for (int s = 0; s < NS; s++)
                Y[r][q][s] = (double)a.ws[((size_t)outb + min(64 * r + 16 * q + (lane >> 2), nl - 1)) * a.ES + col0 +
                                          min(4 * s + (lane & 3), NC - 1)];
    }
    // coefficients of 16 rows: lane 4 u + c holds value c of row u (b, -b d of
    // the next row, f of the row)
    const double *cb = reinterpret_cast<const double *>((lane & 3) < 2 ? sc + 2 : sc) + min(lane & 3, 2);
    auto coef = [&](int c) { return cb[8 * (size_t)min(c + (lane >> 2), iend - 1)]; };
    int c = imin & ~3;
    double cnext = coef(c);
#pragma unroll
    for (int r = 0; r < R; r++) {
        const int i = i0[r] < iend ? i0[r] : imin;
        v0[r] *= sc[2 * i].w;
        v1[r] *= sc[2 * i + 2].w;
    }
    const size_t aoff = (size_t)m * (2 * a.L + 3 - m) / 2;
    // component c = 2 b + (re, im) of row i lives at gb[i * 4 nmaps + c]
    double *gb = a.g + 2 * ((aoff + t) * a.nmaps + a.map0);
    const size_t gstride = 4 * (size_t)a.nmaps;
    const int blk = (lane >> 2) & 3, col = 4 * blk + (lane & 3);
    const bool writer = blk < NS && col < NC && !(m == 0 && (col & 1));
    for (; c < iend; c += 16) {
        cst[lane] = cnext;
        cnext = coef(c + 16);
#pragma unroll
        for (int q = 0; q < 4; q++) {
            if (c + 4 * q >= iend) break;
            const double cv = cst[16 * q + (lane & 15)];
            const double cB[4] = {row_bcast<0>(cv), row_bcast<4>(cv), row_bcast<8>(cv), row_bcast<12>(cv)};
            const double cA[4] = {row_bcast<1>(cv), row_bcast<5>(cv), row_bcast<9>(cv), row_bcast<13>(cv)};
            const double f = cst[16 * q + 4 * (lane >> 4) + 2];
            double D[NS];
#pragma unroll
            for (int s = 0; s < NS; s++) D[s] = 0.0;
#pragma unroll
            for (int r = 0; r < R; r++) {
                // chains start at imin or at a multiple of kChunk
#pragma unroll
                for (int u = 0; u < 4; u++) {
                    const int i = c + 4 * q + u;
                    if (u == 0 || (q == 0 && i == imin)) {
                        const bool st = i0[r] == i;
                        P0[r] = st ? v0[r] : P0[r];
                        P1[r] = st ? v1[r] : P1[r];
                    }
                    tile[u * kBfTileRow + lane] = P0[r];
                    const double nx = __builtin_fma(__builtin_fma(z2[r], cB[u], cA[u]), P1[r], -P0[r]);
                    P0[r] = P1[r];
                    P1[r] = nx;
                }
                // the wave's own tile: its LDS writes and reads complete in order
                double av[4];
#pragma unroll
                for (int k = 0; k < 4; k++) av[k] = tile[(lane & 3) * kBfTileRow + 16 * k + (lane >> 2)];
#pragma unroll
                for (int k = 0; k < 4; k++)
#pragma unroll
                    for (int s = 0; s < NS; s++)
                        D[s] = __builtin_amdgcn_mfma_f64_4x4x4f64(av[k], Y[r][k][s], D[s], 0, 0, 0);
            }
            // the four blocks' sums, in every block; block s adds value set s to g
            double v = row_ror_add<4>(row_ror_add<8>(D[0]));
#pragma unroll
            for (int s = 1; s < NS; s++) {
                const double d = row_ror_add<4>(row_ror_add<8>(D[s]));
                v = blk == s ? d : v;
            }
            const int i = c + 4 * q + (lane >> 4);
            if (writer && i >= imin && i < iend) atomicAdd(gb + (size_t)i * gstride + col, f * v);
        }
    }
}

template <int NB, typename S>
__global__ __launch_bounds__(kBfResThreads) void k_bf_residual_t(BfArgs<S> a, long long t0, long long t1, int col0) {
    const int lane = threadIdx.x & 63;
    const long long tk = t0 + (long long)blockIdx.x * (kBfResThreads / 64) + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (tk >= t1) return;
    const int4 h = a.res_task[2 * tk], h2 = a.res_task[2 * tk + 1];
    const int t = __builtin_amdgcn_readfirstlane(h.x), imin = __builtin_amdgcn_readfirstlane(h.y);
    const int iend = __builtin_amdgcn_readfirstlane(h.z), nl = __builtin_amdgcn_readfirstlane(h.w);
    const int outb = __builtin_amdgcn_readfirstlane(h2.x), m = __builtin_amdgcn_readfirstlane(h2.y);
    __shared__ double lds_all[kBfResThreads / 64][kBfTLds];
    double *lds = lds_all[__builtin_amdgcn_readfirstlane(threadIdx.x >> 6)];
    if constexpr (kBfTaskRings > 192) {
        if (nl > 192) return residual_task_t<NB, 4>(a, tk, lane, t, imin, iend, nl, outb, m, lds, col0);
    }
    if constexpr (kBfTaskRings > 128) {
        if (nl > 128) return residual_task_t<NB, 3>(a, tk, lane, t, imin, iend, nl, outb, m, lds, col0);
    }
    if constexpr (kBfTaskRings > 64) {
        if (nl > 64) return residual_task_t<NB, 2>(a, tk, lane, t, imin, iend, nl, outb, m, lds, col0);
    }
    residual_task_t<NB, 1>(a, tk, lane, t, imin, iend, nl, outb, m, lds, col0);
}

// g = 0 over the nalm rows of maps [map0, map0 + nb) (a kernel, not a
// memset, so that the adjoint can be captured into a graph).
__global__ __launch_bounds__(kBfThreads) void k_bf_zero(double *g, long long nalm, int nmaps, int map0, int nb) {
    const long long e = (long long)blockIdx.x * kBfThreads + threadIdx.x;
    if (e >= nalm * nb * 2) return;
    const long long row = e / (2 * nb);
    const int rest = (int)(e % (2 * nb));
    g[2 * (row * nmaps + map0) + rest] = 0.0;
}

template <int NB, bool TT, typename S, bool ONE>
static hipError_t launch_bf_adj_nbg(const sht_plan_s *p, BfArgs<S> a, hipStream_t st) {
    constexpr int WPB = kBfResThreads / 64;
    const BflyPlan &b = p->bf;
    const long long nalm = (long long)(p->L + 1) * (p->L + 2) / 2;
    const int np = NB * a.G;  // maps of the pass
    hipLaunchKernelGGL(k_bf_zero, dim3((unsigned)((nalm * np * 2 + kBfThreads - 1) / kBfThreads)), dim3(kBfThreads), 0,
                       st, a.g, nalm, a.nmaps, a.map0, np);
    for (int bt = 0; bt < b.nbatch; bt++) {
        // level 1: fused with the unfold where both parities have levels
        const long long s0 = b.fold_off[bt], s1 = b.fold_off[bt + 1];
        const long long nf = (s1 - s0) * b.K * np;
        if (nf > 0)
            hipLaunchKernelGGL((k_bf_unfold<S>), dim3((unsigned)((nf + kBfThreads - 1) / kBfThreads)),
                               dim3(kBfThreads), 0, st, a, bt, b.nbatch, p->d_bf_fold_slot + s0, (int)(s1 - s0));
        const size_t lds1 = bf_level_t_lds<NB, S>(b.lv_max_n[(size_t)bt * kBfMaxLv + kBfMaxLv - 1]);
        const long long p0 = b.l1_off[bt], p1 = b.l1_off[bt + 1];
        if (p1 > p0)
            hipLaunchKernelGGL((k_bf_level_t_list<NB, TT, S, ONE>), dim3((unsigned)(p1 - p0)), dim3(kBfLevelThreads), lds1, st,
                               a, p->d_bf_l1_plain, p0);
        const long long f0 = b.f1_off[bt], f1 = b.f1_off[bt + 1];
        if (f1 > f0)
            hipLaunchKernelGGL((k_bf_unfold_level1<NB, TT, S, ONE>), dim3((unsigned)(f1 - f0)), dim3(kBfUnfoldThreads), 2 * lds1,
                               st, a, reinterpret_cast<const int4 *>(p->d_bf_f1_unit), f0, bt, b.nbatch);
        const long long *lo = b.lv_off.data() + (size_t)bt * (kBfMaxLv + 1);
        for (int q = kBfMaxLv - 2; q >= 0; q--) {  // levels >= 2
            const long long n0 = lo[q], n1 = lo[q + 1];
            if (n1 <= n0) continue;
            const size_t lds = bf_level_t_lds<NB, S>(b.lv_max_n[(size_t)bt * kBfMaxLv + q]);
            hipLaunchKernelGGL((k_bf_level_t<NB, TT, S, ONE>), dim3((unsigned)(n1 - n0)), dim3(kBfLevelThreads), lds, st, a,
                               n0);
        }
        const long long t0 = b.batch_task[bt], t1 = b.batch_task[bt + 1];
        for (int g = 0; g < a.G && t1 > t0; g++) {  // one launch per group of NB maps
            BfArgs<S> ag = a;
            ag.map0 = a.map0 + g * NB;
            hipLaunchKernelGGL((k_bf_residual_t<NB, S>), dim3((unsigned)((t1 - t0 + WPB - 1) / WPB)),
                               dim3(kBfResThreads), 0, st, ag, t0, t1, g * 2 * NB);
        }
    }
    return hipGetLastError();
}

template <int NB, bool TT, typename S>
static hipError_t launch_bf_adj_nb(const sht_plan_s *p, BfArgs<S> a, hipStream_t st) {
    return a.G == 1 ? launch_bf_adj_nbg<NB, TT, S, true>(p, a, st) : launch_bf_adj_nbg<NB, TT, S, false>(p, a, st);
}

template <typename S>
static hipError_t launch_bf_adj(const sht_plan_s *p, int nmaps, const double *ybar, double *g, S *ws, const S *T,
                                const S *Tt, hipStream_t st) {
    BfArgs<S> a = bf_args<S>(p, nmaps, Tt ? Tt : T, ws);
    a.ybar = reinterpret_cast<const double2 *>(ybar);
    a.g = g;
    hipError_t e = hipSuccess;
    for (int b = 0; b < nmaps && e == hipSuccess;) {
        int nb, groups;
        bf_pass_shape(nmaps - b, &nb, &groups);
        a.map0 = b;
        a.G = groups;
        a.ES = 2 * nb * groups;
        if (Tt) {
            switch (nb) {
                case 8: e = launch_bf_adj_nb<8, true, S>(p, a, st); break;
                case 4: e = launch_bf_adj_nb<4, true, S>(p, a, st); break;
                case 2: e = launch_bf_adj_nb<2, true, S>(p, a, st); break;
                default: e = launch_bf_adj_nb<1, true, S>(p, a, st); break;
            }
        } else {
            switch (nb) {
                case 8: e = launch_bf_adj_nb<8, false, S>(p, a, st); break;
                case 4: e = launch_bf_adj_nb<4, false, S>(p, a, st); break;
                case 2: e = launch_bf_adj_nb<2, false, S>(p, a, st); break;
                default: e = launch_bf_adj_nb<1, false, S>(p, a, st); break;
            }
        }
        b += nb * groups;
    }
    return e;
}

hipError_t launch_butterfly_adjoint(const sht_plan_s *p, int nmaps, const double *ybar, double *g, void *scratch,
                                    int fp32, hipStream_t stream) {
    if (fp32) return launch_bf_adj<float>(p, nmaps, ybar, g, (float *)scratch, p->d_bf_T32, p->d_bf_Tt32, stream);
    return launch_bf_adj<double>(p, nmaps, ybar, g, (double *)scratch, p->d_bf_T, p->d_bf_Tt, stream);
}

// Transposed copy of every interpolation block: child ch of a pair node keeps
// its kk x nd matrix T row-major at toff; Tt receives the nd x kk transpose
// at the same offset.  One workgroup per (node, child).
template <typename S>
__global__ __launch_bounds__(kBfThreads) void k_bf_transpose_blocks(const int *__restrict__ node_i,
                                                                    const S *__restrict__ T, S *__restrict__ Tt) {
    const int *ni = node_i + (size_t)(blockIdx.x >> 1) * kBfNodeInts;
    const int ch = blockIdx.x & 1;
    const int kk = ni[2 + ch], nd = ni[4 + ch];
    const long long toff = (long long)(unsigned)ni[12 + 2 * ch] | ((long long)ni[13 + 2 * ch] << 32);
    const int n = kk * nd;
    for (int f = threadIdx.x; f < n; f += kBfThreads) {
        const int d = f / kk, s = f - d * kk;
        Tt[toff + f] = T[toff + (long long)s * nd + d];
    }
}

hipError_t bf_store_transposed(sht_plan_s *p, size_t nT, size_t nnodes, size_t *bytes) {
    const size_t n = std::max<size_t>(nT, 1);
    if (2 * nnodes > 0xFFFFFFFFull) return hipErrorInvalidValue;
    hipError_t e = hipMalloc((void **)&p->d_bf_Tt, n * sizeof(double));
    if (e != hipSuccess) return e;
    *bytes += n * sizeof(double);
    if (nnodes)
        hipLaunchKernelGGL(k_bf_transpose_blocks<double>, dim3((unsigned)(2 * nnodes)), dim3(kBfThreads), 0, 0,
                           p->d_bf_node_i, p->d_bf_T, p->d_bf_Tt);
    if (p->d_bf_T32) {
        e = hipMalloc((void **)&p->d_bf_Tt32, n * sizeof(float));
        if (e != hipSuccess) return e;
        *bytes += n * sizeof(float);
        if (nnodes)
            hipLaunchKernelGGL(k_bf_transpose_blocks<float>, dim3((unsigned)(2 * nnodes)), dim3(kBfThreads), 0, 0,
                               p->d_bf_node_i, p->d_bf_T32, p->d_bf_Tt32);
    }
    e = hipGetLastError();
    if (e == hipSuccess) e = hipDeviceSynchronize();
    return e;
}

}  // namespace sht
