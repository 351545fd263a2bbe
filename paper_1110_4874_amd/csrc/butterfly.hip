// Butterfly-compressed Legendre phase for gfx950 (Sec. 3.2 and App. A.1 of
// the Wavemoth paper): q^t_m = Lambda^T a^t applied as
//   a^T Lambda = (a^T R) S_d P_{d-1} ... P_1 S_1,
// followed by the even/odd fold of Sec. 2.4 (Eqs. 13-14).
//
// The paper walks each order's tree depth first to stay in a CPU's caches.
// Here every level is one launch over all orders at once (breadth first),
// which gives the GPU tens of thousands of independent waves to stream the
// interpolation matrices with; vectors between levels live in a device
// workspace (read and written once per level):
//  1. k_bf_residual: one wave per residual piece (up to kBfPieceRings skeleton
//     rings of one row block, four per lane) regenerates the Legendre values with the
//     two-step recurrence (App. A.2, Eq. A2) over the block's rows from two
//     stored values per ring and accumulates v = sum_l a_lm P~_l^m(z) for
//     every map; the a_lm rows and coefficients are staged through LDS;
//  2. k_bf_level, deepest level first down to level 2: one workgroup (a wave
//     per child) per pair node (two sibling row blocks sharing the column set
//     C) computes u = A~_0^T v_0 + A~_1^T v_1: identity rows copy v, the
//     dense part T^T V runs on the matrix cores;
//  3. level 1 yields q^even and q^odd per north ring: k_bf_level1_fold runs
//     the two level-1 nodes of one order and ring range together and writes
//     q rows k and 4 nside - k from q^even +- q^odd (Eqs. 13-14); orders
//     whose parities split differently run k_bf_level_list, then k_bf_fold.
//
// The adjoint runs the same factorization backwards in butterfly_adjoint.hip.
#include <cstring>
#include <type_traits>

#include "butterfly_common.h"
#include "dpp.h"

namespace sht {


// One ID block (child ch of a pair node) on one wave: child ch's share of
//   u = A~_0^T v_0 + A~_1^T v_1
// over the columns C the two sibling row blocks share.  Its column
// permutation places every column of C exactly once, as a skeleton column
// (u[perm s] = v[s]) or a dense one (u[perm (k + d)] = sum_s T[s][d] v[s]),
// so the wave writes each entry of its own LDS buffer uc once, with plain
// stores, and the two buffers are summed afterwards.  The dense part T^T V
// (nd x k times k x NC) runs on the matrix cores, up to 64 dense rows (four
// 16-row tiles sharing each V operand) by kBfKSteps * 4 rows of T per batch
// of loads.  Loads take clamped (in-block) addresses and rows s past k are
// masked by multiplying V with 0, so a batch issues all its loads without
// branches; dense rows past nd and columns past NC only reach outputs that
// are not stored.
constexpr int kBfKSteps = 4;    // K-steps (4 rows of T each) per batch of loads
constexpr int kBfIdUnroll = 4;  // identity entries per lane in flight

// The results of NT tiles to their positions in C.
template <int NT, int NB, typename S, int N>
__device__ __forceinline__ void store_tiles(const typename Acc<S>::type (&acc)[N], const int16_t *__restrict__ pm, int kk,
                                            int nd, int gw, int lane, S *uc) {
    constexpr int NC = 2 * NB;
    const int i16 = lane & 15, k4 = lane >> 4;
    // the output rows' positions in C, all loads issued before the first
    // store (the empty asm keeps the compiler from moving each load into
    // its store's branch, which would wait on them one by one)
    int pr[NT][4];
#pragma unroll
    for (int tt = 0; tt < NT; tt++)
#pragma unroll
        for (int r = 0; r < 4; r++) pr[tt][r] = pm[kk + min(gw + 16 * tt + acc_row<S>(k4, r), nd - 1)];
    asm volatile("" ::: "memory");
#pragma unroll
    for (int tt = 0; tt < NT; tt++)
#pragma unroll
        for (int r = 0; r < 4; r++) {
            const int dd = gw + 16 * tt + acc_row<S>(k4, r);
            if (dd < nd && i16 < NC) uc[pr[tt][r] * NC + i16] = acc[tt][r];
        }
}

// NT 16-row tiles of dense rows gw .. gw + 16 NT - 1 of one ID block:
// uc[perm (k + d)] = sum_s T[s][d] v[s] (32-bit element offsets from
// wave-uniform bases; the tile count is a template parameter so that the
// products run back to back, without branches between them).
// TWO: the products of the next group of maps as well, left in `next`.
template <int NT, bool TWO, int NB, typename S>
__device__ __forceinline__ void dense_tiles(const S *__restrict__ v, int ES, const S *__restrict__ Tb,
                                            const int16_t *__restrict__ pm, int kk, int nd, int gw, int lane,
                                            S *uc, typename Acc<S>::type (&next)[4]) {
    constexpr int NC = 2 * NB;
    constexpr int KS = TWO ? kBfKSteps / 2 : kBfKSteps;
    typedef typename Acc<S>::type acc_t;
    const int i16 = lane & 15, k4 = lane >> 4;
    const int ic = min(i16, NC - 1);
    acc_t acc[NT];
#pragma unroll
    for (int tt = 0; tt < NT; tt++) {
        acc[tt] = acc_t{0, 0, 0, 0};
        if (TWO) next[tt] = acc_t{0, 0, 0, 0};
    }
    for (int s0 = 0; s0 < kk; s0 += 4 * KS) {
        S av[KS][NT], bv[KS], bn[KS];
#pragma unroll
        for (int j = 0; j < KS; j++) {
            const int s = s0 + 4 * j + k4, sc = min(s, kk - 1);
            bv[j] = ld32(v, sc * ES + ic) * (S)(s < kk);
            if (TWO) bn[j] = ld32(v, sc * ES + NC + ic) * (S)(s < kk);
#pragma unroll
            for (int tt = 0; tt < NT; tt++) av[j][tt] = ld32(Tb, sc * nd + min(gw + 16 * tt + i16, nd - 1));
        }
#pragma unroll
        for (int j = 0; j < KS; j++)
#pragma unroll
            for (int tt = 0; tt < NT; tt++) {
                acc[tt] = mfma_16x16x4(av[j][tt], bv[j], acc[tt]);
                if (TWO) next[tt] = mfma_16x16x4(av[j][tt], bn[j], next[tt]);
            }
    }
    store_tiles<NT, NB, S, NT>(acc, pm, kk, nd, gw, lane, uc);
}

// A pass of several groups streams T once for two of them (the second read of
// a block missed the L2): AHEAD computes the products of the next group with
// this one's and leaves them in `next`, in registers (blocks of up to 64 dense
// rows; others run each group by itself), DONE takes them from there.  Half
// the K-steps a batch and three wavefronts a SIMD keep it from spilling.  L =
// 2047, 16 maps: level launch 693 -> 607 us, fused level 1 the same 1136 us;
// FP32 492 -> 440 and 1019 -> 964 us (with whole batches 678 and 1173 us).
enum class Pair { NONE, AHEAD, DONE };
template <int NB, typename S, bool ONE, Pair PAIR = Pair::NONE>
__device__ __forceinline__ void id_block(const BfArgs<S> &a, int node, int ch, int half, int lane, S *uc, int col,
                                         typename Acc<S>::type (&next)[4]) {
    constexpr int NC = 2 * NB;
    constexpr int TPW = 4 / kBfHalves;  // tiles per wave
    const int *ni = a.node_i + (size_t)node * kBfNodeInts;
    const int n = ni[2] + ni[4];
    const int kk = ni[2 + ch], nd = ni[4 + ch];
    const int ES = ONE ? NC : a.ES;  // one group per pass: the stride is a constant
    const S *__restrict__ v = a.ws + (size_t)ni[ch] * ES + col;
    const int16_t *__restrict__ pm = a.perm + ni[7] + (size_t)ch * n;
    const long long toff = (long long)(unsigned)ni[12 + 2 * ch] | ((long long)ni[13 + 2 * ch] << 32);
    const S *__restrict__ Tb = a.T + toff;
    // identity rows (lanes past the end repeat the last entry's store)
    const int ne = kk * NC;
    for (int e0 = 64 * half; e0 < ne; e0 += 64 * kBfHalves * kBfIdUnroll) {
        S x[kBfIdUnroll];
        int px[kBfIdUnroll];
#pragma unroll
        for (int j = 0; j < kBfIdUnroll; j++) {
            const int ec = min(e0 + lane + 64 * kBfHalves * j, ne - 1);
            x[j] = ld32(v, (ec / NC) * ES + ec % NC);
            px[j] = pm[ec / NC];
        }
#pragma unroll
        for (int j = 0; j < kBfIdUnroll; j++) {
            const int ec = min(e0 + lane + 64 * kBfHalves * j, ne - 1);
            uc[px[j] * NC + ec % NC] = x[j];
        }
    }
    // dense rows, in groups of 64
    auto tiles = [&](auto two, int ntile, int gw) {
        constexpr bool TWO = decltype(two)::value;
        switch (ntile) {
            case 1: dense_tiles<1, TWO, NB>(v, ES, Tb, pm, kk, nd, gw, lane, uc, next); break;
            case 2: dense_tiles<2, TWO, NB>(v, ES, Tb, pm, kk, nd, gw, lane, uc, next); break;
            case 3: dense_tiles<3, TWO, NB>(v, ES, Tb, pm, kk, nd, gw, lane, uc, next); break;
            case 4: dense_tiles<4, TWO, NB>(v, ES, Tb, pm, kk, nd, gw, lane, uc, next); break;
            default: break;
        }
    };
    if constexpr (PAIR != Pair::NONE) {
        if (nd <= 64) {
            const int ntile = min(TPW, (nd + 15) / 16 - half * TPW), gw = 16 * TPW * half;
            if constexpr (PAIR == Pair::AHEAD) {
                tiles(std::true_type{}, ntile, gw);
            } else {
                switch (ntile) {
                    case 1: store_tiles<1, NB, S>(next, pm, kk, nd, gw, lane, uc); break;
                    case 2: store_tiles<2, NB, S>(next, pm, kk, nd, gw, lane, uc); break;
                    case 3: store_tiles<3, NB, S>(next, pm, kk, nd, gw, lane, uc); break;
                    case 4: store_tiles<4, NB, S>(next, pm, kk, nd, gw, lane, uc); break;
                    default: break;
                }
            }
            return;
        }
    }
    for (int g0 = 0; g0 < nd; g0 += 64)
        tiles(std::false_type{}, min(TPW, min(4, (nd - g0 + 15) >> 4) - half * TPW), g0 + 16 * TPW * half);
}

// One residual piece on one wave: R rings per lane (lane j: rings j + 64 r,
// lane records from lbase), rows [imin, iend) of one parity, outputs at
// entries outb + ring.  The scaled recurrence of legendre.hip (two FP64
// operations a step, f_l in the staged a_lm).  The a_lm rows and recurrence
// coefficients of each aligned chunk of kChunk rows are fetched one chunk
// ahead with coalesced vector loads and staged in the wave's own LDS slot
// (stg: two chunks) as rows of 16 (NC <= 14) or 32 values: a_lm components,
// then the two coefficients.  Lane k of every 16-lane row reads value k of a
// row, and the products take the values from there by DPP broadcasts; LDS
// operations of one wave complete in order, so no barrier is needed.  The
// loads are unconditional, of rows clamped into [imin, iend), and rows outside
// are overwritten with zeros in LDS: a select on a load would become a branch
// that waits for memory, twice a chunk.  Start values wait in LDS, where they
// cost no registers.  Residual launch at L = 2047: 4 maps 735 us (781 with
// selected loads and 16-byte stores into 64 entries at once), with FP32 results
// 680 us (808); 8 maps 1210 us (1455; 1386 with those stores alone), FP32 1175.
// FP64 issue bounds it: its products alone take 842 us for 8 maps, and 18% of
// its instructions stage operands.
template <int NB>
constexpr int bf_res_row_doubles() {
    return 2 * NB + 2 <= 16 ? 16 : 32;
}
template <int NB>
constexpr int bf_res_stage_doubles() {
    return 2 * kChunk * bf_res_row_doubles<NB>() + 2 * kBfPieceRings;
}

template <int NB, int R, typename S>
__device__ __forceinline__ void residual_task(const BfArgs<S> &a, S *__restrict__ slot, long long lbase, int lane,
                                              int t, int imin, int iend, int nl, int outb,
                                              const double *__restrict__ ap, const double4 *__restrict__ sc,
                                              int astride, double *stg, int col0) {
    constexpr int NC = 2 * NB;
    constexpr int CW = bf_res_row_doubles<NB>();  // staged values per row
    constexpr int CS = kChunk * CW;                // doubles per staged chunk
    constexpr int E = CS / 64;                     // staged doubles per lane
    constexpr int CO = NC % 16;                    // lane of b within its 16-lane row
    static_assert(NC + 2 <= 16 || NC == 16, "the coefficients share one 16-lane row");
    int i0[R];
    double z2[R], P0[R], P1[R], acc[R][NC];
    double2 *st = reinterpret_cast<double2 *>(stg + 2 * CS);  // the rings' start values
#pragma unroll
    for (int r = 0; r < R; r++) {
        const size_t li = (size_t)lbase + r * 64 + lane;
        const int2 ln = a.res_lane[li];
        st[r * 64 + lane] = a.res_val[li];
        i0[r] = ln.y;
        z2[r] = a.z2[ln.x];
        P0[r] = P1[r] = 0.0;
#pragma unroll
        for (int c = 0; c < NC; c++) acc[r][c] = 0.0;
    }
    auto step_v = [&](double rv, double rc) {
        const double eb = row_bcast<CO>(rc), ea = row_bcast<CO + 1>(rc);
#pragma unroll
        for (int r = 0; r < R; r++) {
            fmac_row_bcast<NC>(acc[r], rv, P0[r]);
            const double P2 = __builtin_fma(__builtin_fma(z2[r], eb, ea), P1[r], -P0[r]);
            P0[r] = P1[r];
            P1[r] = P2;
        }
    };
    // a piece without rows (a parity with no l <= L) writes zeros and loads
    // nothing: its clamped row iend - 1 would lie outside the order's rows
    if (imin < iend) {
        const int comp = lane % CW;
        const bool is_a = comp < NC;
        const double *base = is_a ? ap + comp : reinterpret_cast<const double *>(sc + t + 2) + min(comp - NC, 1);
        const unsigned stride = is_a ? (unsigned)astride : 8u;
        const double *fb = reinterpret_cast<const double *>(sc + t) + 2;
        const double f1 = is_a ? 1.0 : 0.0, f0 = 1.0 - f1;  // factor of a staged value: f_l, or 1
        double pre[E], fac[E];
        auto fetch = [&](int c0) {
#pragma unroll
            for (int e = 0; e < E; e++) {
                const unsigned i = (unsigned)min(c0 + (lane + 64 * e) / CW, iend - 1);
                pre[e] = base[(size_t)i * stride];
                fac[e] = fb[8 * (size_t)i];
            }
        };
        auto stage = [&](int sl, int c0) {
#pragma unroll
            for (int e = 0; e < E; e++) stg[sl * CS + lane + 64 * e] = pre[e] * __builtin_fma(fac[e], f1, f0);
            if (c0 + kChunk > iend) {
#pragma unroll
                for (int e = 0; e < E; e++)
                    if (c0 + (lane + 64 * e) / CW >= iend) stg[sl * CS + lane + 64 * e] = 0.0;
            }
        };
        int c0 = imin & ~(kChunk - 1), sl = 0;
        fetch(c0);
#pragma unroll
        for (int r = 0; r < R; r++) {
            const int i = i0[r] < iend ? i0[r] : imin;
            double2 v = st[r * 64 + lane];
            v.x *= sc[t + 2 * i].w;
            v.y *= sc[t + 2 * i + 2].w;
            st[r * 64 + lane] = v;
        }
        stage(0, c0);
        fetch(c0 + kChunk);
        // The rings that start at imin; a first chunk that begins before imin
        // runs row by row, every later chunk as eight unrolled steps (rows past
        // iend are staged as zeros, which leave the sums unchanged).
#pragma unroll
        for (int r = 0; r < R; r++)
            if (i0[r] == imin) {
                const double2 v = st[r * 64 + lane];
                P0[r] = v.x;
                P1[r] = v.y;
            }
        if (c0 != imin) {
            const int ce = min(iend, c0 + kChunk);
            for (int i = imin; i < ce; i++) {
                const double *row = stg + (i - c0) * CW + (lane & 15);
                const double rv = row[0];
                step_v(rv, CW == 16 ? rv : row[16]);
            }
            stage(1, c0 + kChunk);
            fetch(c0 + 2 * kChunk);
            c0 += kChunk;
            sl = 1;
        }
        for (; c0 < iend; c0 += kChunk, sl ^= 1) {
#pragma unroll
            for (int r = 0; r < R; r++)
                if (i0[r] == c0) {
                    const double2 v = st[r * 64 + lane];
                    P0[r] = v.x;
                    P1[r] = v.y;
                }
            // four rows are read at once (one or two values per lane and row),
            // so that their LDS latency is paid twice per chunk
            const double *cur = stg + sl * CS + (lane & 15);
#pragma unroll
            for (int u0 = 0; u0 < kChunk; u0 += 4) {
                double rv[4], rc[4];
#pragma unroll
                for (int u = 0; u < 4; u++) {
                    rv[u] = cur[(u0 + u) * CW];
                    rc[u] = CW == 16 ? rv[u] : cur[(u0 + u) * CW + 16];
                }
#pragma unroll
                for (int u = 0; u < 4; u++) step_v(rv[u], rc[u]);
            }
            stage(sl ^ 1, c0 + kChunk);
            fetch(c0 + 2 * kChunk);
        }
    }
    // The results leave as whole entries: through LDS, 16-byte units swizzled by
    // the ring, so that a store instruction covers 64 consecutive units and not
    // 16 bytes of each of 64 entries.
    constexpr int V = 16 / sizeof(S), U = NC / V;  // values per unit, units per ring
    S *out = slot + (size_t)outb * a.ES + col0;
    if constexpr (U > 1) {
        typedef S unit_t __attribute__((ext_vector_type(V), aligned(sizeof(S))));
        typedef S lds_t __attribute__((ext_vector_type(V)));
        lds_t *tile = reinterpret_cast<lds_t *>(stg);
        static_assert(64 * U * 16 <= sizeof(double) * bf_res_stage_doubles<NB>(), "a tile of 64 rings");
#pragma unroll
        for (int r = 0; r < R; r++) {
            __builtin_amdgcn_wave_barrier();
#pragma unroll
            for (int u = 0; u < U; u++) {
                lds_t x;
#pragma unroll
                for (int v = 0; v < V; v++) x[v] = (S)acc[r][u * V + v];
                tile[lane * U + (u ^ (lane & (U - 1)))] = x;
            }
            __builtin_amdgcn_wave_barrier();
#pragma unroll
            for (int u = 0; u < U; u++) {
                const int j = (64 * u + lane) / U, c = lane & (U - 1);
                if (r * 64 + j < nl)
                    *reinterpret_cast<unit_t *>(out + (size_t)(r * 64 + j) * a.ES + c * V) = tile[j * U + (c ^ (j & (U - 1)))];
            }
        }
    } else {
#pragma unroll
        for (int r = 0; r < R; r++) {
            const int j = r * 64 + lane;
            if (j < nl) {
#pragma unroll
                for (int c = 0; c < NC; c++) out[(size_t)j * a.ES + c] = (S)acc[r][c];
            }
        }
    }
}

// One wave per residual piece (up to kBfPieceRings skeleton rings of one
// task): short waves keep the register count, and with it the occupancy, low.
template <int NB, typename S>
__device__ __forceinline__ void residual_piece(const BfArgs<S> &a, long long tk, int lane, double *stg, int col0) {
    const int4 h = a.res_sub[2 * tk], h2 = a.res_sub[2 * tk + 1];
    const int t = __builtin_amdgcn_readfirstlane(h.x), imin = __builtin_amdgcn_readfirstlane(h.y);
    const int iend = __builtin_amdgcn_readfirstlane(h.z), nl = __builtin_amdgcn_readfirstlane(h.w);
    const int outb = __builtin_amdgcn_readfirstlane(h2.x), m = __builtin_amdgcn_readfirstlane(h2.y);
    const long long lbase = (unsigned)__builtin_amdgcn_readfirstlane(h2.z);
    const size_t aoff = (size_t)m * (2 * a.L + 3 - m) / 2;
    const double *ap = reinterpret_cast<const double *>(a.alm + (aoff + t) * a.nmaps + a.map0);
    const double4 *sc = reinterpret_cast<const double4 *>(a.coef_sc) + a.coef_off[m];
    const int astride = 4 * a.nmaps;  // doubles between rows i and i+1
    residual_task<NB, kBfPieceRings / 64>(a, a.ws, lbase, lane, t, imin, iend, nl, outb, ap, sc, astride, stg,
                                          col0);
}

template <int NB, typename S>
__global__ __launch_bounds__(kBfResThreads) void k_bf_residual(BfArgs<S> a, long long t0, long long t1, int col0) {
    __shared__ __align__(16) double stg_all[kBfResThreads / 64][bf_res_stage_doubles<NB>()];
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const long long tk = t0 + (long long)blockIdx.x * (kBfResThreads / 64) + w;
    if (tk >= t1) return;
    residual_piece<NB, S>(a, tk, threadIdx.x & 63, stg_all[w], col0);
}

// The groups of a pass, two at a time where there are two.
template <bool ONE, typename F>
__device__ __forceinline__ void for_groups(int G, F &&group) {
    typedef std::integral_constant<Pair, Pair::NONE> none_t;
    if constexpr (ONE) {
        group(none_t{}, 0);
    } else {
        int g = 0;
        for (; g + 1 < G; g += 2) {
            group(std::integral_constant<Pair, Pair::AHEAD>{}, g);
            group(std::integral_constant<Pair, Pair::DONE>{}, g + 1);
        }
        if (g < G) group(none_t{}, g);
    }
}

// One workgroup of 2 kBfHalves waves per pair node (wave w: child w % 2,
// half w / 2): per group of NB maps, each child writes its share of u into
// its own LDS copy, and the two copies are summed into the next level's
// vector with one coalesced store.

template <int NB, typename S, bool ONE>
__device__ __forceinline__ void level_node_g(const BfArgs<S> &a, int node) {
    constexpr int NC = 2 * NB;
    extern __shared__ char lds_raw[];
    S *u0 = reinterpret_cast<S *>(lds_raw);
    const int *ni = a.node_i + (size_t)node * kBfNodeInts;
    const int n = ni[2] + ni[4];
    S *u1 = u0 + (size_t)n * NC;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int ES = ONE ? NC : a.ES, G = ONE ? 1 : a.G;
    S *__restrict__ out = a.ws + (size_t)ni[6] * ES;
    typename Acc<S>::type next[4];
    auto group = [&](auto pair, int g) {
        if (g) __syncthreads();  // the previous group's sums have been read out of LDS
        id_block<NB, S, ONE, decltype(pair)::value>(a, node, w & 1, w >> 1, threadIdx.x & 63, (w & 1) ? u1 : u0, g * NC,
                                                    next);
        __syncthreads();
        if (ONE) {
            for (int e = threadIdx.x; e < n * NC; e += kBfLevelThreads) out[e] = u0[e] + u1[e];
        } else {
            for (int e = threadIdx.x; e < n * NC; e += kBfLevelThreads)
                out[(size_t)(e / NC) * ES + g * NC + e % NC] = u0[e] + u1[e];
        }
    };
    for_groups<ONE>(G, group);
}

// ONE: the pass has a single group of maps (separate instantiations, so the
// common case keeps its constant strides and its register count).
template <int NB, typename S, bool ONE>
__global__ __launch_bounds__(kBfLevelThreads, ONE ? 1 : 3) void k_bf_level(BfArgs<S> a, long long n0) {
    level_node_g<NB, S, ONE>(a, (int)(n0 + blockIdx.x));
}

// Level-1 nodes that run alone (their order is folded afterwards).
template <int NB, typename S, bool ONE>
__global__ __launch_bounds__(kBfLevelThreads) void k_bf_level_list(BfArgs<S> a, const int *__restrict__ list,
                                                                   long long n0) {
    level_node_g<NB, S, ONE>(a, list[n0 + blockIdx.x]);
}

// Level 1 fused with the even/odd fold (Eqs. 13-14): one workgroup per unit
// {even node, odd node, first ring k0, slot}; both nodes cover the rings
// k0 .. k0+n-1 of one order, so q^even and q^odd of those rings meet in LDS
// and q(z) = q^e + q^o, q(-z) = q^e - q^o go straight to q.
constexpr int kBfFoldThreads = 2 * kBfLevelThreads;

template <int NB, typename S, bool ONE>
__global__ __launch_bounds__(kBfFoldThreads, ONE ? 1 : 3) void k_bf_level1_fold(BfArgs<S> a, const int4 *__restrict__ units,
                                                                   long long u0, int batch, int nbatch) {
    constexpr int NC = 2 * NB;
    extern __shared__ char lds_raw[];
    const int4 un = units[u0 + blockIdx.x];
    const int *nie = a.node_i + (size_t)un.x * kBfNodeInts;
    const int n = nie[2] + nie[4];
    S *uE = reinterpret_cast<S *>(lds_raw);  // even node: children 0 and 1, then the odd node's
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int par = w / (2 * kBfHalves), wc = w % (2 * kBfHalves);
    const int m = batch + un.w * nbatch, k0 = un.z;
    const int G = ONE ? 1 : a.G;
    typename Acc<S>::type next[4];
    auto group = [&](auto pair, int g) {
        if (g) __syncthreads();  // the previous group's fold has read LDS
        id_block<NB, S, ONE, decltype(pair)::value>(a, par ? un.y : un.x, wc & 1, wc >> 1, threadIdx.x & 63,
                                                    uE + (size_t)(2 * par + (wc & 1)) * n * NC, g * NC, next);
        __syncthreads();
        const int mb = a.map0 + g * NB;
        for (int e = threadIdx.x; e < n * NB; e += kBfFoldThreads) {
            const int c = e / NB, b = e % NB;
            const S *e0 = uE + c * NC + 2 * b, *e1 = e0 + (size_t)n * NC, *o0 = e1 + (size_t)n * NC,
                    *o1 = o0 + (size_t)n * NC;
            double er = (double)(e0[0] + e1[0]), ei = (double)(e0[1] + e1[1]);
            double orr = (double)(o0[0] + o1[0]), oi = (double)(o0[1] + o1[1]);
            if (m == 0) ei = oi = 0.0;  // real field: Im a_l0 is ignored
            const int k = k0 + c, ks = a.nrings - 1 - k;
            a.q[((size_t)k * (a.L + 1) + m) * a.nmaps + mb + b] = make_double2(er + orr, ei + oi);
            if (ks != k) a.q[((size_t)ks * (a.L + 1) + m) * a.nmaps + mb + b] = make_double2(er - orr, ei - oi);
        }
    };
    for_groups<ONE>(G, group);
}

// Fold of the listed slots of one batch: slot j holds order m = batch + j nbatch.
template <typename S>
__global__ __launch_bounds__(kBfThreads) void k_bf_fold(BfArgs<S> a, int batch, int nbatch, const int *__restrict__ slots,
                                                        int count) {
    const int K = a.K, NP = a.ES / 2;  // maps of the pass
    const long long e = (long long)blockIdx.x * kBfThreads + threadIdx.x;
    if (e >= (long long)count * K * NP) return;
    const int b = (int)(e % NP);
    const long long jk = e / NP;
    const int k = (int)(jk % K), j = slots[jk / K];
    const int m = batch + j * nbatch;
    const S *qe = a.ws + ((size_t)(2 * j) * K + k) * a.ES + 2 * b;
    const S *qo = a.ws + ((size_t)(2 * j + 1) * K + k) * a.ES + 2 * b;
    double er = (double)qe[0], ei = (double)qe[1], orr = (double)qo[0], oi = (double)qo[1];
    if (m == 0) ei = oi = 0.0;  // real field: Im a_l0 is ignored
    a.q[((size_t)k * (a.L + 1) + m) * a.nmaps + a.map0 + b] = make_double2(er + orr, ei + oi);
    const int ks = a.nrings - 1 - k;
    if (ks != k) a.q[((size_t)ks * (a.L + 1) + m) * a.nmaps + a.map0 + b] = make_double2(er - orr, ei - oi);
}

// ---- work-queue batches: one launch per stage for every request pass of
// one map-group width; item = {pass (argument block), index within the
// pass's plan}.  The bodies are the single-request kernels'.
template <int NB, typename S>
__global__ __launch_bounds__(kBfResThreads) void k_bfq_residual(const BfArgs<S> *__restrict__ args,
                                                             const int2 *__restrict__ items, long long n) {
    __shared__ __align__(16) double stg_all[kBfResThreads / 64][bf_res_stage_doubles<NB>()];
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const long long j = (long long)blockIdx.x * (kBfResThreads / 64) + w;
    if (j >= n) return;
    const int2 it = items[j];
    const BfArgs<S> a = args[__builtin_amdgcn_readfirstlane(it.x)];
    residual_piece<NB, S>(a, __builtin_amdgcn_readfirstlane(it.y), threadIdx.x & 63, stg_all[w], 0);
}

// items {pass, node}: level nodes, and level-1 nodes that run alone
template <int NB, typename S>
__global__ __launch_bounds__(kBfLevelThreads) void k_bfq_level(const BfArgs<S> *__restrict__ args,
                                                               const int2 *__restrict__ items) {
    const int2 it = items[blockIdx.x];
    const BfArgs<S> a = args[__builtin_amdgcn_readfirstlane(it.x)];
    level_node_g<NB, S, true>(a, __builtin_amdgcn_readfirstlane(it.y));
}

// items {pass, fused level-1 unit}
template <int NB, typename S>
__global__ __launch_bounds__(kBfFoldThreads) void k_bfq_level1_fold(const BfArgs<S> *__restrict__ args,
                                                                    const int2 *__restrict__ items) {
    constexpr int NC = 2 * NB;
    extern __shared__ char lds_raw[];
    const int2 it = items[blockIdx.x];
    const BfArgs<S> a = args[__builtin_amdgcn_readfirstlane(it.x)];
    const int4 un = a.f1_unit[__builtin_amdgcn_readfirstlane(it.y)];
    const int *nie = a.node_i + (size_t)un.x * kBfNodeInts;
    const int n = nie[2] + nie[4];
    S *uE = reinterpret_cast<S *>(lds_raw);
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int par = w / (2 * kBfHalves), wc = w % (2 * kBfHalves);
    const int m = un.w, k0 = un.z;  // one order batch: slot j holds order j
    typename Acc<S>::type next[4];
    id_block<NB, S, true>(a, par ? un.y : un.x, wc & 1, wc >> 1, threadIdx.x & 63,
                          uE + (size_t)(2 * par + (wc & 1)) * n * NC, 0, next);
    __syncthreads();
    for (int e = threadIdx.x; e < n * NB; e += kBfFoldThreads) {
        const int c = e / NB, b = e % NB;
        const S *e0 = uE + c * NC + 2 * b, *e1 = e0 + (size_t)n * NC, *o0 = e1 + (size_t)n * NC,
                *o1 = o0 + (size_t)n * NC;
        double er = (double)(e0[0] + e1[0]), ei = (double)(e0[1] + e1[1]);
        double orr = (double)(o0[0] + o1[0]), oi = (double)(o0[1] + o1[1]);
        if (m == 0) ei = oi = 0.0;  // real field: Im a_l0 is ignored
        const int k = k0 + c, ks = a.nrings - 1 - k;
        a.q[((size_t)k * (a.L + 1) + m) * a.nmaps + a.map0 + b] = make_double2(er + orr, ei + oi);
        if (ks != k) a.q[((size_t)ks * (a.L + 1) + m) * a.nmaps + a.map0 + b] = make_double2(er - orr, ei - oi);
    }
}

// items {pass, block of kBfThreads fold elements}
template <typename S>
__global__ __launch_bounds__(kBfThreads) void k_bfq_fold(const BfArgs<S> *__restrict__ args,
                                                         const int2 *__restrict__ items) {
    const int2 it = items[blockIdx.x];
    const BfArgs<S> a = args[__builtin_amdgcn_readfirstlane(it.x)];
    const int K = a.K, NP = a.ES / 2;
    const long long e = (long long)__builtin_amdgcn_readfirstlane(it.y) * kBfThreads + threadIdx.x;
    if (e >= (long long)a.fold_count * K * NP) return;
    const int b = (int)(e % NP);
    const long long jk = e / NP;
    const int k = (int)(jk % K), j = a.fold_slot[jk / K];
    const int m = j;
    const S *qe = a.ws + ((size_t)(2 * j) * K + k) * a.ES + 2 * b;
    const S *qo = a.ws + ((size_t)(2 * j + 1) * K + k) * a.ES + 2 * b;
    double er = (double)qe[0], ei = (double)qe[1], orr = (double)qo[0], oi = (double)qo[1];
    if (m == 0) ei = oi = 0.0;
    a.q[((size_t)k * (a.L + 1) + m) * a.nmaps + a.map0 + b] = make_double2(er + orr, ei + oi);
    const int ks = a.nrings - 1 - k;
    if (ks != k) a.q[((size_t)ks * (a.L + 1) + m) * a.nmaps + a.map0 + b] = make_double2(er - orr, ei - oi);
}

template <int NB, typename S>
static hipError_t bfq_stage_nb(int stage, const void *args, const int2 *items, long long n, size_t lds, hipStream_t st) {
    const BfArgs<S> *ar = reinterpret_cast<const BfArgs<S> *>(args);
    constexpr int WPB = kBfResThreads / 64;
    if (n <= 0) return hipSuccess;
    switch (stage) {
        case 0:
            hipLaunchKernelGGL((k_bfq_residual<NB, S>), dim3((unsigned)((n + WPB - 1) / WPB)), dim3(kBfResThreads), 0, st, ar,
                               items, n);
            break;
        case 1:
            hipLaunchKernelGGL((k_bfq_level<NB, S>), dim3((unsigned)n), dim3(kBfLevelThreads), lds, st, ar, items);
            break;
        case 2:
            hipLaunchKernelGGL((k_bfq_level1_fold<NB, S>), dim3((unsigned)n), dim3(kBfFoldThreads), lds, st, ar, items);
            break;
        default:
            hipLaunchKernelGGL((k_bfq_fold<S>), dim3((unsigned)n), dim3(kBfThreads), 0, st, ar, items);
            break;
    }
    return hipGetLastError();
}

// One stage launch of a work-queue batch: stage 0 residual pieces, 1 level
// nodes (lds: widest column set), 2 fused level-1 units, 3 fold blocks.
hipError_t launch_bf_queue_stage(int stage, int nb, int fp32, const void *args, const int2 *items, long long n,
                                 size_t lds, hipStream_t st) {
    if (n > 0x7fffffffLL) return hipErrorInvalidValue;
    if (fp32) {
        switch (nb) {
            case 8: return bfq_stage_nb<8, float>(stage, args, items, n, lds, st);
            case 4: return bfq_stage_nb<4, float>(stage, args, items, n, lds, st);
            case 2: return bfq_stage_nb<2, float>(stage, args, items, n, lds, st);
            default: return bfq_stage_nb<1, float>(stage, args, items, n, lds, st);
        }
    }
    switch (nb) {
        case 8: return bfq_stage_nb<8, double>(stage, args, items, n, lds, st);
        case 4: return bfq_stage_nb<4, double>(stage, args, items, n, lds, st);
        case 2: return bfq_stage_nb<2, double>(stage, args, items, n, lds, st);
        default: return bfq_stage_nb<1, double>(stage, args, items, n, lds, st);
    }
}

// The argument block of one pass of a work-queue batch (G = 1, nb maps).
size_t bf_args_bytes(int fp32) { return fp32 ? sizeof(BfArgs<float>) : sizeof(BfArgs<double>); }
void bf_queue_args(const sht_plan_s *p, int nmaps, int map0, int nb, int fp32, const double *alm, double *q, void *ws,
                   void *out) {
    if (fp32) {
        BfArgs<float> a = bf_args<float>(p, nmaps, p->d_bf_T32, (float *)ws);
        a.alm = reinterpret_cast<const double2 *>(alm);
        a.q = reinterpret_cast<double2 *>(q);
        a.map0 = map0;
        a.ES = 2 * nb;
        a.G = 1;
        std::memcpy(out, &a, sizeof(a));
    } else {
        BfArgs<double> a = bf_args<double>(p, nmaps, p->d_bf_T, (double *)ws);
        a.alm = reinterpret_cast<const double2 *>(alm);
        a.q = reinterpret_cast<double2 *>(q);
        a.map0 = map0;
        a.ES = 2 * nb;
        a.G = 1;
        std::memcpy(out, &a, sizeof(a));
    }
}

// dynamic LDS of a level node / fused unit with n columns
size_t bf_level_lds_bytes(int n, int nb, int fp32) {
    return (size_t)n * 2 * (2 * nb * (fp32 ? sizeof(float) : sizeof(double)));
}

size_t bf_scratch_bytes(const sht_plan_s *p, int nmaps, int fp32) {
    return (size_t)p->bf.ws_entries * bf_entry_values(nmaps) * (fp32 ? sizeof(float) : sizeof(double));
}

// Records the caller's stage event (which = 0 before, 1 after) if given.
static void bf_event(void *const *ev, int stage, int which, hipStream_t st) {
    if (ev && ev[2 * stage + which]) (void)hipEventRecord((hipEvent_t)ev[2 * stage + which], st);
}

template <int NB, typename S, bool ONE>
static hipError_t launch_bf_nbg(const sht_plan_s *p, BfArgs<S> a, hipStream_t st, void *const *ev) {
    constexpr int WPB = kBfResThreads / 64;
    const BflyPlan &b = p->bf;
    if (b.nbatch != 1) ev = nullptr;
    for (int bt = 0; bt < b.nbatch; bt++) {
        const long long t0 = b.batch_sub[bt], t1 = b.batch_sub[bt + 1];
        bf_event(ev, SHT_STAGE_BF_RESIDUAL, 0, st);
        for (int g = 0; g < a.G && t1 > t0; g++) {  // one launch per group of NB maps
            BfArgs<S> ag = a;
            ag.map0 = a.map0 + g * NB;
            hipLaunchKernelGGL((k_bf_residual<NB, S>), dim3((unsigned)((t1 - t0 + WPB - 1) / WPB)), dim3(kBfResThreads), 0,
                               st, ag, t0, t1, g * 2 * NB);
        }
        bf_event(ev, SHT_STAGE_BF_RESIDUAL, 1, st);
        bf_event(ev, SHT_STAGE_BF_LEVELS, 0, st);
        const long long *lo = b.lv_off.data() + (size_t)bt * (kBfMaxLv + 1);
        for (int q = 0; q < kBfMaxLv - 1; q++) {  // levels >= 2
            const long long n0 = lo[q], n1 = lo[q + 1];
            if (n1 <= n0) continue;
            // LDS for the widest column set of this level only
            const size_t lds = bf_level_lds<NB, S>(b.lv_max_n[(size_t)bt * kBfMaxLv + q]);
            hipLaunchKernelGGL((k_bf_level<NB, S, ONE>), dim3((unsigned)(n1 - n0)), dim3(kBfLevelThreads), lds, st, a,
                               n0);
        }
        bf_event(ev, SHT_STAGE_BF_LEVELS, 1, st);
        // level 1: fused with the fold where both parities have levels
        const size_t lds1 = bf_level_lds<NB, S>(b.lv_max_n[(size_t)bt * kBfMaxLv + kBfMaxLv - 1]);
        const long long p0 = b.l1_off[bt], p1 = b.l1_off[bt + 1];
        if (p1 > p0)
            hipLaunchKernelGGL((k_bf_level_list<NB, S, ONE>), dim3((unsigned)(p1 - p0)), dim3(kBfLevelThreads), lds1, st, a,
                               p->d_bf_l1_plain, p0);
        const long long f0 = b.f1_off[bt], f1 = b.f1_off[bt + 1];
        if (f1 > f0)
            hipLaunchKernelGGL((k_bf_level1_fold<NB, S, ONE>), dim3((unsigned)(f1 - f0)), dim3(kBfFoldThreads), 2 * lds1, st,
                               a, reinterpret_cast<const int4 *>(p->d_bf_f1_unit), f0, bt, b.nbatch);
        const long long s0 = b.fold_off[bt], s1 = b.fold_off[bt + 1];
        const long long nf = (s1 - s0) * b.K * (a.ES / 2);
        if (nf > 0)
            hipLaunchKernelGGL((k_bf_fold<S>), dim3((unsigned)((nf + kBfThreads - 1) / kBfThreads)),
                               dim3(kBfThreads), 0, st, a, bt, b.nbatch, p->d_bf_fold_slot + s0, (int)(s1 - s0));
    }
    return hipGetLastError();
}

// The residual kernel over another task list (the interpolation form's node
// tasks): a.res_sub, res_lane, res_val and z2 describe the tasks; one launch
// for a pass of nb maps (G = 1).
hipError_t launch_node_phase(const sht_plan_s *p, int nb, BfArgs<double> a, long long npieces, hipStream_t st) {
    (void)p;
    constexpr int WPB = kBfResThreads / 64;
    if (npieces <= 0) return hipSuccess;
    const dim3 grid((unsigned)((npieces + WPB - 1) / WPB));
    switch (nb) {
        case 4: hipLaunchKernelGGL((k_bf_residual<4, double>), grid, dim3(kBfResThreads), 0, st, a, 0LL, npieces, 0); break;
        case 2: hipLaunchKernelGGL((k_bf_residual<2, double>), grid, dim3(kBfResThreads), 0, st, a, 0LL, npieces, 0); break;
        default: hipLaunchKernelGGL((k_bf_residual<1, double>), grid, dim3(kBfResThreads), 0, st, a, 0LL, npieces, 0); break;
    }
    return hipGetLastError();
}

template <int NB, typename S>
static hipError_t launch_bf_nb(const sht_plan_s *p, BfArgs<S> a, hipStream_t st, void *const *ev) {
    return a.G == 1 ? launch_bf_nbg<NB, S, true>(p, a, st, ev) : launch_bf_nbg<NB, S, false>(p, a, st, ev);
}

template <typename S>
static hipError_t launch_bf(const sht_plan_s *p, int nmaps, const double *alm, double *q, S *ws, const S *T,
                            hipStream_t st, void *const *ev) {
    BfArgs<S> a = bf_args<S>(p, nmaps, T, ws);
    a.alm = reinterpret_cast<const double2 *>(alm);
    a.q = reinterpret_cast<double2 *>(q);
    hipError_t e = hipSuccess;
    for (int b = 0; b < nmaps && e == hipSuccess;) {
        int nb, groups;
        bf_pass_shape(nmaps - b, &nb, &groups);
        a.map0 = b;
        a.G = groups;
        a.ES = 2 * nb * groups;
        switch (nb) {
            case 8: e = launch_bf_nb<8, S>(p, a, st, ev); break;
            case 4: e = launch_bf_nb<4, S>(p, a, st, ev); break;
            case 2: e = launch_bf_nb<2, S>(p, a, st, ev); break;
            default: e = launch_bf_nb<1, S>(p, a, st, ev); break;
        }
        b += nb * groups;
    }
    return e;
}

hipError_t launch_butterfly(const sht_plan_s *p, int nmaps, const double *alm, double *q, void *scratch,
                            int fp32, hipStream_t stream, void *const *stage_events) {
    if (fp32) return launch_bf<float>(p, nmaps, alm, q, (float *)scratch, p->d_bf_T32, stream, stage_events);
    return launch_bf<double>(p, nmaps, alm, q, (double *)scratch, p->d_bf_T, stream, stage_events);
}

}  // namespace sht
