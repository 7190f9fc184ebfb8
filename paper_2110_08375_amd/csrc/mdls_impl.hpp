// mdls_impl.hpp -- MI355X (gfx950) kernels and host drivers of the multiple-double least-squares
// path; instantiated once per precision (mdls_p<P>.hip) and called by the C ABI (mdls_capi.hip).
//
// Hot path of a solve (paper Section 1: A = QR turns A x = b into R x = Q^T b):
//   QR (Section 3, Algorithm 2) as a sequence of narrow Householder panels.  For each panel of
//   W columns:
//     k_panel  -- Householder vectors and betas column by column (Golub-Van Loan 5.1.1 sign
//                 choice), the in-panel reflector updates, and the panel's compact-WY factor T
//                 (H_0 ... H_{W-1} = I - Y T Y^T, so the paper's W = -Y T).  The panel's rows
//                 stay in registers across all its columns; one workgroup reduction (and, when
//                 the panel spans several workgroups, one exchange of tagged words) per column.
//     k_step   -- a panel and the previous panel's trailing update in one launch (double, dd and
//                 qd while their rows fit); elsewhere the update is
//     k_apply_s, k_apply_t, k_apply_u -- the trailing update C := C + Y (W^T C) =
//                 C - Y T^T (Y^T C) (paper's "YWT*C" and "R + YWTC" fused), applied to every
//                 column right of the panel and to the right-hand side, so Q^T b comes out of
//                 the factorisation.
//   Back substitution (Section 2, Algorithm 1):
//     k_trsv   -- one launch, a workgroup per block of rows: its diagonal block inverted, the x of
//                 the blocks below taken as they are published, b_j -= A_{j,i} x_i, x_j := U_j^{-1} b_j;
//     k_invert, k_inv_blocks, k_bs_xi, k_bs_upd -- the tiled form, for the sizes where it is the faster
//                 one (backsub_by_tiles) and for the refined solve, whose corrections use the diagonal
//                 tiles' inverses again: the inverses, then per tile x_i := U_i^{-1} b_i and b_j -= A_{j,i} x_i
//                 for every j < i at once.
//   Q^T B and Q B: k_gemm, k_trmm_v and k_nn_sub_v, in blocks of outputs.
//
// Multiple-double numbers are P limb planes (limb 0 most significant); see md.hpp for the
// arithmetic.
#include <algorithm>
#include <climits>
#include <cmath>
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <functional>
#include <queue>
#include <type_traits>
#include <vector>

#pragma once
#include "mdls.h"
#include "md_lanes.hpp"
#include "mdls_kernels.hpp"
#include "mdls_split_kernels.hpp"

namespace mdls_impl {
using namespace mdk;

// ============================================================================ panel kernel
struct PanelArgs {
    double *A;  // panel column 0 at row (diagonal - off); the panel's diagonal is row off
    long lda, ps;
    int h, wact;   // rows from the diagonal down, active columns (<= W)
    int off;       // W when the previous panel is applied first (rows above the diagonal), else 0
    const double *Yp;  // previous panel's diagonal element (its Y, unit lower trapezoidal), if off
    const double *Tp;  // previous panel's T (W x W, ld W), plane stride tps
    double *beta;  // beta of the panel's first column, plane stride bps
    long bps;
    double *T;  // panel T, W x W column-major (ld W), plane stride tps
    long tps;
    double *gpart;  // [G][W*W][P] look-ahead sums of the workgroups
    unsigned *gbar; // barrier counter of this launch, zero on entry
    unsigned long long *gtag;  // tagged words of the per-column exchange (tag_words), no word of them tagged
                               // tag0 + 1 .. tag0 + wact on entry
    unsigned tag0;  // column index of the panel's first column
    int *err;       // set to 1 if a wait times out
    int G;          // workgroups in the launch
    unsigned spin;  // polls before a wait gives up
};

// Entry (r, c) of a block of Householder vectors stored below the diagonal of A: zero above
// the diagonal, the implicit one on it, the stored value below; zero outside h x wact.
template <int P>
__device__ __forceinline__ V<P> y_entry(const double *Y, long ldy, long psy, long r, int c, int h, int wact)
{
    if (r >= h || c >= wact || r < c) return zero<P>();
    if (r == c) return from_double<P>(1.0);
    return ldm<P>(Y, psy, (long)c * ldy + r);
}

// All workgroups of the launch meet here (called by one whole wave per workgroup).  The
// spin is bounded (spin polls, each after a short sleep): a timed-out barrier raises *err and
// lets the wave continue, so the grid always drains; the host turns *err into a status.
__device__ inline void grid_sync(unsigned *ctr, unsigned target, int *err, unsigned spin)
{
    const int lane = threadIdx.x & 63;
    // the fence before the relaxed arrival releases this workgroup's stores; the relaxed
    // polls need no cache invalidation each, the fence after them acquires the others' stores
    // (a release and an acquire fence: neither side needs the other half of a full fence)
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
    if (lane == 0) {
        __hip_atomic_fetch_add(ctr, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        unsigned spins = 0;
        while (__hip_atomic_load(ctr, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < target) {
            __builtin_amdgcn_s_sleep(1);
            if (++spins > spin) {
                __hip_atomic_store(err, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                break;
            }
        }
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
}

// The per-column exchange between the workgroups of a panel.  Each double goes out as two 8-byte
// words, a 32-bit half beside the 32-bit number of the column, stored and loaded with relaxed
// agent-scope atomics: a word that carries the number awaited is the word of that column, so the
// data are their own flag and one round trip replaces the counter's release fence (a write-back of
// the XCD's L2), arrival, polls and the loads after them.  Slots alternate with the column's parity:
// a workgroup that publishes column j has read every workgroup's column j - 1, which those published
// after they had read column j - 2.  Word w (limb w / 2, low half if w is odd) of column l from
// workgroup b is at w G W + b W + l of its parity's half, the head row a_jl of workgroup 0 behind them.
// n = 1024: dd panel 82 -> 71 us, qd 88 -> 75 us (16 and 8 columns) against the counter barrier.
template <int P, int W>
__host__ __device__ constexpr int tag_words(int G)  // both parities
{
    return 4 * P * W * (G + 1);
}

__device__ __forceinline__ void st_tagged(unsigned long long *p, long stride, double v, unsigned tag)
{
    const unsigned long long u = (unsigned long long)__double_as_longlong(v), t = (unsigned long long)tag << 32;
    __hip_atomic_store(p, t | (u >> 32), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_store(p + stride, t | (u & 0xffffffffull), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ double tagged_value(unsigned long long hi, unsigned long long lo)
{
    return __longlong_as_double((long long)((hi << 32) | (lo & 0xffffffffull)));
}

// One whole wave: loads the words of up to N items (item u of lane i at base + off[u] + w stride, u
// taken where act[u]) until all of them carry the tag.  The polls are bounded (no sleep between them: a poll
// takes as long, 0.18 us, with the sleep of grid_sync), and once another wait has given up every 256th poll
// gives up too; a time-out raises *err.
template <int P, int N>
__device__ __forceinline__ void poll_tagged(const unsigned long long *base, const long (&off)[N], const long (&stride)[N],
                                            const bool (&act)[N], unsigned tag, unsigned long long (&wd)[N][2 * P],
                                            int *err, unsigned spin)
{
    unsigned spins = 0;
    for (;;) {
#pragma unroll
        for (int u = 0; u < N; ++u)
#pragma unroll
            for (int w = 0; w < 2 * P; ++w)
                wd[u][w] = act[u] ? __hip_atomic_load(base + off[u] + w * stride[u], __ATOMIC_RELAXED,
                                                      __HIP_MEMORY_SCOPE_AGENT)
                                  : (unsigned long long)tag << 32;
        bool ok = true;
#pragma unroll
        for (int u = 0; u < N; ++u)
#pragma unroll
            for (int w = 0; w < 2 * P; ++w) ok = ok && (unsigned)(wd[u][w] >> 32) == tag;
        if (__all(ok)) break;
        if ((spins & 255u) == 255u && __hip_atomic_load(err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0) break;
        if (++spins > spin) {
            __hip_atomic_store(err, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            break;
        }
    }
}

// Sum over a workgroup of per-thread partials of WW pairs: thread t holds a partial of pair
// t % WW.  Partials of one pair inside a wave are combined with a butterfly, those of
// different waves through LDS; out[q] (LDS, WW x P doubles) receives the renormalised total,
// negated if NEG.  Called by every thread; ends with a workgroup barrier.
template <int P, int WW, int NT, bool NEG>
__device__ __forceinline__ void pair_sum(Acc<P> t, double *s_comb, double *out)
{
    constexpr int WV = (WW < 64) ? 64 : WW;  // threads that hold each pair once
    constexpr int NP = NT / WV;              // partials per pair left after the butterfly
    static_assert(NT % WV == 0, "pair_sum layout");
    const int tid = threadIdx.x;
#pragma unroll
    for (int m = WW; m < 64; m <<= 1) acc_add_acc(t, shfl_xor_acc(t, m));
    if (tid % WV < WW) {
#pragma unroll
        for (int k = 0; k < P; ++k) s_comb[((tid / WV) * WW + tid % WV) * P + k] = t.s[k];
    }
    __syncthreads();
    for (int q = tid; q < WW; q += NT) {
        Acc<P> s = acc_zero<P>();
        for (int k = 0; k < NP; ++k) {
            Acc<P> o;
#pragma unroll
            for (int e = 0; e < P; ++e) o.s[e] = s_comb[(k * WW + q) * P + e];
            acc_add_acc(s, o);
        }
        const V<P> v = acc_get(s);
        lds_st(&out[q * P], NEG ? neg(v) : v);
    }
    __syncthreads();
}

// Sum of NA lazy accumulators per lane over the row-slot bits of a wave (lane masks 32, 16,
// ..., MMIN): while a lane holds two or more accumulators each level halves the set (the
// partner keeps the other half), then plain butterfly levels follow.  Lane l keeps
// slot_scatter_kept<W>() accumulators, starting at index slot_scatter_index<W>(l); equal
// totals sit on the lanes that differ only in slot_plain_mask bits.
template <int P, int NA, int NH, int MMIN, int M>
__device__ __forceinline__ void slot_scatter(Acc<P> (&s)[NA], int lane)
{
    if constexpr (M >= MMIN) {
        if constexpr (NH >= 2) {
            constexpr int HALF = NH / 2;
            const bool hi = (lane & M) != 0;
#pragma unroll
            for (int q = 0; q < HALF; ++q) {
                Acc<P> mine, give;
#pragma unroll
                for (int k = 0; k < P; ++k) {
                    mine.s[k] = hi ? s[q + HALF].s[k] : s[q].s[k];
                    give.s[k] = hi ? s[q].s[k] : s[q + HALF].s[k];
                }
                acc_add_acc(mine, shfl_xor_acc(give, M));
                s[q] = mine;
            }
            slot_scatter<P, NA, HALF, MMIN, M / 2>(s, lane);
        } else {
            acc_add_acc(s[0], shfl_xor_acc(s[0], M));
            slot_scatter<P, NA, NH, MMIN, M / 2>(s, lane);
        }
    }
}

template <int W>
constexpr int slot_levels()
{
    int n = 0;
    for (int m = 32; m >= W; m >>= 1) ++n;
    return n;
}

template <int W>
constexpr int slot_scatter_kept()
{
    int na = W;
    for (int t = 0; t < slot_levels<W>() && na >= 2; ++t) na /= 2;
    return na;
}

template <int W, int MMIN, int M>
constexpr int slot_plain_mask()
{
    int na = W, mask = 0;
    for (int m = M; m >= MMIN; m >>= 1) {
        if (na >= 2)
            na /= 2;
        else
            mask |= m;
    }
    return mask;
}

// first accumulator index kept by lane l after slot_scatter over masks 32 .. W
template <int W>
__device__ __forceinline__ int slot_scatter_index(int lane)
{
    int idx = 0, na = W;
    for (int m = 32; m >= W && na >= 2; m >>= 1) {
        na /= 2;
        if (lane & m) idx += na;
    }
    return idx;
}

// Thread (slot, c) of workgroup b holds column c of rows b*S + slot + k*G*S, k < R, where
// S = NT/W row slots per workgroup: the W threads of a row are consecutive lanes.  Rows are
// counted from `off` rows above the panel's diagonal.
//
// When off = W the kernel first applies the previous panel's block reflector to its own
// columns, C := C - Y' T'^T (Y'^T C) over the rows from the previous diagonal down (this is
// the look-ahead: the rest of the trailing matrix is updated concurrently, by other workgroups
// of the launch or by the k_apply_s/t/u kernels).  The workgroup's rows of Y' (sy: R W P S doubles
// of LDS) and T' are staged once, one element a thread and row: the W threads of a row then read
// them from LDS, in place of W loads each from a block that other XCDs have just written.
//
// Column j of the panel, x = A(j:h, j) with x1 = a_jj, sigma = sum_{i>j} x_i^2, q = x1^2 + sigma,
// mu = sqrt(q): the Householder vector of Golub-Van Loan 5.1.1 is v = x rho below the
// diagonal with v_j = 1, where rho = 1/v1 and v1 = x1 - mu (x1 <= 0) or -sigma/(x1 + mu)
// (x1 > 0), so rho = -1/(mu - x1) = -(mu + x1)/sigma in both cases; beta = 2/(v^T v) and
// beta rho = -1/mu, so beta = 1 - x1/mu.  For c > j, with d_c = sum_{i>j} x_i a_ic from the
// same reduction as sigma, w_c = v^T a_c = a_jc + rho d_c and the update is
// a_ic += (w_c/mu) x_i (i > j), a_jc -= beta w_c.  The per-column chain is the square root;
// the reciprocals 1/q and 1/sigma are formed beside it in other waves, and then
// 1/mu = mu (1/q), rho = -(mu + x1) (1/sigma) cost one product each.  Where these forms
// cancel (sigma < x1^2: mu + x1 for x1 < 0, 1 - x1/mu for x1 > 0) rho = -1/(mu - x1) and
// beta = -(1/mu)/rho are used instead.  Column j of T follows from
// T(0:j, j) = -beta_j T(0:j, 0:j) (Y(:, 0:j)^T v_j) (Schreiber and Van Loan's compact WY).
template <int P, int W, int NT>
struct PanelLds {
    double part[NT / 64 * W * W * P];
    double comb[NT * P];     // pair_sum partials
    double head[W * P];
    double psum[NT / 128 * W * P];  // column j's reduction by poll wave: sigma (l = j), d_l, Gram sums
    double hd[W * P];        // row j: a_jl
    double mu[P];
    double iq[P];            // 1/q
    double is[P];            // 1/sigma
    double fc[W * W * P];    // [j][c]: w_c = v_j^T a_c (deferred row-j update)
    double info[W * 2 * P];  // per column: 1/mu, x1
    double gram[W * W * P];  // [j][l]: sum_{i>j} x_j(i) x_l(i), l < j
    double hrow[W * W * P];  // [j][l]: a_jl when column j is processed, l < j
    double rho[W * P];
    double beta[W * P];
    double T[W * W * P];     // T, column-major
    double dig[2][64];       // digits of mu and 1/sigma (md_lanes.hpp)
    int flag[W];             // per column: 1 sigma == 0, 2 beta from rho (x1 > 0, sigma < x1^2)
};

template <int P, int W, int R, int NT>
__device__ __forceinline__ void panel_run(const PanelArgs &g, int bid, PanelLds<P, W, NT> &lds, double *sy)
{
    constexpr int S = NT / W;
    constexpr int NW = NT / 64;
    constexpr int NPW = NW / 2;      // waves that collect the workgroups' sums
    constexpr int SLOT = W * W * P;  // doubles per workgroup of the look-ahead exchange
    static_assert(64 % W == 0 && S >= 2 * W && NW >= 4, "panel layout");
    double *const s_part = lds.part, *const s_comb = lds.comb, *const s_head = lds.head, *const s_psum = lds.psum;
    double *const s_hd = lds.hd, *const s_mu = lds.mu, *const s_iq = lds.iq, *const s_is = lds.is;
    double *const s_fc = lds.fc, *const s_info = lds.info, *const s_gram = lds.gram, *const s_hrow = lds.hrow;
    double *const s_rho = lds.rho, *const s_beta = lds.beta, *const s_T = lds.T;
    int *const s_flag = lds.flag;

    // The panel is the critical path of the factorisation: its waves take issue priority over
    // the trailing-update waves that may share their compute unit.
    __builtin_amdgcn_s_setprio(3);
    const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
    const int c = tid % W, slot = tid / W;
    const long rstride = (long)g.G * S;
    const long rbase = (long)bid * S + slot;
    const int src0 = lane & ~(W - 1);
    const int off = g.off;
    const long hh = (long)g.h + off;

    // Off-chain pieces of the compact-WY factor (block 0; beta and T are written by it only).
    // beta_jj = 1 - x1/mu, or -(1/mu)/rho where that form cancels
    auto t_beta = [&](int jj) __attribute__((always_inline)) {
        V<P> beta = zero<P>();
        if (!(s_flag[jj] & 1)) {
            const V<P> r = lds_ld<P>(&s_info[(jj * 2 + 0) * P]);
            if (s_flag[jj] & 2)
                beta = neg(mul(r, recip(lds_ld<P>(&s_rho[jj * P]))));
            else
                beta = fma(from_double<P>(1.0), neg(lds_ld<P>(&s_info[(jj * 2 + 1) * P])), r);
        }
        if (lane == 0) {
            lds_st(&s_beta[jj * P], beta);
            stm(g.beta, g.bps, jj, beta);
        }
    };
    // lane l < jj: g(l, jj) = y_l^T v_jj = rho_l (a_jj,l + rho_jj gsum_jj,l)
    auto t_g = [&](int jj) __attribute__((always_inline)) {
        V<P> gv = zero<P>();
        if (lane < jj) {
            const V<P> rl = lds_ld<P>(&s_rho[lane * P]), rj = lds_ld<P>(&s_rho[jj * P]);
            gv = mul(rl, fma(lds_ld<P>(&s_hrow[(jj * W + lane) * P]), rj, lds_ld<P>(&s_gram[(jj * W + lane) * P])));
        }
        return gv;
    };
    // lane l < jj: w_l = sum_{l <= k < jj} T(l, k) g(k, jj).  W <= 8: a lane forms one product (l = lane / W,
    // k = lane % W) and the W lanes of an l are summed (n = 1024: qd 11.42 -> 11.14 ms, od 54.2 -> 53.6); W = 16: lane l
    // sums, even and odd k in two accumulators, so the two halves of the sum overlap
    auto t_w = [&](int jj, const V<P> &gv) __attribute__((always_inline)) {
        Acc<P> w0 = acc_zero<P>();
        if constexpr (W * W <= 64) {
            const int l = lane / W, k = lane % W;
            const V<P> gk = shfl_md(gv, k);
            if (l < W && l <= k && k < jj) {
                const V<P> t = lds_ld<P>(&s_T[(k * W + l) * P]);
                casc_fma<P, P, P, 0, 0, false>(w0.s, t.x, gk.x, nullptr);
            }
#pragma unroll
            for (int m = 1; m < W; m <<= 1) acc_add_acc(w0, shfl_xor_acc(w0, m));
            return shfl_md(acc_get(w0), (lane % W) * W);
        } else {
            Acc<P> w1 = acc_zero<P>();
#pragma unroll
            for (int k = 0; k < W; ++k) {
                if (k < jj) {
                    const V<P> gk = shfl_md(gv, k);
                    if (lane <= k) {
                        if (k & 1)
                            acc_fma(w1, lds_ld<P>(&s_T[(k * W + lane) * P]), gk);
                        else
                            acc_fma(w0, lds_ld<P>(&s_T[(k * W + lane) * P]), gk);
                    }
                }
            }
            acc_add_acc(w0, w1);
            return acc_get(w0);
        }
    };
    // T(0:jj, jj) = -beta_jj w, T(jj, jj) = beta_jj, zero below
    auto t_store = [&](int jj, const V<P> &w) __attribute__((always_inline)) {
        const V<P> bj = lds_ld<P>(&s_beta[jj * P]);
        if (lane < W) {
            V<P> t = zero<P>();
            if (lane < jj && !(s_flag[jj] & 1)) t = neg(mul(bj, w));
            if (lane == jj) t = bj;
            lds_st(&s_T[(jj * W + lane) * P], t);
            stm(g.T, g.tps, (long)jj * W + lane, t);
        }
    };

    V<P> a[R];
#pragma unroll
    for (int k = 0; k < R; ++k) {
        const long r = rbase + k * rstride;
        a[k] = (r < hh && c < g.wact) ? ldm<P>(g.A, g.ps, c * g.lda + r) : zero<P>();
    }
    auto ysl = [&](int k, int i) __attribute__((always_inline)) {
        V<P> y;
#pragma unroll
        for (int e = 0; e < P; ++e) y.x[e] = sy[((k * W + i) * P + e) * S + slot];
        return y;
    };
    if (off) {
        const int row = tid % S, i = tid / S;
        V<P> yv[R], tv = zero<P>();
#pragma unroll
        for (int k = 0; k < R; ++k)
            yv[k] = y_entry<P>(g.Yp, g.lda, g.ps, (long)bid * S + row + k * rstride, i, (int)hh, W);
        if (tid < W * W) tv = ldm<P>(g.Tp, g.tps, tid);
#pragma unroll
        for (int k = 0; k < R; ++k)
#pragma unroll
            for (int e = 0; e < P; ++e) sy[((k * W + i) * P + e) * S + row] = yv[k].x[e];
        if (tid < W * W) lds_st(&s_T[tid * P], tv);  // T', until the first column of T is formed
        __syncthreads();
    }

    // ---- 0. apply the previous panel's reflectors to this panel (look-ahead update):
    //         S = Y'^T C (W x W), -U = -T'^T S, C += Y' (-U)
    if (off) {
        Acc<P> sacc[W];
#pragma unroll
        for (int i = 0; i < W; ++i) sacc[i] = acc_zero<P>();
#pragma unroll
        for (int k = 0; k < R; ++k) {
            const long r = rbase + k * rstride;
            if (r < hh) {
#pragma unroll
                for (int i = 0; i < W; ++i)
                    acc_fma_step(sacc[i], ysl(k, i), a[k], k);
            }
        }
        // sum over the wave's row slots; lane (.., c) ends with NF accumulators of column c
        constexpr int NF = slot_scatter_kept<W>();
        slot_scatter<P, W, W, W, 32>(sacc, lane);
        if ((lane & slot_plain_mask<W, W, 32>()) == 0) {
            const int i0 = slot_scatter_index<W>(lane);
#pragma unroll
            for (int f = 0; f < NF; ++f)
#pragma unroll
                for (int k = 0; k < P; ++k) s_part[((wid * W + i0 + f) * W + c) * P + k] = sacc[f].s[k];
        }
        __syncthreads();
        // pairs q = (i, cc) = (q / W, q % W); thread t takes pair t % W^2 and every K-th part
        // of its sums (K = NT / W^2 threads per pair), pair_sum combines them
        constexpr int WW = W * W;
        constexpr int K = NT / WW;
        const int pq = tid % WW, psub = tid / WW;
        {
            Acc<P> t = acc_zero<P>();
            for (int w = psub; w < NW; w += K) {
                Acc<P> o;
#pragma unroll
                for (int k = 0; k < P; ++k) o.s[k] = s_part[(w * WW + pq) * P + k];
                acc_add_acc(t, o);
            }
            pair_sum<P, WW, NT, false>(t, s_comb, s_gram);  // this workgroup's S
        }
        if (g.G > 1) {
            if (wid == 0) {
                double *mine = g.gpart + (size_t)bid * SLOT;
                for (int q = lane; q < WW; q += 64) {
#pragma unroll
                    for (int k = 0; k < P; ++k) st_coherent(mine + q * P + k, s_gram[q * P + k]);
                }
                grid_sync(g.gbar, (unsigned)g.G, g.err, g.spin);
            }
            __syncthreads();
            const double *base = g.gpart;
            // the workgroups' slots are loaded in batches of NB before they are added (same
            // order), so a batch costs one round trip
            constexpr int NB = (P >= 8) ? 1 : 8;
            Acc<P> t = acc_zero<P>();
            for (int b0 = psub; b0 < g.G; b0 += NB * K) {
                Acc<P> o[NB];
#pragma unroll
                for (int u = 0; u < NB; ++u) {
                    const int b = b0 + u * K;
#pragma unroll
                    for (int k = 0; k < P; ++k)
                        o[u].s[k] = (b < g.G) ? ld_coherent(base + (size_t)b * SLOT + pq * P + k) : 0.0;
                }
#pragma unroll
                for (int u = 0; u < NB; ++u)
                    if (b0 + u * K < g.G) acc_add_acc(t, o[u]);
            }
            pair_sum<P, WW, NT, false>(t, s_comb, s_gram);
        }
        // -U(i, cc) = -sum_{l<=i} T'(l, i) S(l, cc) into s_hrow (scratch); the K threads of a
        // pair split the sum over l
        {
            const int i = pq / W, cc = pq % W;
            Acc<P> u = acc_zero<P>();
            for (int l = psub; l <= i; l += K)
                acc_fma(u, lds_ld<P>(&s_T[(i * W + l) * P]), lds_ld<P>(&s_gram[(l * W + cc) * P]));
            pair_sum<P, WW, NT, true>(u, s_comb, s_hrow);
        }
        // even and odd i in two accumulators, so the two halves of the sum overlap
#pragma unroll
        for (int k = 0; k < R; ++k) {
            const long r = rbase + k * rstride;
            if (r < hh && c < g.wact) {
                Acc<P> t0 = acc_from(a[k]), t1 = acc_zero<P>();
#pragma unroll
                for (int i = 0; i < W; i += 2) {
                    acc_fma(t0, ysl(k, i), lds_ld<P>(&s_hrow[(i * W + c) * P]));
                    acc_fma(t1, ysl(k, i + 1), lds_ld<P>(&s_hrow[((i + 1) * W + c) * P]));
                }
                acc_add_acc(t0, t1);
                a[k] = acc_get(t0);
            }
        }
        __syncthreads();
    }

    // Per column j the serial chain (reduction, mu, 1/mu, w_c) runs between workgroup barriers, the
    // off-chain work in other waves beside it:
    //   [B1, B2]  wave 0: sum of the partial sums, published; waves 0 .. NPW - 1: the workgroups' sums,
    //             each wave its share of them (one or two items a lane in flight, so that a poll is short);
    //             in block 0 wave NW - 2: beta of column j-1, wave NW - 1: g(l, j-1) and for P <= 4 also
    //             w = T(:, :j-1) g(:, j-1), which is longer than mu there
    //   after B2  every wave adds the NPW sums of its own column
    //   [B2, M]   wave 0: mu = sqrt(q); wave 1: 1/q; wave 2: 1/sigma; last wave (P = 8): w
    //   [M, Tb]   wave 0: 1/mu = mu (1/q); wave 1: rho_j and w_c = a_jc + rho_j d_c;
    //             last wave: T(:, j-1) = -beta w
    //   then      every thread: coef_c = w_c / mu and the update of its rows below row j.
    // Row j of the columns c > j (a_jc -= beta w_c) is not needed again inside the panel, so
    // that update waits for the end of the panel.
    // NPW waves collecting in place of wave 0 alone: dd n = 1024 4.92 -> 4.62 ms, qd 12.0 -> 11.5, od 55.7 ->
    // 54.1.  (dd with the scalars formed in every wave, without M and Tb: 5.04; two waves share a SIMD.)
    // the last wave carries g, then w, across barriers
    V<P> cx = zero<P>();
    // where w is formed: beside the reduction while the md scalars are cheap (P <= 4); beside mu
    // for od, whose reduction window is the shorter one in late panels
    constexpr bool kEarlyW = P <= 4;
    const int tot_items = g.G * W;
    const int npw = (g.G > 1) ? min(NPW, (tot_items + 63) / 64) : 1;  // waves that hold sums
    for (int j = 0; j < g.wact; ++j) {
        const long dj = off + j;  // row of the diagonal element of column j
        // ---- 1. one reduction per column: thread (slot, c) sums x_j(i) a_c(i) over its rows i > j:
        //         sigma (c = j), d_c (c > j), the Gram sums for T (c < j)
        Acc<P> acc = acc_zero<P>();
#pragma unroll
        for (int k = 0; k < R; ++k) {
            const long r = rbase + k * rstride;
            const V<P> xk = shfl_md(a[k], src0 + j);
            if (r > dj && r < hh) acc_fma_step(acc, xk, a[k], k);
        }
        // the partial sums stay lazy (level sums) through every reduction level below and are
        // renormalised once, after the last
#pragma unroll
        for (int m = W; m < 64; m <<= 1) acc_add_acc(acc, shfl_xor_acc(acc, m));
        if (lane < W) {
#pragma unroll
            for (int k = 0; k < P; ++k) s_part[(wid * W + lane) * P + k] = acc.s[k];
        }
        if (bid == 0 && slot == dj) lds_st(&s_head[c * P], a[0]);
        __syncthreads();  // B1
        const unsigned tag = g.tag0 + (unsigned)j + 1u;
        const long GW = tot_items;
        unsigned long long *xbase = g.gtag + (long)(j & 1) * 2 * P * (GW + W);
        if (wid == 0) {
            Acc<P> ta = acc_zero<P>();
            for (int i = lane; i < NW * W; i += 64) {
                Acc<P> o;
#pragma unroll
                for (int k = 0; k < P; ++k) o.s[k] = s_part[i * P + k];
                acc_add_acc(ta, o);
            }
#pragma unroll
            for (int m = W; m < (NW * W < 64 ? NW * W : 64); m <<= 1) acc_add_acc(ta, shfl_xor_acc(ta, m));
            if (lane < W) {
                if (g.G > 1) {
#pragma unroll
                    for (int k = 0; k < P; ++k) st_tagged(xbase + 2 * k * GW + (long)bid * W + lane, GW, ta.s[k], tag);
                } else {
#pragma unroll
                    for (int k = 0; k < P; ++k) s_psum[lane * P + k] = ta.s[k];
                    lds_st(&s_hd[lane * P], lds_ld<P>(&s_head[lane * P]));
                }
            }
        }
        if (bid == 0 && wid == 1 && g.G > 1 && lane < W) {
            const V<P> h = lds_ld<P>(&s_head[lane * P]);
#pragma unroll
            for (int k = 0; k < P; ++k) st_tagged(xbase + 2 * P * GW + 2 * k * W + lane, W, h.x[k], tag);
        }
        if (wid < npw && g.G > 1) {
            // NB items (workgroup, column) a lane in flight at once, and beside the first of them the head
            // row in wave 1 (or the only wave); the summation order is by item
            constexpr int NB = 2;
            Acc<P> ta = acc_zero<P>();
            const bool head = wid == (npw > 1 ? 1 : 0);
            for (int i0 = wid * 64, first = 1; i0 < tot_items; i0 += NB * 64 * npw, first = 0) {
                unsigned long long wd[NB + 1][2 * P];
                long offs[NB + 1], strd[NB + 1];
                bool act[NB + 1];
#pragma unroll
                for (int u = 0; u < NB; ++u) {
                    offs[u] = i0 + lane + u * 64 * npw;
                    strd[u] = GW;
                    act[u] = offs[u] < tot_items;
                }
                offs[NB] = 2 * P * GW + lane % W;
                strd[NB] = W;
                act[NB] = first != 0 && head;
                poll_tagged<P, NB + 1>(xbase, offs, strd, act, tag, wd, g.err, g.spin);
                if (act[NB] && lane < W) {
#pragma unroll
                    for (int k = 0; k < P; ++k) s_hd[lane * P + k] = tagged_value(wd[NB][2 * k], wd[NB][2 * k + 1]);
                }
#pragma unroll
                for (int u = 0; u < NB; ++u) {
                    if (act[u]) {
                        Acc<P> o;
#pragma unroll
                        for (int k = 0; k < P; ++k) o.s[k] = tagged_value(wd[u][2 * k], wd[u][2 * k + 1]);
                        acc_add_acc(ta, o);
                    }
                }
            }
#pragma unroll
            for (int m = W; m < 64; m <<= 1) acc_add_acc(ta, shfl_xor_acc(ta, m));
            if (lane < W) {
#pragma unroll
                for (int k = 0; k < P; ++k) s_psum[(wid * W + lane) * P + k] = ta.s[k];
            }
        } else if (bid == 0 && j > 0) {
            if (wid == NW - 2) t_beta(j - 1);
            if (wid == NW - 1) {
                cx = t_g(j - 1);
                if constexpr (kEarlyW) cx = t_w(j - 1, cx);  // in the shadow of the reduction
            }
        }
        __syncthreads();  // B2
        // ---- 2. the total of column c, and the Householder scalars, identical in every lane and workgroup
        V<P> tot;
        {
            Acc<P> t;
#pragma unroll
            for (int k = 0; k < P; ++k) t.s[k] = s_psum[c * P + k];
            for (int q = 1; q < npw; ++q) {
                Acc<P> o;
#pragma unroll
                for (int k = 0; k < P; ++k) o.s[k] = s_psum[(q * W + c) * P + k];
                acc_add_acc(t, o);
            }
            tot = acc_get(t);
        }
        const V<P> hd = lds_ld<P>(&s_hd[c * P]);
        if (wid == NW - 1 && lane < j) {
            lds_st(&s_gram[(j * W + lane) * P], tot);
            lds_st(&s_hrow[(j * W + lane) * P], hd);
        }
        const V<P> sig = shfl_md(tot, src0 + j);
        const V<P> x1 = shfl_md(hd, src0 + j);
        const bool zs = is_zero(sig);
        const bool pos = x1.x[0] > 0.0;
        const bool small = sig.x[0] < x1.x[0] * x1.x[0];  // sigma < x1^2: the cancelling forms are avoided
        V<P> mu = zero<P>(), coef = zero<P>();  // coef = w_c / mu
        // od spreads mu, 1/mu, 1/sigma and rho over the lanes (md_lanes.hpp) while the exponents leave room;
        // NaN, infinities and the rest take the one-lane forms
        const double q0 = __builtin_fma(x1.x[0], x1.x[0], sig.x[0]);
        const bool spread = P >= 8 && q0 < 0x1p900 && sig.x[0] > 0x1p-900;
        const int pe = spread ? ilogb(q0) >> 1 : 0, se = spread ? ilogb(sig.x[0]) : 0;
        if (wid == 0) {
            if (!zs && spread) {
                if constexpr (P >= 8) {
                    constexpr int L = lanes::kDigits;
                    const double X1 = lanes::digits<P>(x1.x, pe, lane);
                    const double Q = lanes::carry(
                        lanes::mul<L>(X1, X1, lane) + lanes::digits<P>(sig.x, 2 * pe, lane), lane);
                    const double Y = lanes::rsqrt(Q, __builtin_ldexp(q0, -2 * pe), lane);
                    const double S = lanes::mul<L>(Q, Y, lane);
                    lds.dig[0][lane] = S;
                    const V<P> m = lanes::limbs<P>(S, pe), im = lanes::limbs<P>(Y, -pe);
                    if (lane == 0) {
                        lds_st(s_mu, m);
                        lds_st(s_iq, im);  // 1/mu here
                    }
                }
            } else if (!zs) {
                const V<P> m = sqrt_md(fma(sig, x1, x1));
                if (lane == 0) lds_st(s_mu, m);
            }
            if (lane == 0) s_flag[j] = zs ? 1 : ((pos && small) ? 2 : 0);
        } else if (wid == 1) {
            if (!zs && !spread) {
                const V<P> iq = recip(fma(sig, x1, x1));
                if (lane == 0) lds_st(s_iq, iq);
            }
        } else if (wid == 2) {
            if (!zs && (pos || !small)) {
                if (spread) {
                    if constexpr (P >= 8)
                        lds.dig[1][lane] = lanes::recip(lanes::digits<P>(sig.x, se, lane),
                                                           __builtin_ldexp(sig.x[0], -se), lane);
                } else {
                    const V<P> is = recip(sig);
                    if (lane == 0) lds_st(s_is, is);
                }
            }
        } else if (wid == NW - 1 && bid == 0 && j > 0) {
            if constexpr (!kEarlyW) cx = t_w(j - 1, cx);
        }
        __syncthreads();  // M
        if (wid == 0) {
            if (!zs && lane == 0) {
                const V<P> iq = lds_ld<P>(s_iq);
                lds_st(&s_info[(j * 2 + 0) * P], spread ? iq : mul(lds_ld<P>(s_mu), iq));  // 1/mu
                lds_st(&s_info[(j * 2 + 1) * P], x1);
            }
        } else if (wid == 1) {
            // rho = 1/v1, then w_c = a_jc + rho d_c for the columns right of j
            V<P> rho = from_double<P>(1.0);
            if (!zs) {
                if (spread) {
                    if constexpr (P >= 8) {
                        const double S = lds.dig[0][lane], X1 = lanes::digits<P>(x1.x, pe, lane);
                        if (!pos && small) {
                            const double D = lanes::carry(S - X1, lane);  // mu - x1, in [1, 4)
                            const double d0 = __builtin_ldexp(s_mu[0] - x1.x[0], -pe);
                            rho = lanes::limbs<P>(-lanes::recip(D, d0, lane), -pe);
                        } else {
                            const double F = lanes::carry(S + X1, lane);
                            rho = lanes::limbs<P>(-lanes::mul<lanes::kDigits>(F, lds.dig[1][lane], lane), pe - se);
                        }
                    }
                } else {
                    const V<P> m = lds_ld<P>(s_mu);
                    rho = (!pos && small) ? neg(recip(sub(m, x1))) : neg(mul(add(m, x1), lds_ld<P>(s_is)));
                }
                if (lane > j && lane < W) lds_st(&s_fc[(j * W + lane) * P], fma(hd, tot, rho));
            }
            if (lane == 0) lds_st(&s_rho[j * P], rho);
        } else if (wid == NW - 1 && bid == 0 && j > 0) {
            t_store(j - 1, cx);
        }
        __syncthreads();  // Tb
        if (!zs) {
            mu = lds_ld<P>(s_mu);
            if (c > j) coef = mul(lds_ld<P>(&s_fc[(j * W + c) * P]), lds_ld<P>(&s_info[(j * 2 + 0) * P]));
        }
        // ---- 3. reflector j applied to the columns c > j below row j; mu on the diagonal
        if (!zs) {
#pragma unroll
            for (int k = 0; k < R; ++k) {
                const long r = rbase + k * rstride;
                const V<P> xk = shfl_md(a[k], src0 + j);  // column j is unchanged below row j
                if (r == dj) {
                    if (c == j) a[k] = mu;
                } else if (r > dj && r < hh && c > j) {
                    a[k] = fma(a[k], coef, xk);
                }
            }
        }
    }
    __syncthreads();
    // ---- 4. the last column's beta and T column; the deferred row updates; v = x rho below
    //         the diagonal; store the panel (rows from the previous diagonal)
    if (bid == 0 && g.wact > 0) {
        if (wid == NW - 2) t_beta(g.wact - 1);
        if (wid == NW - 1) cx = t_w(g.wact - 1, t_g(g.wact - 1));
    }
    const V<P> rc = lds_ld<P>(&s_rho[c * P]);
#pragma unroll
    for (int k = 0; k < R; ++k) {
        const long r = rbase + k * rstride;
        if (r < hh && c < g.wact) {
            const long jr = r - off;  // panel row
            if (jr >= 0 && jr < c) {
                if (!(s_flag[jr] & 1))
                    a[k] = fma(a[k], neg(lds_ld<P>(&s_beta[jr * P])), lds_ld<P>(&s_fc[(jr * W + c) * P]));
            } else if (jr > c && !(s_flag[c] & 1)) {
                a[k] = mul(a[k], rc);
            }
            stm(g.A, g.ps, c * g.lda + r, a[k]);
        }
    }
    __syncthreads();
    if (bid == 0 && wid == NW - 1) {
        if (g.wact > 0) t_store(g.wact - 1, cx);
        for (int jj = g.wact; jj < W; ++jj)
            if (lane < W) stm(g.T, g.tps, (long)jj * W + lane, zero<P>());
    }
}

// One panel launch: workgroup b runs panel_run(g, b).
template <int P, int W, int R, int NT>
__global__ __launch_bounds__(NT) void k_panel(PanelArgs g)
{
    __shared__ PanelLds<P, W, NT> lds;
    __shared__ double sy[R * P * NT];  // R W P S doubles
    panel_run<P, W, R, NT>(g, blockIdx.x, lds, sy);
}

// ============================================================================ trailing update
// C := C - Y T^T (Y^T C) for the columns right of the panel (those of C, then those of B, as
// one index space).  The work is cut into units of four columns (one per wave) by rb rows, so
// that every launch has many equal units whatever its shape:
//   k_apply_s -- each unit's partial sums Y^T c over its rows (lazy level sums, not rounded);
//   k_apply_t -- per column, the partial sums combined in a fixed order into S = Y^T c, and
//                -U = -T^T S;
//   k_apply_u -- each unit's rows: c -= Y U.
// All three walk their units grid-stride, so a capped grid leaves CUs free for a concurrent
// panel.  Y is staged through LDS per unit; lanes walk rows (unit-stride limb planes).
// most rows per unit: 256, or 128 where W P 256 doubles of staged Y would exceed 64 KiB of LDS
template <int P, int W>
constexpr int rb_max()
{
    return W * P * 256 * 8 <= 65536 ? 256 : 128;
}

struct ApplyArgs {
    const double *Y;  // panel top-left (diagonal) element; Y is unit lower trapezoidal
    long ldy, psy;
    int h, wact;
    const double *T;  // W x W (ld W)
    long tps;
    double *C;  // first trailing column, panel's first row
    long ldc, psc;
    int nc;
    double *B;  // extra columns (right-hand sides), panel's first row
    long ldb, psb;
    int nb;
    int c0, ncol;  // this launch covers columns c0 .. c0 + ncol - 1 of the (C, B) index space
    int rb, nrb;   // rows per unit (a multiple of 64, at most rb_max) and row blocks
    double *part;  // [ncol][nrb][W][P] partial sums
    double *nu;    // [ncol][W][P] -U
    int rs;        // update_run: waves per column, 1 or 2
};

// Column gc of this launch (null past the end); its plane stride in *cps.
__device__ __forceinline__ double *apply_col(const ApplyArgs &g, int gc, long *cps)
{
    if (gc >= g.ncol) return nullptr;
    const int q = g.c0 + gc;
    if (q < g.nc) {
        *cps = g.psc;
        return g.C + (long)q * g.ldc;
    }
    *cps = g.psb;
    return g.B + (long)(q - g.nc) * g.ldb;
}

template <int P, int W>
__device__ __forceinline__ void stage_y(const ApplyArgs &g, double *sY, long r0, int tid)
{
    for (int e = tid; e < W * g.rb; e += kThreads) {
        const int r = e % g.rb, i = e / g.rb;
        const V<P> y = y_entry<P>(g.Y, g.ldy, g.psy, r0 + r, i, g.h, g.wact);
#pragma unroll
        for (int k = 0; k < P; ++k) sY[(i * P + k) * rb_max<P, W>() + r] = y.x[k];
    }
}

// Sum W lazy accumulators over the 64 lanes of a wave; afterwards s[0] of lane l holds the
// total of accumulator l / (64 / W).  Each level first halves the set a lane keeps (the
// partner keeps the other half), so W accumulators cost W - 1 + 6 - log2(W) additions
// instead of 6 W.
template <int P, int W, int HALF, int M>
__device__ __forceinline__ void reduce_scatter_level(Acc<P> (&s)[W], int lane)
{
    if constexpr (HALF >= 1) {
        const bool hi = (lane & M) != 0;
#pragma unroll
        for (int q = 0; q < HALF; ++q) {
            Acc<P> mine, give;
#pragma unroll
            for (int k = 0; k < P; ++k) {
                mine.s[k] = hi ? s[q + HALF].s[k] : s[q].s[k];
                give.s[k] = hi ? s[q].s[k] : s[q + HALF].s[k];
            }
            acc_add_acc(mine, shfl_xor_acc(give, M));
            s[q] = mine;
        }
        reduce_scatter_level<P, W, HALF / 2, M / 2>(s, lane);
    } else {
#pragma unroll
        for (int m = M; m >= 1; m >>= 1) acc_add_acc(s[0], shfl_xor_acc(s[0], m));
    }
}

template <int P, int W>
__device__ __forceinline__ void reduce_scatter(Acc<P> (&s)[W], int lane)
{
    static_assert(W >= 1 && W <= 32 && (W & (W - 1)) == 0, "reduce_scatter: W a power of two");
    reduce_scatter_level<P, W, W / 2, 32>(s, lane);
}

// Accumulators a lane keeps at once in k_apply_s: all W, or for octo double at most 4 (the
// partial sums of the other columns of Y take further passes over the unit's rows), so that
// the kernel keeps two waves per SIMD.
template <int P, int W>
constexpr int apply_pass_width()
{
    return (P >= 8 && W > 4) ? 4 : W;
}

template <int P, int W>
__global__ __launch_bounds__(kThreads, 2) void k_apply_s(ApplyArgs g)
{
    constexpr int WH = apply_pass_width<P, W>();
    __shared__ double sY[W * P * rb_max<P, W>()];
    const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
    const int ncg = (g.ncol + 3) / 4;
    const int units = ncg * g.nrb;
    for (int u = blockIdx.x; u < units; u += gridDim.x) {
        const int cg = u % ncg, rbk = u / ncg;
        const long r0 = (long)rbk * g.rb;
        __syncthreads();
        stage_y<P, W>(g, sY, r0, tid);
        __syncthreads();
        const int gc = cg * 4 + wid;
        long cps = 0;
        const double *col = apply_col(g, gc, &cps);
        if (!col) continue;  // whole wave
#pragma unroll 1
        for (int i0 = 0; i0 < W; i0 += WH) {
            Acc<P> s[WH];
#pragma unroll
            for (int i = 0; i < WH; ++i) s[i] = acc_zero<P>();
            int nterm = 0;
            for (int r = lane; r < g.rb; r += 64) {
                const long gr = r0 + r;
                if (gr < g.h) {
                    const V<P> cv = ldm<P>(col, cps, gr);
#pragma unroll
                    for (int i = 0; i < WH; ++i) {
                        V<P> y;
#pragma unroll
                        for (int k = 0; k < P; ++k) y.x[k] = sY[((i0 + i) * P + k) * rb_max<P, W>() + r];
                        acc_fma_step(s[i], y, cv, nterm);
                    }
                    ++nterm;
                }
            }
            reduce_scatter<P, WH>(s, lane);
            constexpr int LPI = 64 / WH;
            if (lane % LPI == 0) {
                double *dst = g.part + (((long)gc * g.nrb + rbk) * W + i0 + lane / LPI) * P;
#pragma unroll
                for (int k = 0; k < P; ++k) dst[k] = s[0].s[k];
            }
        }
    }
}

template <int P, int W>
__global__ __launch_bounds__(kThreads) void k_apply_t(ApplyArgs g)
{
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    for (int gc = blockIdx.x * 4 + wid; gc < g.ncol; gc += gridDim.x * 4) {
        // lane q adds the partial sums (b, i) = (q / W + 64 k / W, q % W), then the lanes of
        // one i are combined
        Acc<P> t = acc_zero<P>();
        const double *src = g.part + (long)gc * g.nrb * W * P;
        for (int q = lane; q < g.nrb * W; q += 64) {
            Acc<P> o;
#pragma unroll
            for (int k = 0; k < P; ++k) o.s[k] = src[(long)q * P + k];
            acc_add_acc(t, o);
        }
#pragma unroll
        for (int m = W; m < 64; m <<= 1) acc_add_acc(t, shfl_xor_acc(t, m));
        const V<P> S = acc_get(t);  // lane l: S_(l mod W)
        // U_i = sum_{l <= i} T(l, i) S_l: lane p = i W + l (+ 64 k) forms one product, then
        // the W lanes of an i are summed
        constexpr int NQ = (W * W + 63) / 64;
        Acc<P> u[NQ];
#pragma unroll
        for (int k = 0; k < NQ; ++k) u[k] = acc_zero<P>();
        const int l = lane % W;
        const V<P> sl = shfl_md(S, l);
#pragma unroll
        for (int k = 0; k < NQ; ++k) {
            const int i = (lane + 64 * k) / W;
            if (l <= i && i < g.wact) acc_fma(u[k], ldm<P>(g.T, g.tps, (long)i * W + l), sl);
#pragma unroll
            for (int m = 1; m < W; m <<= 1) acc_add_acc(u[k], shfl_xor_acc(u[k], m));
            if (l == 0 && i < W) {
                const V<P> nv = neg(acc_get(u[k]));
#pragma unroll
                for (int q = 0; q < P; ++q) g.nu[((long)gc * W + i) * P + q] = nv.x[q];
            }
        }
    }
}

template <int P, int W>
__global__ __launch_bounds__(kThreads) void k_apply_u(ApplyArgs g)
{
    __shared__ double sY[W * P * rb_max<P, W>()];
    __shared__ double sU[4][W * P];  // -U of each wave's column
    const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
    const int ncg = (g.ncol + 3) / 4;
    const int units = ncg * g.nrb;
    for (int u = blockIdx.x; u < units; u += gridDim.x) {
        const int cg = u % ncg, rbk = u / ncg;
        const long r0 = (long)rbk * g.rb;
        __syncthreads();
        stage_y<P, W>(g, sY, r0, tid);
        const int gc = cg * 4 + wid;
        if (gc < g.ncol && lane < W * P) sU[wid][lane] = g.nu[(long)gc * W * P + lane];
        __syncthreads();
        long cps = 0;
        double *col = apply_col(g, gc, &cps);
        if (!col) continue;  // whole wave
        for (int r = lane; r < g.rb; r += 64) {
            const long gr = r0 + r;
            if (gr < g.h) {
                Acc<P> t = acc_from(ldm<P>(col, cps, gr));
#pragma unroll
                for (int i = 0; i < W; ++i) {
                    V<P> y;
#pragma unroll
                    for (int k = 0; k < P; ++k) y.x[k] = sY[(i * P + k) * rb_max<P, W>() + r];
                    acc_fma(t, y, lds_ld<P>(&sU[wid][i * P]));
                }
                stm(col, cps, gr, acc_get(t));
            }
        }
    }
}

// ============================================================================ factorisation step
// One launch per panel l: workgroups 0 .. G - 1 factor panel l (panel_run, which first applies panel
// l - 1 to its own columns) and the others apply panel l - 1 to the columns right of panel l and to B,
// C := C - Y T^T (Y^T C), whole columns at a time: a wave (or two, half the rows each) forms Y^T c over all
// rows, U = T^T (Y^T c) lane parallel, then c -= Y U, with Y passing through LDS in chunks of kStepRows rows
// for the workgroup's columns (the next chunk's loads in flight).  The panel is a latency chain on few
// workgroups, so the update costs nothing while its columns find compute units of their own.  Against
// a side stream for the update (three kernels, and events in front of every panel) this saves the event
// wait, about 11 us a panel, the launches (host time of a dd n = 1024 solve 3.3 -> 0.25 ms) and the update's
// partial sums: dd n = 1024 5.85 -> 4.86 ms, qd 13.0 -> 12.1, dd 128 x 128 0.67 -> 0.54, refined od
// n = 2048 23.1 -> 17.4.  The panel's workgroups come first in the grid and no other workgroup waits for
// anything, so all of them become resident.  The update is bound by the FP64 issue rate: qd, 1008
// columns of 1024 rows, 94 us alone, 81 % of the issue slots of its waves' life time.
constexpr int kStepRows = 128;  // rows of Y staged at once, twice

struct StepArgs {
    PanelArgs p;   // p.G workgroups, 0 for the launch after the last panel
    ApplyArgs a;   // the previous panel's update (a.ncol columns, 0 before the first)
};

// Plane k of a column block at a 32-bit byte offset: base and plane in scalar registers, so a lane's
// addresses cost one register (64-bit addresses of every limb and column, kept across the loops, spilled
// more, and their reloads waited for the loads in flight: qd 200 us a launch in place of 75).  What is left:
// k_step<qd> takes all 256 registers of two waves a SIMD and spills 55 of them (224 bytes a lane), dd 2.
template <int P>
__device__ __forceinline__ V<P> ldm32(const double *X, long ps, unsigned boff)
{
    V<P> v;
#pragma unroll
    for (int k = 0; k < P; ++k) v.x[k] = *(const double *)((const char *)(X + k * ps) + boff);
    return v;
}

template <int P, int W, int NT>
struct UpdateLds {
    double y[2][W * P * kStepRows];  // chunks of Y: limb k of column i at (i P + k) kStepRows + row
    double s[NT / 64][W * P];        // a wave's S, for the wave that shares its column
    double u[NT / 64][W * P];        // a wave's -U
};

template <int P, int W, int NT>
__device__ __forceinline__ void update_run(const ApplyArgs &g, int u, int nu, UpdateLds<P, W, NT> &lds)
{
    constexpr int NW = NT / 64, RC = kStepRows, RL = RC / 64, EPT = W * RC / NT;
    constexpr int LPI = 64 / W, NQ = (W * W + 63) / 64;
    // columns of Y loaded from LDS ahead of their multiply-adds: as many instructions as an LDS read
    // takes to come back (dd 48, qd 224); the barrier keeps the scheduler from pulling more of them
    // forward, which spills
    constexpr int GC = P <= 2 ? 4 : 2, NG = W / GC;
    static_assert(W * RC % NT == 0 && NT % RC == 0 && RL == 2 && NG >= 2, "update_run layout");
    const int tid = threadIdx.x, lane = tid & 63, wid = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int half = (g.rs == 2) ? (wid & 1) : -1;  // the rows this wave takes of a chunk; -1: all
    const int wcol = (g.rs == 2) ? (wid >> 1) : wid, ncw = NW / g.rs;
    const int er = tid % RC, ei = tid / RC;  // this thread stages Y(er, ei + q NT / RC) of a chunk
    const int nch = (g.h + RC - 1) / RC;
    V<P> ys[EPT], cs[RL];
    // loads from clamped places in bounds; stage() puts the zeros and the unit diagonal in
    auto fetch_y = [&](int ch) __attribute__((always_inline)) {
        const unsigned r = min(ch * RC + er, g.h - 1);
#pragma unroll
        for (int q = 0; q < EPT; ++q) {
            const unsigned i = min(ei + q * (NT / RC), g.wact - 1);
            ys[q] = ldm32<P>(g.Y, g.psy, (i * (unsigned)g.ldy + r) * 8u);
        }
    };
    auto stage = [&](int ch) __attribute__((always_inline)) {
        double *sY = lds.y[ch & 1];
        const int r = ch * RC + er;
#pragma unroll
        for (int q = 0; q < EPT; ++q) {
            const int i = ei + q * (NT / RC);
            const bool in = i < g.wact && r < g.h;
            const double one = (in && r == i) ? 1.0 : 0.0;
#pragma unroll
            for (int k = 0; k < P; ++k) sY[(i * P + k) * RC + er] = (in && r > i) ? ys[q].x[k] : (k == 0 ? one : 0.0);
        }
    };
    // columns GC grp .. GC grp + GC - 1 of Y at row q 64 + lane of a chunk
    auto load_y = [&](const double *sY, int q, int grp, V<P> (&y)[GC]) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < GC; ++i)
#pragma unroll
            for (int k = 0; k < P; ++k) y[i].x[k] = sY[((grp * GC + i) * P + k) * RC + q * 64 + lane];
    };
#pragma unroll 1
    for (int cg = u; cg * ncw < g.ncol; cg += nu) {
        long cps = 0;
        double *col = apply_col(g, cg * ncw + wcol, &cps);  // null past the end: the wave only stages
        auto fetch_c = [&](int ch) __attribute__((always_inline)) {
#pragma unroll
            for (int q = 0; q < RL; ++q)
                if (col && q != 1 - half) cs[q] = ldm32<P>(col, cps, (unsigned)min(ch * RC + q * 64 + lane, g.h - 1) * 8u);
        };
        // ---- S = Y^T c
        Acc<P> s[W];
#pragma unroll
        for (int i = 0; i < W; ++i) s[i] = acc_zero<P>();
        int nt = 0;
        __syncthreads();  // the last column group's readers
        fetch_y(0);
        fetch_c(0);
        stage(0);
        __syncthreads();
#pragma unroll 1
        for (int ch = 0; ch < nch; ++ch) {
            const double *sY = lds.y[ch & 1];
            V<P> cv[RL];
#pragma unroll
            for (int q = 0; q < RL; ++q) cv[q] = cs[q];
            if (ch + 1 < nch) {
                fetch_y(ch + 1);
                fetch_c(ch + 1);
            }
#pragma unroll
            for (int q = 0; q < RL; ++q) {
                if (!col || q == 1 - half) continue;  // uniform
                V<P> y[2][GC];
                load_y(sY, q, 0, y[0]);
#pragma unroll
                for (int grp = 0; grp < NG; ++grp) {
                    if (grp + 1 < NG) load_y(sY, q, grp + 1, y[(grp + 1) & 1]);
                    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                    for (int i = 0; i < GC; ++i) acc_fma(s[grp * GC + i], y[grp & 1][i], cv[q]);
                }
                if (++nt % kLazy<P> == 0) {
#pragma unroll
                    for (int i = 0; i < W; ++i) {
                        s[i] = acc_from(acc_get(s[i]));
                        __builtin_amdgcn_sched_barrier(0);
                    }
                }
            }
            if (ch + 1 < nch) stage(ch + 1);
            __syncthreads();
        }
        reduce_scatter<P, W>(s, lane);  // lane q: S_(q / LPI)
        if (g.rs == 2) {                // the two waves' sums, in the same order in both
            if (lane % LPI == 0) {
#pragma unroll
                for (int k = 0; k < P; ++k) lds.s[wid][(lane / LPI) * P + k] = s[0].s[k];
            }
            __syncthreads();
            V<P> o;
#pragma unroll
            for (int k = 0; k < P; ++k) {
                s[0].s[k] = lds.s[wid & ~1][(lane / LPI) * P + k];
                o.x[k] = lds.s[wid | 1][(lane / LPI) * P + k];
            }
            acc_add(s[0], o);
        }
        // ---- U = T^T S: lane q = i W + l (+ 64 k) forms one product, the W lanes of an i are summed
        const V<P> S = acc_get(s[0]);
        const int l = lane % W;
        const V<P> sl = shfl_md(S, l * LPI);
#pragma unroll
        for (int k = 0; k < NQ; ++k) {
            const int i = (lane + 64 * k) / W;
            Acc<P> t = acc_zero<P>();
            if (l <= i && i < g.wact) acc_fma(t, ldm32<P>(g.T, g.tps, (unsigned)(i * W + l) * 8u), sl);
#pragma unroll
            for (int m = 1; m < W; m <<= 1) acc_add_acc(t, shfl_xor_acc(t, m));
            if (l == 0 && i < W) lds_st(&lds.u[wid][i * P], neg(acc_get(t)));
        }
        // ---- c -= Y U, the chunks from the last one back (it is still staged); even and odd columns of Y
        // in two accumulators
        V<P> nU[W];
#pragma unroll
        for (int i = 0; i < W; ++i) nU[i] = lds_ld<P>(&lds.u[wid][i * P]);
        fetch_c(nch - 1);
#pragma unroll 1
        for (int ch = nch - 1; ch >= 0; --ch) {
            const double *sY = lds.y[ch & 1];
            V<P> cv[RL];
#pragma unroll
            for (int q = 0; q < RL; ++q) cv[q] = cs[q];
            if (ch > 0) {
                fetch_y(ch - 1);
                fetch_c(ch - 1);
            }
#pragma unroll
            for (int q = 0; q < RL; ++q) {
                if (!col || q == 1 - half) continue;  // uniform
                Acc<P> t0 = acc_from(cv[q]), t1 = acc_zero<P>();
                V<P> y[2][GC];
                load_y(sY, q, 0, y[0]);
#pragma unroll
                for (int grp = 0; grp < NG; ++grp) {
                    if (grp + 1 < NG) load_y(sY, q, grp + 1, y[(grp + 1) & 1]);
                    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                    for (int i = 0; i < GC; i += 2) {
                        acc_fma(t0, y[grp & 1][i], nU[grp * GC + i]);
                        acc_fma(t1, y[grp & 1][i + 1], nU[grp * GC + i + 1]);
                    }
                }
                acc_add_acc(t0, t1);
                const int r = ch * RC + q * 64 + lane;
                const V<P> v = acc_get(t0);
                if (r < g.h) {
#pragma unroll
                    for (int k = 0; k < P; ++k) *(double *)((char *)(col + k * cps) + (unsigned)r * 8u) = v.x[k];
                }
            }
            if (ch > 0) stage(ch - 1);
            __syncthreads();
        }
    }
}

template <int P, int W, int R, int NT>
__global__ __launch_bounds__(NT, 2) void k_step(StepArgs g)
{
    // one workgroup is either kind: the two layouts share the LDS
    struct Panel {
        PanelLds<P, W, NT> lds;
        double sy[R * P * NT];
    };
    using Update = UpdateLds<P, W, NT>;
    constexpr size_t bytes = sizeof(Panel) > sizeof(Update) ? sizeof(Panel) : sizeof(Update);
    __shared__ double raw[bytes / sizeof(double)];
    if ((int)blockIdx.x < g.p.G) {
        Panel &l = *reinterpret_cast<Panel *>(raw);
        panel_run<P, W, R, NT>(g.p, blockIdx.x, l.lds, l.sy);
    } else {
        update_run<P, W, NT>(g.a, blockIdx.x - g.p.G, gridDim.x - g.p.G, *reinterpret_cast<Update *>(raw));
    }
}

// ============================================================================ batched solves
// Many independent least-squares problems (m <= kBatchRows) in one persistent launch.  Each
// workgroup takes the next slot from a counter; a slot names a problem and a member index.
// The plan lists the problems longest first and gives the longer ones a team of T workgroups
// (T consecutive slots; batch_schedule), the others one.  A team solves its problem with narrow Householder panels
// (panel_run with T workgroups and the team's own barrier counters and exchange slots), the
// update of the columns right of the panel and of b split over the team's waves (one column
// per wave), a team barrier after each step, and member 0 does the back substitution of
// R x = (Q^T b) with the reciprocals of R's diagonal formed in parallel.  Start and end
// times (wall clock ticks) are recorded per problem.
constexpr int kBatchRows = 512;
constexpr int kTeamMax = 16;      // most workgroups on one problem
constexpr int kTeamCtrs = 1;      // a team's barrier counter
// Polls before a team's first barrier gives up, at least: its members take their slots one after the
// other as workgroups come free, so the first of them waits for the end of another problem (0.13 s for
// qd 512 x 512 on one workgroup) and not, as every later wait, for a workgroup that is running beside it.
// A poll takes 0.19 us on an idle device, so this is 3 s.
constexpr unsigned kTeamPolls = 1u << 24;

struct BatchDesc {
    int m, n;
    long long a_off, b_off, x_off;  // doubles from the A, b, x base pointers
    int idx;                        // position of the problem in the caller's list
    int team;                       // workgroups on this problem
};

struct BatchArgs {
    const BatchDesc *desc;  // in processing order
    const int *slots;       // per slot: index into desc * kTeamMax + member
    const int *nslots;      // number of slots (device)
    double *A, *b, *x;
    double *scratch;    // per workgroup: beta (kBatchRows*P)
    unsigned *counter;  // zero on entry
    unsigned *tctr;     // per problem: kTeamCtrs barrier counters, zero on entry
    double *xch;        // per problem: T (W^2 P) and panel_run's exchange words (2 kTeamMax (W^2 + 2W) P doubles)
    int *err;           // set if a wait inside a team times out
    unsigned spin;      // polls before a wait inside a team gives up
    int *info;          // per problem
    long long *times;   // per problem: start, end; or null
};

// C := C - Y T^T (Y^T C) for the ncols columns at C0 (plane stride ps, ld lda) and the column
// b0 (plane stride bps, index ncols), h rows from the panel's diagonal; one column per wave,
// columns first, first + step, ... for this wave.
template <int P, int W, int NT, bool STAGED>
__device__ __forceinline__ void batch_update(const double *Y, long lda, long ps, int h, int wact, const double *T,
                                             double *C0, int ncols, double *b0, long bps, int first, int step,
                                             const double *sY)
{
    constexpr int LPI = 64 / W, NQ = (W * W + 63) / 64;
    const int lane = threadIdx.x & 63;
    // Y(r, i): from the LDS copy (limb k of column i at sY[(i P + k) kBatchRows + r]) or global
    auto yv = [&](int r, int i) __attribute__((always_inline)) {
        if constexpr (STAGED) {
            V<P> y;
#pragma unroll
            for (int k = 0; k < P; ++k) y.x[k] = sY[(i * P + k) * kBatchRows + r];
            return y;
        } else {
            return y_entry<P>(Y, lda, ps, r, i, h, wact);
        }
    };
    for (int col = first; col <= ncols; col += step) {
        double *cp = (col < ncols) ? C0 + (long)col * lda : b0;
        const long cps = (col < ncols) ? ps : bps;
        Acc<P> s[W];
#pragma unroll
        for (int i = 0; i < W; ++i) s[i] = acc_zero<P>();
        int nt = 0;
        for (int r = lane; r < h; r += 64) {
            const V<P> cv = ldm<P>(cp, cps, r);
#pragma unroll
            for (int i = 0; i < W; ++i) acc_fma_step(s[i], yv(r, i), cv, nt);
            ++nt;
        }
        reduce_scatter<P, W>(s, lane);
        const V<P> S = acc_get(s[0]);  // lane q: S_(q / LPI)
        // -U_i = -sum_{l <= i} T(l, i) S_l: lane q = i W + l (+ 64 k) forms one product
        const int l = lane % W;
        const V<P> sl = shfl_md(S, l * LPI);
        V<P> un[NQ];
#pragma unroll
        for (int k = 0; k < NQ; ++k) {
            const int i = (lane + 64 * k) / W;
            Acc<P> u = acc_zero<P>();
            if (l <= i && i < wact) acc_fma(u, ldm<P>(T, (long)W * W, (long)i * W + l), sl);
#pragma unroll
            for (int m = 1; m < W; m <<= 1) acc_add_acc(u, shfl_xor_acc(u, m));
            un[k] = neg(acc_get(u));
        }
        V<P> nU[W];
#pragma unroll
        for (int i = 0; i < W; ++i) nU[i] = shfl_md(un[(i * W) / 64], (i * W) % 64);
        for (int r = lane; r < h; r += 64) {
            Acc<P> t = acc_from(ldm<P>(cp, cps, r));
#pragma unroll
            for (int i = 0; i < W; ++i) acc_fma(t, yv(r, i), nU[i]);
            stm(cp, cps, r, acc_get(t));
        }
    }
}

// x = R^-1 y for the n x n upper triangle of A and y = b(0:n) (Algorithm 1 with one tile,
// column-oriented): x_i = y_i / R_ii, then y_t -= R_ti x_i for t < i.  Returns the 1-based
// index of the first exactly-zero diagonal element, or 0.
template <int P, int NT>
__device__ __forceinline__ int batch_backsub(const double *A, long lda, long ps, int n, const double *b, long bps,
                                             double *x, long xps, double *s_y, double *s_r, int *s_zero)
{
    const int tid = threadIdx.x;
    if (tid == 0) *s_zero = INT_MAX;
    __syncthreads();
    for (int i = tid; i < n; i += NT) {
        const V<P> d = ldm<P>(A, ps, (long)i * lda + i);
        const bool z = is_zero(d);
        if (z) atomicMin(s_zero, i);
        lds_st(&s_r[i * P], z ? zero<P>() : recip(d));
        lds_st(&s_y[i * P], ldm<P>(b, bps, i));
    }
    __syncthreads();
    const int zi = *s_zero;
    for (int i = n - 1; i >= 0; --i) {
        const V<P> xi = mul(lds_ld<P>(&s_y[i * P]), lds_ld<P>(&s_r[i * P]));
        if (tid == 0) stm(x, xps, i, xi);
        for (int t = tid; t < i; t += NT)
            lds_st(&s_y[t * P], fma(lds_ld<P>(&s_y[t * P]), neg(ldm<P>(A, ps, (long)i * lda + t)), xi));
        __syncthreads();
    }
    return zi == INT_MAX ? 0 : zi + 1;
}

template <int P, int W, int R, int NT>
__global__ __launch_bounds__(NT) void k_batch(BatchArgs g)
{
    static_assert((NT / W) * R >= kBatchRows, "k_batch: a panel must hold kBatchRows rows");
    constexpr int NW = NT / 64;
    constexpr long WWP = (long)W * W * P;
    constexpr long XCHP = WWP + 2L * kTeamMax * (W * W + 2 * W) * P;
    static_assert(tag_words<P, W>(kTeamMax) <= 2 * kTeamMax * (W * W + 2 * W) * P, "k_batch: exchange area");
    constexpr bool STAGED = W * P <= 16;  // the panel's Y staged in LDS (at most 64 KiB)
    __shared__ PanelLds<P, W, NT> lds;
    __shared__ double sY[STAGED ? W * P * kBatchRows : 1];
    __shared__ double s_y[kBatchRows * P];
    __shared__ double s_r[kBatchRows * P];
    __shared__ int s_next, s_zero;
    const int wid = threadIdx.x >> 6;
    double *beta = g.scratch + (long)blockIdx.x * kBatchRows * P;
    const int nslots = *g.nslots;
    for (;;) {
        __syncthreads();
        if (threadIdx.x == 0) s_next = (int)atomicAdd(g.counter, 1u);
        __syncthreads();
        const int slot = s_next;
        if (slot >= nslots) break;  // every workgroup leaves once the list is exhausted
        const long long t0 = wall_clock64();
        const int q = g.slots[slot] / kTeamMax, mem = g.slots[slot] % kTeamMax;
        const BatchDesc d = g.desc[q];
        const int team = d.team;
        unsigned *ctr = g.tctr + (long)d.idx * kTeamCtrs;
        unsigned nsync = 0;
        // all members meet (team > 1); the barrier's fences make every member's stores visible
        auto team_sync = [&]() __attribute__((always_inline)) {
            if (team > 1) {
                __syncthreads();
                ++nsync;
                if (wid == 0) grid_sync(ctr, nsync * (unsigned)team, g.err, nsync > 1 ? g.spin : max(g.spin, kTeamPolls));
                __syncthreads();
            }
        };
        double *A = g.A + d.a_off;
        double *bp = g.b + d.b_off;
        double *pxch = g.xch + (long)d.idx * XCHP;
        const long lda = d.m, ps = (long)d.m * d.n;
        // the exchange words of an earlier problem or batch carry the same column numbers
        unsigned long long *gtag = (unsigned long long *)(pxch + WWP);
        if (team > 1) {
            for (int e = mem * NT + threadIdx.x; e < tag_words<P, W>(team); e += team * NT)
                __hip_atomic_store(gtag + e, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            team_sync();
        }
        for (int c0 = 0; c0 < d.n; c0 += W) {
            PanelArgs pa;
            pa.A = A + (long)c0 * lda + c0;
            pa.lda = lda;
            pa.ps = ps;
            pa.h = d.m - c0;
            pa.wact = (d.n - c0 < W) ? (d.n - c0) : W;
            pa.off = 0;
            pa.Yp = nullptr;
            pa.Tp = nullptr;
            pa.beta = beta + c0;
            pa.bps = kBatchRows;
            pa.T = pxch;  // written by member 0, read by every member after the team barrier
            pa.tps = (long)W * W;
            pa.gpart = nullptr;  // no look-ahead (off = 0)
            pa.gbar = nullptr;
            pa.gtag = gtag;
            pa.tag0 = (unsigned)c0;
            pa.err = g.err;
            pa.G = team;
            pa.spin = g.spin;
            panel_run<P, W, R, NT>(pa, mem, lds, nullptr);
            team_sync();
            if constexpr (STAGED) {
                for (int e = threadIdx.x; e < W * pa.h; e += NT) {
                    const int r = e % pa.h, i = e / pa.h;
                    const V<P> y = y_entry<P>(pa.A, lda, ps, r, i, pa.h, pa.wact);
#pragma unroll
                    for (int k = 0; k < P; ++k) sY[(i * P + k) * kBatchRows + r] = y.x[k];
                }
            }
            __syncthreads();  // sY, and of a workgroup alone T's last column, which one wave stored last
            batch_update<P, W, NT, STAGED>(pa.A, lda, ps, pa.h, pa.wact, pa.T, A + (long)(c0 + pa.wact) * lda + c0,
                                           d.n - c0 - pa.wact, bp + c0, d.m, mem * NW + wid, team * NW, sY);
            __syncthreads();
            team_sync();
        }
        if (mem == 0) {
            const int inf = batch_backsub<P, NT>(A, lda, ps, d.n, bp, d.m, g.x + d.x_off, d.n, s_y, s_r, &s_zero);
            if (threadIdx.x == 0) {
                const bool late = team > 1 && __hip_atomic_load(g.err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0;
                g.info[d.idx] = late ? -1 : inf;
                if (g.times) {
                    g.times[2L * d.idx] = t0;
                    g.times[2L * d.idx + 1] = wall_clock64();
                }
            }
        }
    }
}

// ============================================================================ iterative refinement
// Mixed-precision kernels of the refined solve: the residual r = b - A x of a PA-limb matrix
// and a PX-limb vector, formed in PX limbs, and x += d with running maxima of |d| and |x|.
constexpr int kResidCols = 128;  // columns per residual chunk

// part[ch][k][i] = level sums of sum_{j in chunk ch} A_ij x_j (not renormalised), one row per
// thread, chunk ch = blockIdx.y of kResidCols columns
template <int PA, int PX>
__global__ __launch_bounds__(kThreads) void k_resid_part(const double *A, long lda, long psa, int m, int n,
                                                         const double *x, long xps, double *part, const int *skip)
{
    __shared__ double sx[kResidCols * PX];
    if (*skip) return;
    const int c0 = blockIdx.y * kResidCols;
    const int c1 = (n - c0 < kResidCols) ? n : c0 + kResidCols;
    for (int j = threadIdx.x; j < c1 - c0; j += kThreads) lds_st(&sx[j * PX], ldm<PX>(x, xps, c0 + j));
    __syncthreads();
    const long i = (long)blockIdx.x * kThreads + threadIdx.x;
    if (i >= m) return;
    Acc<PX> acc = acc_zero<PX>();
    for (int j = c0; j < c1; ++j) {
        const V<PA> a = ldm<PA>(A, psa, (long)j * lda + i);
        const V<PX> xv = lds_ld<PX>(&sx[(j - c0) * PX]);
        casc_fma<PX, PA, PX, 0, 0, true>(acc.s, a.x, xv.x, nullptr);
        if (((j - c0 + 1) % kLazy<PX>) == 0) acc = acc_from(acc_get(acc));
    }
#pragma unroll
    for (int k = 0; k < PX; ++k) part[((long)blockIdx.y * PX + k) * m + i] = acc.s[k];
}

// r_i = b_i - c_i - sum_ch part[ch][.][i] (chunks in order; c, PX limbs, may be null)
template <int PX>
__global__ __launch_bounds__(kThreads) void k_resid_fin(const double *b, long bps, const double *c, long cps,
                                                        const double *part, int m, int nch, double *r, long rps,
                                                        const int *skip)
{
    if (*skip) return;
    const long i = (long)blockIdx.x * kThreads + threadIdx.x;
    if (i >= m) return;
    Acc<PX> t = acc_from(ldm<PX>(b, bps, i));
    if (c) acc_add(t, neg(ldm<PX>(c, cps, i)));
    for (int ch = 0; ch < nch; ++ch) {
        V<PX> o;
#pragma unroll
        for (int k = 0; k < PX; ++k) o.x[k] = -part[((long)ch * PX + k) * m + i];
        acc_add(t, o);
    }
    stm(r, rps, i, acc_get(t));
}

// g_i = -sum_k A_ki r_k (A of PA limbs, r of PX limbs, formed in PX limbs), rounded to PG <= PX
// limbs: one wave per column of A, the lanes walk its rows
template <int PA, int PX, int PG>
__global__ __launch_bounds__(kThreads) void k_resid_t(const double *A, long lda, long psa, int m, int n,
                                                      const double *r, long rps, double *g, long gps, const int *skip)
{
    if (*skip) return;
    const int lane = threadIdx.x & 63;
    const int col = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (col >= n) return;
    Acc<PX> acc = acc_zero<PX>();
    int nt = 0;
    for (int i = lane; i < m; i += 64) {
        const V<PA> a = ldm<PA>(A, psa, (long)col * lda + i);
        const V<PX> rv = ldm<PX>(r, rps, i);
        casc_fma<PX, PA, PX, 0, 0, true>(acc.s, a.x, rv.x, nullptr);
        if (((++nt) % kLazy<PX>) == 0) acc = acc_from(acc_get(acc));
    }
    const V<PX> t = wave_sum(acc_get(acc));
    if (lane == 0) stm(g, gps, col, resize<PG>(neg(t)));
}

// i < n: y_i = d_i - h_i, then d_i = h_i (d of length >= n; all P limbs)
template <int P>
__global__ __launch_bounds__(kThreads) void k_aug_split(double *d, long dps, const double *h, long hps, double *y,
                                                        long yps, int n, const int *skip)
{
    if (*skip) return;
    const long i = (long)blockIdx.x * kThreads + threadIdx.x;
    if (i >= n) return;
    const V<P> hv = ldm<P>(h, hps, i);
    stm(y, yps, i, sub(ldm<P>(d, dps, i), hv));
    stm(d, dps, i, hv);
}

// x_i += d_i (d of PD <= PX limbs), i < n
template <int PX, int PD>
__global__ __launch_bounds__(kThreads) void k_md_add(double *x, long xps, const double *d, long dps, int n,
                                                     const int *skip)
{
    if (*skip) return;
    const long i = (long)blockIdx.x * kThreads + threadIdx.x;
    if (i >= n) return;
    stm(x, xps, i, add(ldm<PX>(x, xps, i), resize<PX>(ldm<PD>(d, dps, i))));
}

// x_i += d_i (d of PD <= PX limbs); norms[0] = max |d_i|, norms[1] = max |x_i| (leading limbs;
// non-negative doubles ordered as their bit patterns; both zero on entry)
template <int PX, int PD>
__global__ __launch_bounds__(kThreads) void k_refine_add(double *x, long xps, const double *d, long dps, int n,
                                                         unsigned long long *norms, const int *skip)
{
    if (*skip) return;
    const long i = (long)blockIdx.x * kThreads + threadIdx.x;
    if (i >= n) return;
    const V<PD> dv = ldm<PD>(d, dps, i);
    const V<PX> xn = add(ldm<PX>(x, xps, i), resize<PX>(dv));
    stm(x, xps, i, xn);
    atomicMax(&norms[0], (unsigned long long)__double_as_longlong(fabs(dv.x[0])));
    atomicMax(&norms[1], (unsigned long long)__double_as_longlong(fabs(xn.x[0])));
}

// After refinement step it: stop (*done = 1) once x has converged to PX limbs, judged from the
// correction norms d_k = max |d| of the steps so far: converged when d_it <= u max|x|, or when
// the next correction, estimated from the observed contraction as d_it^2 / d_(it-1), would be
// below u max|x| (u = 2^-(53 PX - (PX - 1))).  Otherwise the next step's norms are cleared
// (they hold -1 until a step runs, so the steps taken can be counted).  One thread.
template <int PX>
__global__ void k_refine_check(int it, int iters, double *norms, int *done)
{
    if (threadIdx.x != 0 || *done) return;
    const double u = ldexp(1.0, -(53 * PX - (PX - 1)));
    const double d = norms[2 * it], xm = norms[2 * it + 1];
    bool conv = d <= u * xm;
    if (!conv && it > 0) {
        const double dp = norms[2 * it - 2];
        conv = dp > 0.0 && d * (d / dp) <= u * xm;
    }
    if (conv) {
        *done = 1;
    } else if (it + 1 < iters) {
        norms[2 * it + 2] = 0.0;
        norms[2 * it + 3] = 0.0;
    }
}

namespace {
// norms := -1 (steps not taken), except step 0's pair := 0; *done := 0
__global__ void k_refine_init(double *norms, int iters, int *done)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < 2 * iters) norms[i] = (i < 2) ? 0.0 : -1.0;
    if (i == 0) *done = 0;
}
}  // namespace

namespace {
__global__ void k_zero_f64(double *p, long n)
{
    const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = 0.0;
}
}  // namespace

// ============================================================================ small kernels
namespace {
__global__ void k_zero_u32(unsigned *p, int n)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = 0u;
}

// before a factorisation: barrier counters (ctr, n of them), the time-out flag and the exchange words
__global__ void k_zero_sync(unsigned *ctr, int n, int *err, unsigned long long *tags, int ntag)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    for (int k = i; k < n; k += gridDim.x * blockDim.x) ctr[k] = 0u;
    if (i < 4) err[i] = 0;
    if (i < ntag) tags[i] = 0ull;
}

__global__ void k_copy(const double *src, long sps, double *dst, long dps, int n, int P)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n)
        for (int k = 0; k < P; ++k) dst[k * dps + i] = src[k * sps + i];
}

// k_copy unless *skip
__global__ void k_copy_if(const double *src, long sps, double *dst, long dps, int n, int P, const int *skip)
{
    if (*skip) return;
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n)
        for (int k = 0; k < P; ++k) dst[k * dps + i] = src[k * sps + i];
}

// *d_info = smallest 1-based i with R(i,i) exactly zero, else 0
__global__ __launch_bounds__(kThreads) void k_diag_check(const double *R, long ldr, long ps, int n, int P, int *d_info)
{
    __shared__ int smin;
    if (threadIdx.x == 0) smin = INT_MAX;
    __syncthreads();
    for (int i = threadIdx.x; i < n; i += kThreads) {
        bool z = true;
        for (int k = 0; k < P; ++k) z = z && (R[k * ps + (long)i * ldr + i] == 0.0);
        if (z) atomicMin(&smin, i);
    }
    __syncthreads();
    if (threadIdx.x == 0) *d_info = (smin == INT_MAX) ? 0 : smin + 1;
}

// A grid barrier of the factorisation timed out (*err != 0): *d_info := -1 (x unspecified)
__global__ void k_fold_err(const int *err, int *d_info)
{
    if (threadIdx.x == 0 && *err != 0) *d_info = -1;
}

// *d_info := -1 if a grid barrier timed out, else 0
__global__ void k_set_info(const int *err, int *d_info)
{
    if (threadIdx.x == 0) *d_info = (*err != 0) ? -1 : 0;
}
}  // namespace

// ============================================================================ tile inversion
// X = U^{-1} for upper-triangular tiles, NC columns per workgroup.  Column j solves
// U x = e_j (paper Algorithm 1, stage 1); here all NC columns advance together one row
// at a time from the bottom: x_i = r_i * d_i, then r_k -= U(k,i) x_i for k < i.
// d_i = 1/U(i,i), or supplied (then U's diagonal is not read): forming T from
// K = striu(Y^T Y) + diag(1/beta) passes d_i = beta_i, which also covers beta_i = 0.
struct InvArgs {
    const double *U;  // tile t: U + t * ustride
    long ldu, psu, ustride;
    const double *dsup;  // supplied diagonal (tile t: dsup + t * tile), or null
    long dps;
    double *X;  // tile t: X + t * xstride, ld ldx
    long ldx, psx, xstride;
    int tile;
};

template <int P, int NC, int RPT>
__global__ __launch_bounds__(kThreads) void k_invert(InvArgs g)
{
    constexpr int RG = kThreads / NC;  // row groups
    __shared__ double sD[256 * P];
    __shared__ double sX[2][NC * P];
    __shared__ double sU[2][256 * P];  // column i of the tile; column i-1 is loaded during step i
    const int t = blockIdx.y;
    const int c0 = blockIdx.x * NC;
    const int tid = threadIdx.x;
    const int jl = tid % NC, rg = tid / NC;
    const int j = c0 + jl;
    const double *U = g.U + (long)t * g.ustride;
    double *X = g.X + (long)t * g.xstride;
    const int c1 = min(c0 + NC, g.tile);

    for (int i = tid; i < c1; i += kThreads) {
        V<P> d;
        if (g.dsup)
            d = ldm<P>(g.dsup + (long)t * g.tile, g.dps, i);
        else
            d = recip(ldm<P>(U, g.psu, (long)i * g.ldu + i));
        lds_st(&sD[i * P], d);
    }
    // the rows' right-hand sides stay lazy accumulators (level sums), renormalised every
    // kLazy<P> steps and when their row is published
    Acc<P> r[RPT];
#pragma unroll
    for (int q = 0; q < RPT; ++q) {
        const int k = rg + q * RG;
        r[q] = acc_from((k == j) ? from_double<P>(1.0) : zero<P>());
        if (j < g.tile && k < g.tile && k > j) stm(X, g.psx, (long)j * g.ldx + k, zero<P>());
    }
    if (c1 > 0 && tid < c1 - 1) lds_st(&sU[(c1 - 1) & 1][tid * P], ldm<P>(U, g.psu, (long)(c1 - 1) * g.ldu + tid));
    __syncthreads();
    for (int i = c1 - 1; i >= 0; --i) {
        const int buf = i & 1;
        // column i-1 (rows above i-1) for the next step, in flight during this one
        V<P> unext = zero<P>();
        const bool pre = i > 0 && tid < i - 1;
        if (pre) unext = ldm<P>(U, g.psu, (long)(i - 1) * g.ldu + tid);
        // owner of row i in column j publishes x_ij
        if (j < c1 && j >= i && (i % RG) == rg) {
            const int qi = i / RG;
            V<P> xv = zero<P>();
#pragma unroll
            for (int q = 0; q < RPT; ++q)
                if (q == qi) xv = mul(acc_get(r[q]), lds_ld<P>(&sD[i * P]));
            lds_st(&sX[buf][jl * P], xv);
            stm(X, g.psx, (long)j * g.ldx + i, xv);
        }
        __syncthreads();
        if (j < c1 && j >= i) {
            const V<P> xv = neg(lds_ld<P>(&sX[buf][jl * P]));
            const bool renorm = ((c1 - i) % kLazy<P>) == 0;
#pragma unroll
            for (int q = 0; q < RPT; ++q) {
                const int k = rg + q * RG;
                if (k < i) {
                    acc_fma(r[q], lds_ld<P>(&sU[buf][k * P]), xv);
                    if (renorm) r[q] = acc_from(acc_get(r[q]));
                }
            }
        }
        // sU[buf ^ 1] was last read in step i + 1, before this step's barrier
        if (pre) lds_st(&sU[buf ^ 1][tid * P], unext);
    }
}

// Blocked tile inversion (Algorithm 1, stage 1, for tiles of 64 rows or more): with the
// 32 x 32 diagonal blocks U_II of every tile inverted first (k_invert, 32 dependent row steps
// instead of one per row of the tile), the blocks of X = U^-1 above the diagonal follow by
// block rows from the bottom, X_IK = -X_II sum_{I < J <= K} U_IJ X_JK.  Workgroup (slice, K - 1,
// tile) forms block column K for NCB of its columns: thread (r, c) holds row r of the block
// row being formed, column c.  The block column is kept in LDS; the diagonal blocks' inverses
// come from Xd (nb x nb each, ld nb, tile t's block I at Xd + (t NB + I) nb^2, plane stride
// dps).
constexpr int kInvNB = 32;  // rows of a diagonal block

template <int P>
constexpr int inv_blk_cols()
{
    return P >= 8 ? 4 : 8;  // columns per workgroup: (tile rows x NCB x P) doubles of LDS <= 64 KiB
}

struct InvBlkArgs {
    const double *U;  // tile t at U + t (tile ldu + tile)
    long ldu, psu;
    const double *Xd;  // diagonal-block inverses
    long dps;
    double *X;  // tile t at X + t tile^2, ld tile, plane stride psx
    long psx;
    int tile;
    const int *skip;
};

template <int P>
__global__ __launch_bounds__(kThreads) void k_inv_blocks(InvBlkArgs g)
{
    constexpr int NB = kInvNB, NCB = inv_blk_cols<P>();
    constexpr int NTH = NB * NCB;  // threads that hold an entry
    __shared__ double sX[256 * NCB * P];  // rows 0 .. (K+1) NB - 1 of this workgroup's columns
    __shared__ double sR[NB * NCB * P];
    if (g.skip && *g.skip) return;
    const int tid = threadIdx.x;
    const int r = tid % NB, c = tid / NB;
    const int K = blockIdx.y + 1, t = blockIdx.z;
    const int col = K * NB + blockIdx.x * NCB + c;  // column of the tile
    const bool act = tid < NTH;
    const long tt = (long)t * g.tile;
    const double *U = g.U + tt * g.ldu + tt;
    double *X = g.X + tt * g.tile;
    const int nbt = g.tile / NB;
    auto xd = [&](int I, int row, int k) __attribute__((always_inline)) {
        return ldm<P>(g.Xd, g.dps, ((long)t * nbt + I) * NB * NB + (long)k * NB + row);
    };
    // the diagonal block X_KK: copied into place and into LDS (block column 1 also places X_00)
    if (act) {
        const V<P> v = xd(K, r, blockIdx.x * NCB + c);
        lds_st(&sX[((K * NB + r) * NCB + c) * P], v);
        stm(X, g.psx, (long)col * g.tile + K * NB + r, v);
        if (K == 1) {
            const int c0 = blockIdx.x * NCB + c;
            stm(X, g.psx, (long)c0 * g.tile + r, xd(0, r, c0));
        }
    }
    __syncthreads();
    for (int I = K - 1; I >= 0; --I) {
        // R(r, c) = sum over the rows k of block rows I+1 .. K of U(I NB + r, k) X(k, c)
        if (act) {
            Acc<P> a0 = acc_zero<P>(), a1 = acc_zero<P>();
            const int k0 = (I + 1) * NB, k1 = (K + 1) * NB;
            int nt = 0;
            for (int k = k0; k < k1; k += 2) {
                acc_fma(a0, ldm<P>(U, g.psu, (long)k * g.ldu + I * NB + r), lds_ld<P>(&sX[(k * NCB + c) * P]));
                acc_fma(a1, ldm<P>(U, g.psu, (long)(k + 1) * g.ldu + I * NB + r), lds_ld<P>(&sX[((k + 1) * NCB + c) * P]));
                if ((++nt) % kLazy<P> == 0) {
                    a0 = acc_from(acc_get(a0));
                    a1 = acc_from(acc_get(a1));
                }
            }
            acc_add_acc(a0, a1);
            lds_st(&sR[(r * NCB + c) * P], acc_get(a0));
        }
        __syncthreads();
        // X_IK(r, c) = -sum_{k >= r} X_II(r, k) R(k, c)
        if (act) {
            Acc<P> a = acc_zero<P>();
            int nt = 0;
            for (int k = r; k < NB; ++k) acc_fma_step(a, xd(I, r, k), lds_ld<P>(&sR[(k * NCB + c) * P]), nt++);
            const V<P> v = neg(acc_get(a));
            lds_st(&sX[((I * NB + r) * NCB + c) * P], v);
            stm(X, g.psx, (long)col * g.tile + I * NB + r, v);
        }
        __syncthreads();
    }
}

// x_i := Xinv_i y_i, one wave per output row
template <int P>
__global__ __launch_bounds__(kThreads) void k_bs_xi(const double *Xi, long ldx, long psx, const double *y, long yps,
                                                   double *x, long xps, int tile, const int *skip)
{
    if (skip && *skip) return;
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    const int row = blockIdx.x * 4 + wid;
    if (row >= tile) return;
    Acc<P> acc = acc_zero<P>();
    int nt = 0;
    for (int c = row + lane; c < tile; c += 64) acc_fma_step(acc, ldm<P>(Xi, psx, (long)c * ldx + row), ldm<P>(y, yps, c), nt++);
    const V<P> s = wave_sum(acc_get(acc));
    if (lane == 0) stm(x, xps, row, s);
}

// The update of the sweep split over column slices, for more workgroups in flight: workgroup
// (row block, slice cs) forms part[cs][row] = R(row, cols of slice cs) x_i(slice) for 64 rows,
// the slice's columns split over the four waves (four accumulators per lane each); k_bs_comb then
// subtracts the slices' partial sums from y in a fixed order.
constexpr int kBsSlices = 4;

template <int P>
__global__ __launch_bounds__(kThreads) void k_bs_upd_part(const double *Rc, long ldr, long psr, const double *xi,
                                                         long xps, double *part, long pps, int rows, int tile,
                                                         const int *skip)
{
    __shared__ double sx[256 * P];
    __shared__ double sp[4][64 * P];
    if (skip && *skip) return;
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    const int per = tile / kBsSlices;
    const int s0 = blockIdx.y * per;
    for (int c = threadIdx.x; c < per; c += kThreads) lds_st(&sx[c * P], ldm<P>(xi, xps, s0 + c));
    __syncthreads();
    const long row = (long)blockIdx.x * 64 + lane;
    const int q = (per + 3) / 4;
    const int cb = wid * q, ce = min(per, cb + q);
    constexpr int NA = 4;
    Acc<P> acc[NA];
#pragma unroll
    for (int a = 0; a < NA; ++a) acc[a] = acc_zero<P>();
    if (row < rows) {
        int nt = 0;
        for (int c = cb; c < ce; c += NA) {
            V<P> u[NA];
#pragma unroll
            for (int k = 0; k < NA; ++k) u[k] = (c + k < ce) ? ldm<P>(Rc, psr, (long)(s0 + c + k) * ldr + row) : zero<P>();
#pragma unroll
            for (int k = 0; k < NA; ++k)
                if (c + k < ce) acc_fma(acc[k], u[k], lds_ld<P>(&sx[(c + k) * P]));
            if ((++nt) % kLazy<P> == 0) {
#pragma unroll
                for (int a = 0; a < NA; ++a) acc[a] = acc_from(acc_get(acc[a]));
            }
        }
#pragma unroll
        for (int a = 1; a < NA; ++a) acc_add_acc(acc[0], acc[a]);
    }
    lds_st(&sp[wid][lane * P], acc_get(acc[0]));
    __syncthreads();
    if (wid == 0 && row < rows) {
        V<P> v = lds_ld<P>(&sp[0][lane * P]);
        for (int w = 1; w < 4; ++w) v = add(v, lds_ld<P>(&sp[w][lane * P]));
        stm(part + (long)blockIdx.y * rows, pps, row, v);
    }
}

// y(row) -= sum over the slices cs of part[cs][row] (in slice order)
template <int P>
__global__ __launch_bounds__(kThreads) void k_bs_comb(const double *part, long pps, double *y, long yps, int rows,
                                                     const int *skip)
{
    if (skip && *skip) return;
    const long row = (long)blockIdx.x * kThreads + threadIdx.x;
    if (row >= rows) return;
    V<P> v = ldm<P>(part, pps, row);
    for (int cs = 1; cs < kBsSlices; ++cs) v = add(v, ldm<P>(part + (long)cs * rows, pps, row));
    stm(y, yps, row, sub(ldm<P>(y, yps, row), v));
}

// The transposed sweep (forward substitution with R^T, whose diagonal tiles have the inverses
// Xinv_i^T): h_i := Xinv_i^T g_i, one wave per output row; skipped while *skip is set
template <int P>
__global__ __launch_bounds__(kThreads) void k_bs_xi_t(const double *Xi, long ldx, long psx, const double *g, long gps,
                                                     double *h, long hps, int tile, const int *skip)
{
    if (skip && *skip) return;
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    const int row = blockIdx.x * 4 + wid;
    if (row >= tile) return;
    Acc<P> acc = acc_zero<P>();
    int nt = 0;
    for (int c = lane; c <= row; c += 64) acc_fma_step(acc, ldm<P>(Xi, psx, (long)row * ldx + c), ldm<P>(g, gps, c), nt++);
    const V<P> s = wave_sum(acc_get(acc));
    if (lane == 0) stm(h, hps, row, s);
}

// g(col) -= sum_k R(k, col) h_k over the tile's rows k, for the ncols columns right of the tile
// (R points at the tile's first row and the first of those columns); one wave per column
template <int P>
__global__ __launch_bounds__(kThreads) void k_bs_upd_t(const double *R, long ldr, long psr, const double *h, long hps,
                                                      double *g, long gps, int ncols, int tile, const int *skip)
{
    if (skip && *skip) return;
    const int lane = threadIdx.x & 63;
    const int col = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (col >= ncols) return;
    Acc<P> acc = acc_zero<P>();
    int nt = 0;
    for (int k = lane; k < tile; k += 64) acc_fma_step(acc, ldm<P>(R, psr, (long)col * ldr + k), ldm<P>(h, hps, k), nt++);
    const V<P> s = wave_sum(acc_get(acc));
    if (lane == 0) stm(g, gps, col, sub(ldm<P>(g, gps, col), s));
}

// y(0:rows) -= R(0:rows, cols of tile i) x_i ; 64 rows per workgroup, the tile's columns
// split over the 4 waves and combined in a fixed order
template <int P>
__global__ __launch_bounds__(kThreads) void k_bs_upd(const double *Rc, long ldr, long psr, const double *xi, long xps,
                                                    double *y, long yps, int rows, int tile, const int *skip)
{
    __shared__ double sx[256 * P];
    __shared__ double sp[4][64 * P];
    if (skip && *skip) return;
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    for (int c = threadIdx.x; c < tile; c += kThreads) lds_st(&sx[c * P], ldm<P>(xi, xps, c));
    __syncthreads();
    const long row = (long)blockIdx.x * 64 + lane;
    const int q = (tile + 3) / 4;
    const int cb = wid * q, ce = min(tile, cb + q);
    // NA independent accumulators (column k goes to k mod NA), so that NA multiply-adds are
    // in flight at once, added in a fixed order at the end
    constexpr int NA = 4;
    Acc<P> acc[NA];
#pragma unroll
    for (int a = 0; a < NA; ++a) acc[a] = acc_zero<P>();
    if (row < rows) {
        // B columns of R per batch; the next batch's loads are issued before the current
        // batch's multiply-adds, so the HBM latency overlaps the accumulation
        constexpr int B = 32 / P < NA ? NA : 32 / P;
        static_assert(B % NA == 0, "k_bs_upd batch");
        V<P> cur[B], nxt[B];
        auto load = [&](V<P> (&u)[B], int c) __attribute__((always_inline)) {
#pragma unroll
            for (int k = 0; k < B; ++k) u[k] = (c + k < ce) ? ldm<P>(Rc, psr, (long)(c + k) * ldr + row) : zero<P>();
        };
        load(cur, cb);
        int nt = 0;
        for (int c = cb; c < ce; c += B) {
            if (c + B < ce) load(nxt, c + B);
#pragma unroll
            for (int k = 0; k < B; ++k)
                if (c + k < ce) acc_fma(acc[k % NA], cur[k], lds_ld<P>(&sx[(c + k) * P]));
            nt += B / NA;
            if (nt % kLazy<P> == 0) {
#pragma unroll
                for (int a = 0; a < NA; ++a) acc[a] = acc_from(acc_get(acc[a]));
            }
#pragma unroll
            for (int k = 0; k < B; ++k) cur[k] = nxt[k];
        }
#pragma unroll
        for (int a = 1; a < NA; ++a) acc_add_acc(acc[0], acc[a]);
    }
    lds_st(&sp[wid][lane * P], acc_get(acc[0]));
    __syncthreads();
    if (wid == 0 && row < rows) {
        V<P> s = lds_ld<P>(&sp[0][lane * P]);
        for (int w = 1; w < 4; ++w) s = add(s, lds_ld<P>(&sp[w][lane * P]));
        stm(y, yps, row, sub(ldm<P>(y, yps, row), s));
    }
}

// ============================================================================ one-launch back substitution
// R x = y for one right-hand side, every row block of kTrB rows by its own workgroup (Algorithm 1's sweep
// turned into a data flow): workgroup b owns row block j = nblk - 1 - b, inverts its diagonal block U_j, adds
// R_ji x_i to its sum as the x_i are published, and publishes x_j = U_j^-1 (y_j - sum).
// The words of x hold a signalling NaN until they are published: no arithmetic result is one, so the data
// are their own flag and a wait is one polled load.  A workgroup waits
// for lower-numbered ones only, and workgroups start in order, so the lowest unfinished one always runs
// whatever is resident; the polls are bounded all the same.  Wave w holds rows 4 w .. 4 w + 3, its lanes 16
// columns of each (and the 16 after them): sums over a row stay in the wave.
// Bound by the chain of nblk steps; the reading of R goes on beside it (the next blocks in flight).  Before,
// the tiles were inverted in full, b^3/6 multiply-adds each, and every tile took three launches.  n = 128 (tile 32),
// 1024 (tile 128), 8192 (tile 128), before and now: dd 67, 156, 822 -> 34, 103, 458 us, qd 105, 321, 1709 -> 91, 271,
// 1220 us; od n = 4096, tile 128, 3689 -> 3008 us (smaller ones by tiles: backsub_by_tiles); qd n = 17920, tile 256,
// 4194 -> 3123 us (past 256 blocks the later workgroups start when the first end, and read R at 1.7 TB/s).
// AH = 0: the last block's product, its sum, U_j^-1 and another sum all stand between x_{j+1} and x_j.
// AH = 2: with M_a = U_j^-1 R_{j,j+a}, x_j = z_j - M_2 x_{j+2} - M_1 x_{j+1}, where z_j = U_j^-1 (y_j -
// sum_{i > j+2} R_ji x_i) is ready before x_{j+2} comes: a step is one exchange, two multiply-adds a thread and
// one sum in the wave.  The M_a are formed at the start, which costs the first steps their wait (qd 80 us),
// so this form takes over where the chain is long (trsv_ahead).
// Registers: dd 93 / 119 (AH = 0 / 2), qd 170 / 218; od takes all 256 of two waves a SIMD and spills 28 / 122 of them
// (92 / 356 bytes a lane).
constexpr int kTrB = 32;    // rows of a block
constexpr int kTrNT = 512;  // threads of a workgroup
constexpr unsigned long long kTrEmpty = 0x7ff4000000007153ull;

struct TrsvArgs {
    const double *R;
    long ldr, psr;
    const double *y;  // may be x (yps = xps): a workgroup reads only the rows it writes
    long yps;
    double *x;
    long xps;
    unsigned long long *xw;  // P planes of n words, kTrEmpty on entry
    int n, nblk;
    int *err, *d_info;
    unsigned spin;
};

template <int P>
struct TrsvLds {
    double inv[kTrB * P * kTrB];  // U_j, then its inverse: limb k of column c at (c P + k) kTrB + row
    double nxt[kTrB * P * kTrB];  // R_{j,j+1}, the same layout
    double row[2][kTrB * P];      // inversion: the row just formed
    double diag[kTrB * P];
    double x[2][2 * kTrB * P];    // x_i, x_{i-1}
    double v[kTrB * P];           // y_j - sum
};

template <int P, int AH>
__global__ __launch_bounds__(kTrNT, 2) void k_trsv(TrsvArgs g)
{
    constexpr int B = kTrB, NT = kTrNT;
    constexpr int U = P <= 4 ? 2 : 1;  // blocks of the sum at a time (od: registers)
    static_assert(B == 32 && NT == 16 * B, "k_trsv layout");
    __shared__ TrsvLds<P> lds;
    const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
    const int j = g.nblk - 1 - (int)blockIdx.x;
    const int r0 = j * B, nr = min(B, g.n - r0);
    const int row = 4 * wid + (lane >> 4), c0 = lane & 15;  // columns c0, c0 + 16 of a block
    const double *Rrow = g.R + r0 + (row < nr ? row : 0);
    // R_ji and R_j,i-1 at this thread's columns (R_j,i-1 zero where i - 1 is below the sum's last block)
    V<P> rb[2 * U];
    auto fetch = [&](int i, int last) __attribute__((always_inline)) {
#pragma unroll
        for (int t = 0; t < 2 * U; ++t) {
            const long c = (long)(i - t / 2) * B + c0 + 16 * (t & 1);
            rb[t] = (c < g.n && i - t / 2 >= last) ? ldm<P>(Rrow, g.psr, c * g.ldr) : zero<P>();
        }
    };
    auto at = [&](const double *m, int c, int r) __attribute__((always_inline)) {
        V<P> v;
#pragma unroll
        for (int k = 0; k < P; ++k) v.x[k] = m[(c * P + k) * B + r];
        return v;
    };
    // the sum over a row's 16 lanes, in every one of them
    auto row_sum = [&](Acc<P> t) __attribute__((always_inline)) {
#pragma unroll
        for (int m = 1; m < 16; m <<= 1) {
            acc_add_acc(t, shfl_xor_acc(t, m));
            if (kLazy<P> <= 4 && m == 2) t = acc_from(acc_get(t));
        }
        return acc_get(t);
    };
    // words of element e of x (zero where e is outside x): loaded, and whether they are there
    auto load_x = [&](long e, bool want, unsigned long long (&wd)[P]) __attribute__((always_inline)) {
#pragma unroll
        for (int w = 0; w < P; ++w)
            wd[w] = (want && e < g.n)
                        ? __hip_atomic_load(g.xw + (long)w * g.n + e, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)
                        : 0ull;
    };
    auto there = [&](const unsigned long long (&wd)[P]) __attribute__((always_inline)) {
        bool ok = true;
#pragma unroll
        for (int w = 0; w < P; ++w) ok = ok && wd[w] != kTrEmpty;
        return ok;
    };
    // after a failed poll: whether to give up.  Who gives up writes the status: its x carries no order, so no
    // other workgroup that has taken it can be sure to see *err.
    auto give_up = [&](unsigned &spins) __attribute__((always_inline)) {
        if ((spins & 255u) == 255u && __hip_atomic_load(g.err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0) return true;
        if (++spins > g.spin) {
            __hip_atomic_store(g.err, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __hip_atomic_store(g.d_info, -1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            return true;
        }
        return false;
    };
    auto value = [&](const unsigned long long (&wd)[P]) __attribute__((always_inline)) {
        V<P> v;
#pragma unroll
        for (int k = 0; k < P; ++k) v.x[k] = __longlong_as_double((long long)wd[k]);
        return v;
    };

    const int ib = j + 1 + AH;  // the last block of the sum
    const V<P> yj = row < nr ? ldm<P>(g.y, g.yps, r0 + row) : zero<P>();
    if (g.nblk - 1 >= ib) fetch(g.nblk - 1, ib);
    // ---- U_j^-1: all columns advance together, one row at a time from the bottom; thread (c, gq) holds
    //      rows gq and gq + 16 of column c.  Then M_j.
    for (int e = tid; e < B * B; e += NT) {
        const int r = e % B, c = e / B;
        const V<P> u = (r <= c && c < nr) ? ldm<P>(g.R, g.psr, (long)(r0 + c) * g.ldr + r0 + r)
                                          : (r == c ? from_double<P>(1.0) : zero<P>());
#pragma unroll
        for (int k = 0; k < P; ++k) lds.inv[(c * P + k) * B + r] = u.x[k];
    }
    __syncthreads();
    if (tid < B) lds_st(&lds.diag[tid * P], recip(at(lds.inv, tid, tid)));
    {
        const int c = tid & 31, gq = tid >> 5;
        Acc<P> a[2];
        V<P> res[2];
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            a[q] = acc_from(gq + 16 * q == c ? from_double<P>(1.0) : zero<P>());
            res[q] = zero<P>();
        }
        __syncthreads();
        for (int i = nr - 1; i >= 0; --i) {  // (the last block may have fewer rows than B)
            if (gq == (i & 15)) {
                const V<P> xv = mul(acc_get(i >= 16 ? a[1] : a[0]), lds_ld<P>(&lds.diag[i * P]));
                lds_st(&lds.row[i & 1][c * P], xv);
                if (i >= 16)
                    res[1] = xv;
                else
                    res[0] = xv;
            }
            __syncthreads();
            const V<P> xv = neg(lds_ld<P>(&lds.row[i & 1][c * P]));
            const bool renorm = ((nr - i) % kLazy<P>) == 0;
#pragma unroll
            for (int q = 0; q < 2; ++q)
                if (gq + 16 * q < i) {
                    acc_fma(a[q], at(lds.inv, i, gq + 16 * q), xv);
                    if (renorm) a[q] = acc_from(acc_get(a[q]));
                }
        }
        __syncthreads();
#pragma unroll
        for (int q = 0; q < 2; ++q)
#pragma unroll
            for (int k = 0; k < P; ++k) lds.inv[(c * P + k) * B + gq + 16 * q] = res[q].x[k];
        __syncthreads();
    }
    V<P> mj[AH > 0 ? AH : 1][2];  // M_a(row, c0), M_a(row, c0 + 16) at a - 1
    if constexpr (AH > 0) {
#pragma unroll
        for (int a = 0; a < AH; ++a) {
            const long rc = r0 + (long)B * (a + 1);
            for (int e = tid; e < B * B; e += NT) {
                const int r = e % B, c = e / B;
                const V<P> m = (r < nr && rc + c < g.n) ? ldm<P>(g.R, g.psr, (rc + c) * g.ldr + r0 + r) : zero<P>();
#pragma unroll
                for (int k = 0; k < P; ++k) lds.nxt[(c * P + k) * B + r] = m.x[k];
            }
            __syncthreads();
            Acc<P> a0 = acc_zero<P>(), a1 = acc_zero<P>();
#pragma unroll 1
            for (int k = 4 * wid, nt = 0; k < B; ++k) {
                if (k >= row) {  // U_j^-1 is upper triangular; a product with its zeros would spread a NaN or Inf of row k downwards
                    const V<P> u = at(lds.inv, k, row);
                    acc_fma(a0, u, at(lds.nxt, c0, k));
                    acc_fma(a1, u, at(lds.nxt, c0 + 16, k));
                }
                if (++nt % kLazy<P> == 0) {
                    a0 = acc_from(acc_get(a0));
                    a1 = acc_from(acc_get(a1));
                }
            }
            mj[a][0] = acc_get(a0);
            mj[a][1] = acc_get(a1);
            __syncthreads();
        }
    }
    // Everything below runs twice: first on nothing, with no wait and no store, so that its instructions are
    // in this CU's cache when the chain comes by (each step of the chain is another CU's, and fetches of
    // straight-line code that it had never run cost several us a step).
    // Wave 0 polls for blocks i and i - 1 at once (a lane an element) while all work on the two before them;
    // workgroups whose turn is far off poll less often, so that the words the chain waits for are not fought over.
    unsigned long long wd[P];
    auto ask = [&](int i) __attribute__((always_inline)) {
        load_x(lane < B ? (long)i * B + lane : (long)(i - 1) * B + lane - B, lane < B || (U == 2 && i - 1 >= ib), wd);
    };
    auto receive = [&](int i, int buf) __attribute__((always_inline)) {  // the words asked for
        unsigned spins = 0;
        while (!__all(there(wd))) {
            if (i > j + 8)
                __builtin_amdgcn_s_sleep(64);
            else if (i > ib + 1)
                __builtin_amdgcn_s_sleep(8);
            if (give_up(spins)) break;
            ask(i);
        }
        lds_st(&lds.x[buf][lane * P], value(wd));
    };
#pragma unroll 1
    for (int live = P <= 4 ? 0 : 1; live < 2; ++live) {  // od's code exceeds the cache
        // ---- the sum of R_ji x_i, i >= ib, U blocks at a time
        Acc<P> acc[2] = {acc_zero<P>(), acc_zero<P>()};
        const int i1 = live ? g.nblk - 1 : ib - 1;
        if (wid == 0 && i1 >= ib) {
            ask(i1);
            receive(i1, 0);
        }
        int nt = 0;
#pragma unroll 1
        for (int i = i1, buf = 0; i >= ib; i -= U, buf ^= 1) {
            V<P> cur[2 * U];
#pragma unroll
            for (int t = 0; t < 2 * U; ++t) cur[t] = rb[t];
            if (i - U >= ib) fetch(i - U, ib);
            __syncthreads();
            if (wid == 0 && i - U >= ib) ask(i - U);
#pragma unroll
            for (int t = 0; t < 2 * U; ++t)
                acc_fma(acc[t & 1], cur[t], lds_ld<P>(&lds.x[buf][(c0 + 16 * t) * P]));
            nt += U;
            if (nt % kLazy<P> == 0) {
#pragma unroll
                for (int t = 0; t < 2; ++t) acc[t] = acc_from(acc_get(acc[t]));
            }
            if (wid == 0 && i - U >= ib) receive(i - U, buf ^ 1);
        }
        acc_add_acc(acc[0], acc[1]);
        const V<P> sum = row_sum(acc_from(acc_get(acc[0])));
        if (c0 == 0) lds_st(&lds.v[row * P], row < nr ? sub(yj, sum) : zero<P>());
        __syncthreads();
        // ---- z_j = U_j^-1 (y_j - sum), x_j = z_j - M_2 x_{j+2} - M_1 x_{j+1}
        V<P> xj;
        {
            Acc<P> t0 = acc_zero<P>(), t1 = acc_zero<P>();
            if (c0 >= row) acc_fma(t0, at(lds.inv, c0, row), lds_ld<P>(&lds.v[c0 * P]));
            if (c0 + 16 >= row) acc_fma(t1, at(lds.inv, c0 + 16, row), lds_ld<P>(&lds.v[(c0 + 16) * P]));
            acc_add_acc(t0, t1);
            xj = row_sum(t0);
        }
        if constexpr (AH > 0) {
#pragma unroll
            for (int a = AH - 1; a >= 0; --a) {
                if (j + 1 + a >= g.nblk) continue;
                V<P> xv[2];
                unsigned long long wa[P], wb[P];
                unsigned spins = 0;
                for (;;) {  // every wave polls for itself: this lane's two elements
                    load_x((long)(j + 1 + a) * B + c0, true, wa);
                    load_x((long)(j + 1 + a) * B + c0 + 16, true, wb);
                    if (__all(there(wa) && there(wb)) || !live || give_up(spins)) break;
                }
                xv[0] = value(wa);
                xv[1] = value(wb);
                Acc<P> t0 = acc_zero<P>(), t1 = acc_zero<P>();
                acc_fma(t0, mj[a][0], xv[0]);
                acc_fma(t1, mj[a][1], xv[1]);
                acc_add_acc(t0, t1);
                xj = sub(xj, row_sum(t0));
            }
        }
        if (live && c0 == 0 && row < nr) {
#pragma unroll
            for (int k = 0; k < P; ++k)
                __hip_atomic_store(g.xw + (long)k * g.n + r0 + row, (unsigned long long)__double_as_longlong(xj.x[k]),
                                   __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            stm(g.x, g.xps, r0 + row, xj);
        }
        __syncthreads();  // lds.v is written again
    }
    // a wait that gave up before this launch (the factorisation's)
    if (j == 0 && tid == 0 && __hip_atomic_load(g.err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0) *g.d_info = -1;
}

namespace {
// before k_trsv: every word of x empty, *d_info = smallest 1-based i with R(i,i) exactly zero, else 0, and with
// clear_err the time-out flag
__global__ __launch_bounds__(kThreads) void k_trsv_init(unsigned long long *xw, long nw, int *err, int clear_err,
                                                       const double *R, long ldr, long ps, int n, int P, int *d_info)
{
    for (long i = (long)blockIdx.x * kThreads + threadIdx.x; i < nw; i += (long)gridDim.x * kThreads) xw[i] = kTrEmpty;
    if (blockIdx.x != 0) return;
    __shared__ int smin;
    if (threadIdx.x == 0) {
        smin = INT_MAX;
        if (clear_err) *err = 0;
    }
    __syncthreads();
    for (int i = threadIdx.x; i < n; i += kThreads) {
        bool z = true;
        for (int k = 0; k < P; ++k) z = z && (R[k * ps + (long)i * ldr + i] == 0.0);
        if (z) atomicMin(&smin, i);
    }
    __syncthreads();
    if (threadIdx.x == 0) *d_info = (smin == INT_MAX) ? 0 : smin + 1;
}
}  // namespace

// ============================================================================ T, W, Q^T B helpers
// G(l, j) = y_l^T y_j (l < j) for tile block k: block (j, k), one wave per l.  The form for od and for tiles of
// fewer than 96 columns, whose 16 x 16 blocks of sums (k_gemm) leave the chip idle (gram_blocks).
template <int P>
__global__ __launch_bounds__(kThreads) void k_gram(const double *A, long lda, long ps, int m, int tile, double *G,
                                                  long gps)
{
    const int j = blockIdx.x, k = blockIdx.y;
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    const long kt = (long)k * tile;
    const double *Y = A + kt * lda + kt;
    const int h = m - (int)kt;
    double *Gk = G + kt * tile;
    for (int l = wid; l < tile; l += 4) {
        if (l >= j) {
            if (lane == 0) stm(Gk, gps, (long)j * tile + l, zero<P>());
            continue;
        }
        Acc<P> acc = acc_zero<P>();
        int nt = 0;
        for (int r = j + lane; r < h; r += 64)  // y_j is zero above row j
            acc_fma_step(acc, y_entry<P>(Y, lda, ps, r, l, h, tile), y_entry<P>(Y, lda, ps, r, j, h, tile), nt++);
        const V<P> s = wave_sum(acc_get(acc));
        if (lane == 0) stm(Gk, gps, (long)j * tile + l, s);
    }
}

// W(r, k*tile + j) = -sum_{l<=j} Y_k(r, l) T_k(l, j) for r >= k*tile; zero above.
template <int P>
__global__ __launch_bounds__(kThreads) void k_form_w(const double *A, long lda, long ps, const double *T, long ldt,
                                                    long tps, double *W, long ldw, long wps, int m, int tile)
{
    const long r = (long)blockIdx.x * kThreads + threadIdx.x;
    const int gj = blockIdx.y;
    if (r >= m) return;
    const int k = gj / tile, j = gj % tile;
    const long kt = (long)k * tile;
    if (r < kt) {
        stm(W, wps, (long)gj * ldw + r, zero<P>());
        return;
    }
    const double *Y = A + kt * lda + kt;
    const int h = m - (int)kt;
    Acc<P> acc = acc_zero<P>();
    for (int l = 0; l <= j; ++l)
        acc_fma_step(acc, y_entry<P>(Y, lda, ps, r - kt, l, h, tile), ldm<P>(T, tps, (long)gj * ldt + l), l);
    stm(W, wps, (long)gj * ldw + r, neg(acc_get(acc)));
}

// S(l, c) = Y_k(:, l)^T B(kt:, c): one wave per (l, c)
template <int P>
__global__ __launch_bounds__(kThreads) void k_tn(const double *Y, long lda, long ps, int h, int tile, const double *B,
                                                long ldb, long bps, int nrhs, double *S, long sps, const int *skip)
{
    if (skip && *skip) return;
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    const int l = blockIdx.x * 4 + wid, c = blockIdx.y;
    if (l >= tile || c >= nrhs) return;
    Acc<P> acc = acc_zero<P>();
    int nt = 0;
    for (int r = l + lane; r < h; r += 64)
        acc_fma_step(acc, y_entry<P>(Y, lda, ps, r, l, h, tile), ldm<P>(B, bps, (long)c * ldb + r), nt++);
    const V<P> s = wave_sum(acc_get(acc));
    if (lane == 0) stm(S, sps, (long)c * tile + l, s);
}

// U(i, c) = sum_l op(T)(i, l) S(l, c) (op(T) = T^T: l <= i, or T: l >= i), one thread per (i, c): for tiles of at
// most four columns, whose sums are too short for a wave (od, tile 1 and 4: 7 and 14 us a launch, k_trmm_v 13 and 18).
template <int P, bool TRANS>
__global__ __launch_bounds__(kThreads) void k_trmm(const double *T, long ldt, long tps, const double *S, long sps,
                                                  double *U, int tile, int nrhs, const int *skip)
{
    if (skip && *skip) return;
    const int i = blockIdx.x * kThreads + threadIdx.x, c = blockIdx.y;
    if (i >= tile || c >= nrhs) return;
    Acc<P> acc = acc_zero<P>();
    int nt = 0;
    for (int l = TRANS ? 0 : i; l < (TRANS ? i + 1 : tile); ++l)
        acc_fma_step(acc, ldm<P>(T, tps, TRANS ? (long)i * ldt + l : (long)l * ldt + i),
                     ldm<P>(S, sps, (long)c * tile + l), nt++);
    stm(U, sps, (long)c * tile + i, acc_get(acc));
}

// B(r, c) -= sum_l Y(r, l) U(l, c), one thread per row: for one or two columns of Y, and for a few of them where
// the rows alone fill the chip (qd, tile 8, 2048 rows x 256 columns: 19 us a launch, k_nn_sub_v 28, k_gemm 26).
template <int P>
__global__ __launch_bounds__(kThreads) void k_nn_sub(const double *Y, long lda, long ps, int h, int tile, const double *U,
                                                    long ups, double *B, long ldb, long bps, const int *skip)
{
    if (skip && *skip) return;
    const long r = (long)blockIdx.x * kThreads + threadIdx.x;
    const int c = blockIdx.y;
    if (r >= h) return;
    Acc<P> acc = acc_from(ldm<P>(B, bps, (long)c * ldb + r));
    const long lmax = ((long)tile - 1 < r) ? (long)tile - 1 : r;
    for (int l = 0; l <= (int)lmax; ++l)
        acc_fma_step(acc, neg(y_entry<P>(Y, lda, ps, r, l, h, tile)), ldm<P>(U, ups, (long)c * tile + l), l);
    stm(B, bps, (long)c * ldb + r, acc_get(acc));
}

// The products where k_gemm's blocks are too few: U(i, c) = sum_l op(T)(i, l) S(l, c), one
// wave per (i, c), the lanes over l (op(T) = T^T: l <= i, or T: l >= i).  One thread per output with
// its chain of tile multiply-adds took 13.6 us for one dd column and tile 128; this takes 3.2.
template <int P, bool TRANS>
__global__ __launch_bounds__(kThreads) void k_trmm_v(const double *T, long ldt, long tps, const double *S, long sps,
                                                    double *U, int tile, int nrhs, const int *skip)
{
    if (skip && *skip) return;
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    const int i = blockIdx.x * 4 + wid, c = blockIdx.y;
    if (i >= tile || c >= nrhs) return;
    Acc<P> acc = acc_zero<P>();
    int nt = 0;
    for (int l = TRANS ? lane : i + lane; l < (TRANS ? i + 1 : tile); l += 64)
        acc_fma_step(acc, ldm<P>(T, tps, TRANS ? (long)i * ldt + l : (long)l * ldt + i),
                     ldm<P>(S, sps, (long)c * tile + l), nt++);
    const V<P> s = wave_sum(acc_get(acc));
    if (lane == 0) stm(U, sps, (long)c * tile + i, s);
}

// B(r, c) -= sum_l Y(r, l) U(l, c) for a few columns: 64 rows of one column per workgroup, the
// columns of Y split over the four waves (two accumulators a lane) and combined in a fixed order.
// One thread per row with its chain of tile multiply-adds (8 workgroups at 2048 rows) took 30.4 us
// (a mean over the tiles of n = 2048) for one dd column and tile 128; this takes 7.0.
template <int P>
__global__ __launch_bounds__(kThreads) void k_nn_sub_v(const double *Y, long lda, long ps, int h, int tile,
                                                      const double *U, long ups, double *B, long ldb, long bps,
                                                      const int *skip)
{
    __shared__ double su[256 * P];
    __shared__ double sp[4][64 * P];
    if (skip && *skip) return;
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6, c = blockIdx.y;
    for (int l = threadIdx.x; l < tile; l += kThreads) lds_st(&su[l * P], ldm<P>(U, ups, (long)c * tile + l));
    __syncthreads();
    const long r = (long)blockIdx.x * 64 + lane;
    const int q = (tile + 3) / 4;
    const int lb = wid * q, le = min(tile, lb + q);
    constexpr int NA = 2;
    Acc<P> acc[NA];
#pragma unroll
    for (int a = 0; a < NA; ++a) acc[a] = acc_zero<P>();
    auto sums = [&](auto edge) __attribute__((always_inline)) {
        int nt = 0;
        for (int l = lb; l < le; l += NA) {
            V<P> y[NA];
#pragma unroll
            for (int k = 0; k < NA; ++k) y[k] = (l + k < le) ? y_entry<P>(Y, lda, ps, r, l + k, h, tile) : zero<P>();
#pragma unroll
            for (int k = 0; k < NA; ++k)
                if (l + k < le && (!decltype(edge)::value || l + k <= r)) acc_fma(acc[k], y[k], lds_ld<P>(&su[(l + k) * P]));
            if ((++nt) % kLazy<P> == 0) {
#pragma unroll
                for (int a = 0; a < NA; ++a) acc[a] = acc_from(acc_get(acc[a]));
            }
        }
    };
    // beside the diagonal not with Y's zeros: U(l) may be NaN or Inf, and row r < l does not depend on it
    if ((int)blockIdx.x * 64 < le)
        sums(std::true_type{});
    else
        sums(std::false_type{});
    acc_add_acc(acc[0], acc[1]);
    lds_st(&sp[wid][lane * P], acc_get(acc[0]));
    __syncthreads();
    if (wid == 0 && r < h) {
        V<P> v = lds_ld<P>(&sp[0][lane * P]);
        for (int w = 1; w < 4; ++w) v = add(v, lds_ld<P>(&sp[w][lane * P]));
        stm(B, bps, (long)c * ldb + r, sub(ldm<P>(B, bps, (long)c * ldb + r), v));
    }
}

// The same three products, and the Gram block of a tile, for many columns: Out(i, c) =
// [Out(i, c) -] sum_k X(i, k) Z(k, c), a workgroup per block of 16 RB x 16 RB outputs, each thread
// RB x RB of them (rows i = tx + 16 a, columns c = ty + 16 b).  Chunks of 16 k of X and Z are staged
// in LDS, the next chunk's loads in flight during the current one's multiply-adds; a thread's
// multiply-adds take 2 P RB LDS words for RB^2 of them.  dd (12 instructions a multiply-add) needs
// RB = 2 to stay below the LDS rate, qd and od (108, 952) do not.  Sums are kept in two levels (64
// terms, then the sums), so that the error grows as slowly as in a wave's butterfly.
//   kTN    S = Y^T B          X(i, k) = Y(k, i)
//   kTT    U = T^T S          X(i, k) = T(k, i), k <= i
//   kTNo   U = T S            X(i, k) = T(i, k), k >= i
//   kNN    B -= Y U           X(i, k) = Y(i, k); not od
//   kGram  G = striu(Y^T Y)   as kTN with Z = Y; tile block blockIdx.z; not od
// A block skips the k where its X is zero.  In the chunks that hold zeros for some of its rows (kTT and kNN,
// k > i) the products with them are left out too: Z(k, c) may be NaN or Inf, on which row i does not depend.
// (kTN, kTNo and kGram need no such care: there a NaN Z(k, c) makes all of the product that follows NaN.)
// Bound by the FP64 instruction rate: qd, m = n = 1024,
// tile 128, all 1024 columns, 2.31 ms for the eight Y^T B, 2.17 for B -= Y U and 0.54 for T S, 72 to
// 77 % of that rate for the first two (one wave per (l, c), one thread per row and one thread per (i, c)
// before, 64 columns at a time: 4.66, 9.77 and 10.2 ms).
enum { kTN, kTT, kTNo, kNN, kGram };

struct GemmArgs {
    const double *X;  // Y (unit lower trapezoidal, h x tile) or T
    long ldx, psx;
    const double *Z;
    long ldz, psz;
    double *O;
    long ldo, pso;
    int h, tile, nc;
    long xstep, ostep;  // kGram: tile block t at X + t xstep (h - t tile rows), O + t ostep
    const int *skip;
};

template <int P>
constexpr int gemm_rb()
{
    return P <= 2 ? 2 : 1;
}

template <int P, int MODE>
__global__ __launch_bounds__(kThreads) void k_gemm(GemmArgs g)
{
    constexpr int RB = gemm_rb<P>(), BT = 16 * RB, KC = 16;
    constexpr int LD = BT * P + 2;  // doubles per staged k (the 2 keep the staging stores off one bank)
    __shared__ double sX[2][KC * LD];
    __shared__ double sZ[2][KC * LD];
    if (g.skip && *g.skip) return;
    const int tid = threadIdx.x, tx = tid % 16, ty = tid / 16;
    const int i0 = blockIdx.x * BT, c0 = blockIdx.y * BT;
    const double *X = g.X;
    double *O = g.O;
    int h = g.h;
    if constexpr (MODE == kGram) {
        X += (long)blockIdx.z * g.xstep;
        O += (long)blockIdx.z * g.ostep;
        h -= (int)blockIdx.z * g.tile;
    }
    const int mo = (MODE == kNN) ? h : g.tile;                 // rows of the output
    const int nc = (MODE == kGram) ? g.tile : g.nc;
    // the k with X(i, k) not zero for some i of the block
    int kb = 0, ke = (MODE == kTN || MODE == kGram) ? h : g.tile;
    if constexpr (MODE == kTN || MODE == kTNo) kb = i0;
    if constexpr (MODE == kGram) kb = (c0 > i0) ? c0 : i0;     // y_j is zero above row j
    if constexpr (MODE == kTT || MODE == kNN) ke = (i0 + BT < ke) ? i0 + BT : ke;
    if constexpr (MODE == kGram) {
        if (i0 >= c0 + BT) ke = kb;  // below the diagonal: zeros
    }
    auto xval = [&](int i, int k) __attribute__((always_inline)) {
        if constexpr (MODE == kTN || MODE == kGram) {
            return y_entry<P>(X, g.ldx, g.psx, k, i, h, g.tile);
        } else if constexpr (MODE == kNN) {
            return neg(y_entry<P>(X, g.ldx, g.psx, i, k, h, g.tile));
        } else if constexpr (MODE == kTT) {
            return (k <= i && i < g.tile) ? ldm<P>(X, g.psx, (long)i * g.ldx + k) : zero<P>();
        } else {
            return (k >= i && k < g.tile) ? ldm<P>(X, g.psx, (long)k * g.ldx + i) : zero<P>();
        }
    };
    auto zval = [&](int k, int c) __attribute__((always_inline)) {
        if constexpr (MODE == kGram) return y_entry<P>(X, g.ldx, g.psx, k, c, h, g.tile);
        return (k < ke && c < nc) ? ldm<P>(g.Z, g.psz, (long)c * g.ldz + k) : zero<P>();
    };
    // staging: X is contiguous along k for kTN, kTT and kGram, along i for kTNo and kNN; Z along k
    constexpr bool XK = MODE == kTN || MODE == kTT || MODE == kGram;
    V<P> xs[RB], zs[RB];
    auto fetch = [&](int k0) __attribute__((always_inline)) {
#pragma unroll
        for (int a = 0; a < RB; ++a) {
            xs[a] = XK ? xval(i0 + ty + 16 * a, k0 + tx) : xval(i0 + tx + 16 * a, k0 + ty);
            zs[a] = zval(k0 + tx, c0 + ty + 16 * a);
        }
    };
    auto stage = [&](int buf) __attribute__((always_inline)) {
#pragma unroll
        for (int a = 0; a < RB; ++a) {
            const int xi = (XK ? ty : tx) + 16 * a, xk = XK ? tx : ty;
            lds_st(&sX[buf][xk * LD + xi * P], xs[a]);
            lds_st(&sZ[buf][tx * LD + (ty + 16 * a) * P], zs[a]);
        }
    };
    Acc<P> acc[RB][RB], tot[RB][RB];
#pragma unroll
    for (int a = 0; a < RB; ++a)
#pragma unroll
        for (int b = 0; b < RB; ++b) {
            acc[a][b] = acc_zero<P>();
            const int i = i0 + tx + 16 * a, c = c0 + ty + 16 * b;
            tot[a][b] = acc_zero<P>();
            if (MODE == kNN && i < mo && c < nc) tot[a][b] = acc_from(ldm<P>(O, g.pso, (long)c * g.ldo + i));
        }
    if (kb < ke) {
        fetch(kb);
        stage(0);
    }
    __syncthreads();
    int nch = 0;
    for (int k0 = kb; k0 < ke; k0 += KC) {
        const int buf = nch & 1;
        const bool more = k0 + KC < ke;
        if (more) fetch(k0 + KC);
        auto chunk = [&](auto edge) __attribute__((always_inline)) {
#pragma unroll 1
            for (int k = 0; k < KC; ++k) {
                V<P> x[RB], z[RB];
#pragma unroll
                for (int a = 0; a < RB; ++a) {
                    x[a] = lds_ld<P>(&sX[buf][k * LD + (tx + 16 * a) * P]);
                    z[a] = lds_ld<P>(&sZ[buf][k * LD + (ty + 16 * a) * P]);
                }
#pragma unroll
                for (int a = 0; a < RB; ++a)
                    if (!decltype(edge)::value || k0 + k <= i0 + tx + 16 * a) {
#pragma unroll
                        for (int b = 0; b < RB; ++b) acc_fma(acc[a][b], x[a], z[b]);
                    }
                if constexpr (kLazy<P> < KC) {
                    if ((k + 1) % kLazy<P> == 0) {
#pragma unroll
                        for (int a = 0; a < RB; ++a)
#pragma unroll
                            for (int b = 0; b < RB; ++b) acc[a][b] = acc_from(acc_get(acc[a][b]));
                    }
                }
            }
        };
        // od in one form: the test is nothing beside its multiply-adds, and two forms take it to one wave per SIMD
        if ((MODE == kTT || MODE == kNN) && (P >= 8 || k0 + KC > i0 + 1))
            chunk(std::true_type{});
        else
            chunk(std::false_type{});
        ++nch;
        if (nch % 4 == 0 || !more) {
#pragma unroll
            for (int a = 0; a < RB; ++a)
#pragma unroll
                for (int b = 0; b < RB; ++b) {
                    acc_add(tot[a][b], acc_get(acc[a][b]));
                    tot[a][b] = acc_from(acc_get(tot[a][b]));
                    acc[a][b] = acc_zero<P>();
                }
        } else if (kLazy<P> >= KC && kLazy<P> < 64) {
#pragma unroll
            for (int a = 0; a < RB; ++a)
#pragma unroll
                for (int b = 0; b < RB; ++b) acc[a][b] = acc_from(acc_get(acc[a][b]));
        }
        if (more) stage(buf ^ 1);
        __syncthreads();
    }
#pragma unroll
    for (int a = 0; a < RB; ++a)
#pragma unroll
        for (int b = 0; b < RB; ++b) {
            const int i = i0 + tx + 16 * a, c = c0 + ty + 16 * b;
            if (i >= mo || c >= nc) continue;
            V<P> v = acc_get(tot[a][b]);
            if (MODE == kGram && i >= c) v = zero<P>();
            stm(O, g.pso, (long)c * g.ldo + i, v);
        }
}

namespace {
// B(i, c) = 1 if i == c else 0, for i < rows and c < cols (P planes, ld ldb)
__global__ void k_identity(double *B, long ldb, long bps, int rows, int cols, int P)
{
    const long r = (long)blockIdx.x * blockDim.x + threadIdx.x;
    const int c = blockIdx.y;
    if (r >= rows || c >= cols) return;
    for (int k = 0; k < P; ++k) B[k * bps + (long)c * ldb + r] = (k == 0 && r == c) ? 1.0 : 0.0;
}
}  // namespace

// ============================================================================ launch timing
// When timing is on (mdls_timing_enable), every launch is bracketed by two events on its
// stream and recorded with the kernel's name, precision and algorithmic md multiply-add
// count.  Defined in mdls_capi.hip.
bool timing_on();
void timing_begin(hipStream_t s, void **ev);
void timing_end(hipStream_t s, void *ev, const char *name, int P, double work);

// Side stream and events of the calling host thread on the current device, created by
// mdls_init (default priority); null when mdls_init has not run on this thread for this device,
// and then the trailing updates run on the caller's stream.
struct SideStream {
    hipStream_t q;
    hipEvent_t ev_panel, ev_wide[2];
};
SideStream *side_stream();

// Process-wide tuning (mdls_set_tuning); the defaults are compile-time constants and nothing is
// read from the environment.  Only panel_variant changes results (the panel's reduction order).
struct Tuning {
    int lookahead;         // 1: trailing updates concurrently on the side stream (when it exists)
    int panel_variant;     // 0: default panel shape, 1: the alternative shape (more rows per thread)
    int apply_grid_cap;    // > 0: workgroups of a concurrent trailing update; 0: the built-in rule
    int apply_wide_rows;   // od: trailing updates of at least this many rows take two workgroups per CU
    unsigned spin_limit;   // polls before a wait of one workgroup for another gives up
    int split_update;      // 1: the refined solve's factorisation forms Y^T C on the matrix cores
    int cpanel;            // complex QR panels: 0 a launch per column, 1 persistent, 2 the faster form of each (cqr_t)
};
Tuning tuning();
int apply_grid_cap(int P, int h);
// Workgroups of the panel kernel of precision P (current variant) that can be resident at once on
// the current device (occupancy x compute units); 0 if the device cannot be queried.
int panel_capacity(int P, int m);
// The same of the step kernel of precision P (P <= 4).
int step_capacity(int P);

#define MDLS_LAUNCH(NAME, PREC, WORK, KERNEL, GRID, BLOCK, STREAM, ...)                       \
    do {                                                                                     \
        void *ev_ = nullptr;                                                                 \
        const bool tm_ = timing_on();                                                        \
        if (tm_) timing_begin((STREAM), &ev_);                                               \
        hipLaunchKernelGGL(KERNEL, GRID, BLOCK, 0, STREAM, __VA_ARGS__);                     \
        if (tm_) timing_end((STREAM), ev_, (NAME), (PREC), (double)(WORK));                  \
    } while (0)

// the same with SHM bytes of dynamic LDS
#define MDLS_LAUNCH_SHM(NAME, PREC, WORK, KERNEL, GRID, BLOCK, SHM, STREAM, ...)              \
    do {                                                                                     \
        void *ev_ = nullptr;                                                                 \
        const bool tm_ = timing_on();                                                        \
        if (tm_) timing_begin((STREAM), &ev_);                                               \
        hipLaunchKernelGGL(KERNEL, GRID, BLOCK, (SHM), STREAM, __VA_ARGS__);                 \
        if (tm_) timing_end((STREAM), ev_, (NAME), (PREC), (double)(WORK));                  \
    } while (0)

// ============================================================================ host side
constexpr int kGMax = 256;  // most workgroups one panel launch may use
constexpr int kCUs = 256;   // compute units of an MI355X

template <int P>
struct Cfg;
template <>
struct Cfg<1> {
    static constexpr int W = 16, NCI = 16;
};
template <>
struct Cfg<2> {
    static constexpr int W = 16, NCI = 16;
};
template <>
struct Cfg<4> {
    static constexpr int W = 8, NCI = 8;
};
template <>
struct Cfg<8> {
    static constexpr int W = 8, NCI = 4;
};

inline int leaf_width(int P)
{
    switch (P) {
    case 1: return Cfg<1>::W;
    case 2: return Cfg<2>::W;
    case 4: return Cfg<4>::W;
    case 8: return Cfg<8>::W;
    }
    return 0;
}

inline size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

struct Layout {
    size_t beta, leafT, gpart, ctr, err, yw, apart, anu, big, total;
    int W, nleaves, acols;
};

inline Layout layout(int P, int m, int n, int tile)
{
    Layout L{};
    L.W = leaf_width(P);
    L.nleaves = (n + L.W - 1) / L.W;
    size_t off = 0;
    auto take = [&](size_t bytes) {
        size_t at = off;
        off += align256(bytes);
        return at;
    };
    L.beta = take(sizeof(double) * (size_t)P * n);
    L.leafT = take(sizeof(double) * (size_t)P * L.W * L.W * L.nleaves);
    L.gpart = take(sizeof(double) * 2 * kGMax * (L.W * L.W + 2 * L.W) * P);
    L.ctr = take(sizeof(unsigned) * (size_t)(L.nleaves + 1));
    L.err = take(sizeof(int) * 4);
    L.yw = take(sizeof(double) * (size_t)P * (m > n ? m : n));
    // trailing update: partial sums and -U of at most acols columns per launch
    L.acols = n + 1;
    L.apart = take(sizeof(double) * (size_t)P * L.W * L.acols * ((m + 63) / 64));
    L.anu = take(sizeof(double) * (size_t)P * L.W * L.acols);
    // back substitution inverses / Gram blocks (P x tile x n) or Q^T B scratch (2 x P x tile x 64)
    // tile inverses (P x tile x n), and for blocked inversion the 32 x 32 diagonal blocks' (P x 32 x n)
    const size_t big1 = sizeof(double) * (size_t)P * (tile + (tile >= 64 ? kInvNB : 0)) * n;
    const size_t big2 = sizeof(double) * 2 * (size_t)P * tile * 64;
    L.big = take(big1 > big2 ? big1 : big2);
    L.total = off;
    (void)m;
    return L;
}

inline bool valid_p(int p) { return p == 1 || p == 2 || p == 4 || p == 8; }
inline bool valid_tile(int t) { return t >= 1 && t <= 256; }

template <int P>
struct Ctx {
    char *ws;
    Layout L;
    hipStream_t s;
    // scratch of the split-limb trailing-update product (double double only), or null: then the
    // products Y^T C run on the vector units
    double *split = nullptr;
    double *beta() const { return (double *)(ws + L.beta); }
    double *leafT() const { return (double *)(ws + L.leafT); }
    double *gpart() const { return (double *)(ws + L.gpart); }
    unsigned *ctr() const { return (unsigned *)(ws + L.ctr); }
    int *err() const { return (int *)(ws + L.err); }
    double *yw() const { return (double *)(ws + L.yw); }
    double *apart() const { return (double *)(ws + L.apart); }
    double *anu() const { return (double *)(ws + L.anu); }
    double *big() const { return (double *)(ws + L.big); }
};

struct PanelCfg {
    int nt, r;
};

// Threads per workgroup and rows per thread of the panel kernel: variant 0 (default) or 1 (the
// alternative shape, for tests of the multi-workgroup path and for tuning).
inline PanelCfg panel_cfg(int P, int variant)
{
    switch (P) {
    case 1:
    case 2: return variant ? PanelCfg{512, 8} : PanelCfg{512, 2};
    case 4: return variant ? PanelCfg{256, 4} : PanelCfg{256, 1};
    default: return variant ? PanelCfg{256, 2} : PanelCfg{256, 1};
    }
}

// The shape an m-row factorisation uses: the tuning variant, except that octo-double panels of
// more than 1024 rows always hold two rows per thread (half the workgroups, which leaves more
// compute units to the concurrent trailing update; measured on the 2048 x 1024 solve).
inline int panel_variant_for(int P, int m) { return (tuning().panel_variant || (P >= 8 && m > 1024)) ? 1 : 0; }
inline PanelCfg panel_cfg_for(int P, int m) { return panel_cfg(P, panel_variant_for(P, m)); }

inline int panel_groups(int P, int m)
{
    const PanelCfg cf = panel_cfg_for(P, m);
    const int rows_per_wg = cf.nt / leaf_width(P) * cf.r;
    const int g = (m + rows_per_wg - 1) / rows_per_wg;
    return g < 1 ? 1 : g;
}

template <int P, int W>
void launch_panel(const PanelArgs &a, PanelCfg cf, hipStream_t s)
{
    double work = a.off ? 2.0 * (a.h + a.off) * a.off * a.wact : 0.0;  // the look-ahead update
    for (int j = 0; j < a.wact; ++j) work += (a.h - j - 1) + 2.0 * (a.wact - j - 1) * (a.h - j);
#define MDLS_PANEL_CASE(NT_, R_)                                                                       \
    if (cf.nt == NT_ && cf.r == R_) {                                                                 \
        MDLS_LAUNCH("k_panel", P, work, (k_panel<P, W, R_, NT_>), dim3(a.G), dim3(NT_), s, a);        \
        return;                                                                                       \
    }
    if constexpr (P <= 2) {
        MDLS_PANEL_CASE(512, 8)
        MDLS_PANEL_CASE(512, 2)
    } else if constexpr (P == 4) {
        MDLS_PANEL_CASE(256, 4)
        MDLS_PANEL_CASE(256, 1)
    } else {
        MDLS_PANEL_CASE(256, 1)
        MDLS_PANEL_CASE(256, 2)
    }
#undef MDLS_PANEL_CASE
}

// The factorisation step kernel takes the default panel shape of P <= 4 up to this many rows.  A wave
// of it updates whole columns, so beyond them the columns of a tall matrix, few and long, outlast the panel.
// k_panel and k_apply_s/t/u on two streams over k_step, in time, for n = 64, 256 and (up to 4096 rows) 1024: double
// 4096 rows 1.09, 1.14, 1.40, 6144 1.03, 1.11, 8192 0.96, 1.03; dd 3072 rows 1.07, 1.12, 1.27, 4096 0.97, 1.02, 1.29,
// 6144 0.84, 0.89; qd 1536 rows 1.04, 1.08, 1.06, 2048 0.96, 1.01, 0.99, 3072 0.79, 0.86, 1.06.
template <int P>
constexpr int step_rows()
{
    return P <= 2 ? 4096 : (P == 4 ? 2048 : 0);
}

// The last panel's update has no panel beside it and only B's columns: with more rows than this it goes to
// k_apply_s/t/u, whose units cut them up, in place of one or two waves a column.  Solves of one column, us, k_step /
// the three: double 1024 rows 39 / 39, 2048 43 / 40, 3000 53 / 36; dd 500 44 / 42, 768 50 / 40, 2048 64 / 42,
// 4096 98 / 46; qd 64 55 / 52, 256 65 / 54, 768 101 / 54, 2048 135 / 56.
template <int P>
constexpr int step_tail_rows()
{
    return P == 1 ? 1024 : (P == 2 ? 512 : 128);
}

constexpr long kStepLd = 1L << 24;  // the step kernel's byte offsets (16 columns of lda doubles) stay below 2^32

template <int P>
void launch_step(const StepArgs &a, int grid_cap, hipStream_t s)
{
    if constexpr (P <= 4) {
        constexpr int W = Cfg<P>::W, NT = P <= 2 ? 512 : 256, R = P <= 2 ? 2 : 1, NW = NT / 64;
        const PanelArgs &p = a.p;
        const ApplyArgs &u = a.a;
        double work = 0.0;
        if (p.G > 0) {
            work = p.off ? 2.0 * (p.h + p.off) * p.off * p.wact : 0.0;
            for (int j = 0; j < p.wact; ++j) work += (p.h - j - 1) + 2.0 * (p.wact - j - 1) * (p.h - j);
        }
        if (u.ncol > 0) work += (2.0 * u.h * u.wact + 0.5 * u.wact * (u.wact + 1)) * u.ncol;
        // two waves share a column of more than 1024 (dd) or 768 (qd) rows: alone a wave takes 67 us (dd)
        // or 100 us (qd) for 1024 rows of it, and the panel beside it 77 or 88; below, one wave has
        // half the staging.  Time with one wave over that with two, n = 64, 128, 512, 1024: dd 1024 rows 1.02, 1.01,
        // 1.00, 0.99, 1536 1.03, 1.02, 1.00, 1.00, 2048 1.08, 1.09, 1.04, 0.99; qd 768 rows 1.03, 1.01, 0.99 (n = 512), 1024
        // 1.11, 1.09, 1.01, 1.00, 2048 1.52, 1.55, 1.43, 1.14; double 0.99 to 1.01 throughout
        StepArgs b = a;
        b.a.rs = u.h > (P <= 2 ? 1024 : 768) ? 2 : 1;
        const int ncw = NW / b.a.rs;
        int nu = (u.ncol + ncw - 1) / ncw;
        if (grid_cap > 0 && nu > grid_cap) nu = grid_cap;
        if (p.G + nu > 0)
            MDLS_LAUNCH("k_step", P, work, (k_step<P, W, R, NT>), dim3(p.G + nu), dim3(NT), s, b);
    }
}

// Resident workgroups per CU of the step kernel (0 if the query fails).
template <int P>
int step_occupancy_t()
{
    int per_cu = 0;
    if constexpr (P <= 4) {
        constexpr int W = Cfg<P>::W, NT = P <= 2 ? 512 : 256, R = P <= 2 ? 2 : 1;
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, k_step<P, W, R, NT>, NT, 0) != hipSuccess) per_cu = 0;
    }
    return per_cu;
}

// Resident workgroups per CU of the panel kernel of shape cf (0 if the query fails).
template <int P>
int panel_occupancy_t(PanelCfg cf)
{
    constexpr int W = Cfg<P>::W;
    int per_cu = 0;
    hipError_t e = hipErrorInvalidValue;
#define MDLS_OCC_CASE(NT_, R_) \
    if (cf.nt == NT_ && cf.r == R_) e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, k_panel<P, W, R_, NT_>, NT_, 0);
    if constexpr (P <= 2) {
        MDLS_OCC_CASE(512, 8)
        MDLS_OCC_CASE(512, 2)
    } else if constexpr (P == 4) {
        MDLS_OCC_CASE(256, 4)
        MDLS_OCC_CASE(256, 1)
    } else {
        MDLS_OCC_CASE(256, 1)
        MDLS_OCC_CASE(256, 2)
    }
#undef MDLS_OCC_CASE
    return e == hipSuccess ? per_cu : 0;
}

// Householder QR of A (m x n) in narrow panels; B (nb columns, may be null) receives Q^T B.
// The trailing update (k_apply_s, k_apply_t, k_apply_u) in launches of at most L.acols
// columns.  Rows per unit: the largest of 256, 128, 64 that still gives two units per CU.
// Bytes of Ctx::split for factorisations of n columns: the panel's Householder block staged
// densely (2 planes of kSplitMaxRows x 16), the exact level sums and the column exponents.
inline size_t split_scratch_bytes(int n)
{
    return align256(sizeof(double) * 2 * (size_t)kSplitMaxRows * 16) + split_workspace_bytes(16, n + 1) + 256;
}

// The trailing update of a double-double panel with S = Y^T C formed exactly on the FP64 matrix
// cores (k_split_tn; the precision form's split-limb product), then -U = -T^T S and C -= Y U on
// the vector units as in launch_apply.
template <int P>
void launch_apply_split(const Ctx<P> &cx, ApplyArgs aa, int grid_cap, hipStream_t st)
{
    constexpr int W = Cfg<P>::W;
    static_assert(P == 2 && W <= 16, "split-limb products: double double, at most 16 columns of Y");
    double *Yd = cx.split;
    double *spart = Yd + 2L * kSplitMaxRows * 16;
    const size_t spart_bytes = align256(sizeof(double) * (size_t)((cx.L.acols + 15) / 16) * kSplitK * kSlices * 256);
    int *exps = (int *)((char *)spart + spart_bytes);
    MDLS_LAUNCH("k_stage_y", P, 0, k_stage_y, dim3((unsigned)(((long)aa.h * W + kThreads - 1) / kThreads)), dim3(kThreads),
                st, aa.Y, aa.ldy, aa.psy, aa.h, aa.wact, W, Yd);
    aa.part = cx.apart();
    aa.nu = cx.anu();
    for (int c0 = 0; c0 < aa.nc; c0 += cx.L.acols) {
        aa.c0 = c0;
        aa.ncol = (aa.nc - c0 < cx.L.acols) ? (aa.nc - c0) : cx.L.acols;
        SplitArgs sa{Yd, (long)aa.h, (long)aa.h * W, aa.C + (long)c0 * aa.ldc, aa.ldc, aa.psc, spart, exps, aa.h, W,
                     aa.ncol};
        const int tiles = (aa.ncol + 15) / 16;
        MDLS_LAUNCH("k_split_exp", P, 0, k_split_exp, dim3((W + aa.ncol + 3) / 4), dim3(kThreads), st, sa);
        MDLS_LAUNCH("k_split_tn", P, (double)aa.h * aa.wact * aa.ncol, k_split_tn, dim3(tiles, kSplitK),
                    dim3(64 * kSplitWaves), st, sa);
        MDLS_LAUNCH("k_split_fin", P, 0, k_split_fin_part, dim3(tiles), dim3(256), st, sa, aa.part);
        const int ncg = (aa.ncol + 3) / 4;
        ApplyArgs at = aa;
        at.rb = aa.h;
        at.nrb = 1;  // S is complete: one partial sum per column
        int tgrid = ncg;
        if (grid_cap > 0 && tgrid > grid_cap) tgrid = grid_cap;
        MDLS_LAUNCH("k_apply_t", P, 0.5 * aa.wact * (aa.wact + 1) * aa.ncol, (k_apply_t<P, W>), dim3(tgrid),
                    dim3(kThreads), st, at);
        int rb = rb_max<P, W>();
        while (rb > 64 && (long)ncg * ((aa.h + rb - 1) / rb) < 2L * kCUs) rb >>= 1;
        aa.rb = rb;
        aa.nrb = (aa.h + rb - 1) / rb;
        int grid = ncg * aa.nrb;
        if (grid_cap > 0 && grid > grid_cap) grid = grid_cap;
        MDLS_LAUNCH("k_apply_u", P, (double)aa.h * aa.wact * aa.ncol, (k_apply_u<P, W>), dim3(grid), dim3(kThreads), st,
                    aa);
    }
}

template <int P>
void launch_apply(const Ctx<P> &cx, ApplyArgs aa, int grid_cap, hipStream_t st)
{
    constexpr int W = Cfg<P>::W;
    if constexpr (P == 2) {
        if (cx.split && aa.nb == 0 && aa.h <= kSplitMaxRows) {
            launch_apply_split<P>(cx, aa, grid_cap, st);
            return;
        }
    }
    const int ntot = aa.nc + aa.nb;
    aa.part = cx.apart();
    aa.nu = cx.anu();
    for (int c0 = 0; c0 < ntot; c0 += cx.L.acols) {
        aa.c0 = c0;
        aa.ncol = (ntot - c0 < cx.L.acols) ? (ntot - c0) : cx.L.acols;
        const int ncg = (aa.ncol + 3) / 4;
        int rb = rb_max<P, W>();
        while (rb > 64 && (long)ncg * ((aa.h + rb - 1) / rb) < 2L * kCUs) rb >>= 1;
        aa.rb = rb;
        aa.nrb = (aa.h + rb - 1) / rb;
        int grid = ncg * aa.nrb, tgrid = ncg;
        if (grid_cap > 0 && grid > grid_cap) grid = grid_cap;
        if (grid_cap > 0 && tgrid > grid_cap) tgrid = grid_cap;
        const double half = (double)aa.h * aa.wact * aa.ncol;
        MDLS_LAUNCH("k_apply_s", P, half, (k_apply_s<P, W>), dim3(grid), dim3(kThreads), st, aa);
        MDLS_LAUNCH("k_apply_t", P, 0.5 * aa.wact * (aa.wact + 1) * aa.ncol, (k_apply_t<P, W>), dim3(tgrid),
                    dim3(kThreads), st, aa);
        MDLS_LAUNCH("k_apply_u", P, half, (k_apply_u<P, W>), dim3(grid), dim3(kThreads), st, aa);
    }
}

// Householder QR of A (m x n) in narrow panels of W columns; B (nb columns, may be null)
// receives Q^T B.  Panel l (l > 0) first applies panel l-1 to its own columns (off = W); apply(l) updates
// the columns from panel l+2 on, and B.
// Up to step_rows<P>() rows one k_step launch per panel does panel l and apply(l-1) side by side.
// Otherwise (od, taller matrices, the alternative panel shape, the split-limb products) apply(l) is
// k_apply_s, k_apply_t, k_apply_u, on a side stream concurrently with panel l+1 where mdls_init made
// one:
//   caller: panel(l) -> [wait apply(l-1)] -> panel(l+1) -> [wait apply(l)] -> panel(l+2) ...
//   side:   [wait panel(l)] -> apply(l) -> [wait panel(l+1)] -> apply(l+1) ...
// and its grid is capped so that CUs stay free for the panel's workgroups.
template <int P>
int qr_panels(const Ctx<P> &cx, int m, int n, double *A, long lda, long psa, double *B, long ldb, long psb, int nb)
{
    constexpr int W = Cfg<P>::W;
    const PanelCfg cf = panel_cfg_for(P, m);
    const int rows_per_wg = cf.nt / W * cf.r;
    const int nleaves = cx.L.nleaves;
    const Tuning tu = tuning();
    // the exchange words behind the look-ahead sums of kGMax workgroups
    static_assert(kGMax * W * W * P + tag_words<P, W>(kGMax) <= 2 * kGMax * (W * W + 2 * W) * P, "exchange area");
    unsigned long long *gtag = (unsigned long long *)(cx.gpart() + (size_t)kGMax * W * W * P);
    const int ntag = tag_words<P, W>(panel_groups(P, m));
    MDLS_LAUNCH("k_zero", P, 0, k_zero_sync, dim3((ntag + 255) / 256), dim3(256), cx.s, cx.ctr(), nleaves + 1, cx.err(),
                gtag, ntag);
    const long tps = (long)W * W * nleaves;
    // panel l's arguments
    auto panel_args = [&](int l) {
        const int c0 = l * W;
        const int off = (l > 0) ? W : 0;
        PanelArgs pa;
        pa.A = A + (long)c0 * lda + (c0 - off);
        pa.lda = lda;
        pa.ps = psa;
        pa.h = m - c0;
        pa.wact = (n - c0 < W) ? (n - c0) : W;
        pa.off = off;
        pa.Yp = off ? A + (long)(c0 - W) * lda + (c0 - W) : nullptr;
        pa.Tp = off ? cx.leafT() + (long)(l - 1) * W * W : nullptr;
        pa.beta = cx.beta() + c0;
        pa.bps = n;
        pa.T = cx.leafT() + (long)l * W * W;
        pa.tps = tps;
        pa.gpart = cx.gpart();
        pa.gbar = cx.ctr() + l;
        pa.gtag = gtag;
        pa.tag0 = (unsigned)c0;
        pa.err = cx.err();
        pa.spin = tu.spin_limit;
        pa.G = (pa.h + off + rows_per_wg - 1) / rows_per_wg;
        if (pa.G < 1) pa.G = 1;
        return pa;
    };
    // panel l applied to the columns right of panel l + 1, and to B
    auto apply_args = [&](int l) {
        const int c0 = l * W;
        const int wact = (n - c0 < W) ? (n - c0) : W;
        const int nc = n - c0 - wact;
        const int nn = (nc < W) ? nc : W;  // the next panel's columns: updated by panel l + 1 itself
        ApplyArgs aa{};
        aa.Y = A + (long)c0 * lda + c0;
        aa.ldy = lda;
        aa.psy = psa;
        aa.h = m - c0;
        aa.wact = wact;
        aa.T = cx.leafT() + (long)l * W * W;
        aa.tps = tps;
        aa.C = A + (long)(c0 + wact + nn) * lda + c0;
        aa.ldc = lda;
        aa.psc = psa;
        aa.nc = nc - nn;
        aa.B = B ? B + c0 : nullptr;
        aa.ldb = ldb;
        aa.psb = psb;
        aa.nb = B ? nb : 0;
        return aa;
    };
    if (m <= step_rows<P>() && lda <= kStepLd && !tu.panel_variant && !cx.split &&
        panel_groups(P, m) <= step_capacity(P)) {
        for (int l = 0; l <= nleaves; ++l) {
            StepArgs sa{};
            if (l < nleaves) sa.p = panel_args(l);
            if (l > 0) {
                sa.a = apply_args(l - 1);
                sa.a.ncol = sa.a.nc + sa.a.nb;
            }
            if (l == nleaves && sa.a.h > step_tail_rows<P>())
                launch_apply<P>(cx, sa.a, 0, cx.s);
            else
                launch_step<P>(sa, tu.apply_grid_cap, cx.s);
        }
        return 0;
    }
    SideStream *ss = (nleaves > 1 && tu.lookahead) ? side_stream() : nullptr;
    for (int l = 0; l < nleaves; ++l) {
        const PanelArgs pa = panel_args(l);
        if (ss && l >= 2 && hipStreamWaitEvent(cx.s, ss->ev_wide[l & 1], 0) != hipSuccess)  // apply(l-2)
            return MDLS_EHIP;
        launch_panel<P, W>(pa, cf, cx.s);

        const ApplyArgs aa = apply_args(l);
        if (ss) {
            if (hipEventRecord(ss->ev_panel, cx.s) != hipSuccess ||
                hipStreamWaitEvent(ss->q, ss->ev_panel, 0) != hipSuccess)
                return MDLS_EHIP;
            launch_apply<P>(cx, aa, apply_grid_cap(P, aa.h), ss->q);
            if (hipEventRecord(ss->ev_wide[l & 1], ss->q) != hipSuccess) return MDLS_EHIP;
        } else {
            launch_apply<P>(cx, aa, 0, cx.s);
        }
    }
    if (ss && (hipStreamWaitEvent(cx.s, ss->ev_wide[(nleaves - 1) & 1], 0) != hipSuccess ||
               (nleaves >= 2 && hipStreamWaitEvent(cx.s, ss->ev_wide[nleaves & 1], 0) != hipSuccess)))
        return MDLS_EHIP;
    return 0;
}

template <int P>
void invert_tiles(const Ctx<P> &cx, const InvArgs &ia, int ntiles)
{
    constexpr int NC = Cfg<P>::NCI;
    constexpr int RPT = 256 / (kThreads / NC);
    dim3 grid((ia.tile + NC - 1) / NC, ntiles);
    MDLS_LAUNCH("k_invert", P, (double)ntiles * ia.tile * ia.tile * ia.tile / 6.0, (k_invert<P, NC, RPT>), grid,
                dim3(kThreads), cx.s, ia);
}

// Stage 1 of the tiled back substitution (Algorithm 1): *d_info from R's diagonal, and the
// inverses of the n / tile diagonal tiles into Xinv (tile t at Xinv + t tile^2, ld tile, plane
// stride tile n).
template <int P>
void backsub_prep(const Ctx<P> &cx, int n, int tile, const double *R, long ldr, long psr, double *Xinv, int *d_info)
{
    const int N = n / tile;
    MDLS_LAUNCH("k_diag_check", P, 0, k_diag_check, dim3(1), dim3(kThreads), cx.s, R, ldr, psr, n, P, d_info);
    const long xips = (long)tile * n;
    InvArgs ia;
    ia.U = R;
    ia.ldu = ldr;
    ia.psu = psr;
    ia.ustride = (long)tile * (ldr + 1);
    ia.dsup = nullptr;
    ia.dps = 0;
    if (tile < 64 || tile % kInvNB != 0) {
        ia.X = Xinv;
        ia.ldx = tile;
        ia.psx = xips;
        ia.xstride = (long)tile * tile;
        ia.tile = tile;
        invert_tiles<P>(cx, ia, N);
        return;
    }
    // blocked: the 32 x 32 diagonal blocks first (into Xd, after the P planes of Xinv), then the
    // blocks above them by block rows
    double *Xd = Xinv + (long)P * xips;
    const long dps = (long)kInvNB * n;
    ia.ustride = (long)kInvNB * (ldr + 1);
    ia.X = Xd;
    ia.ldx = kInvNB;
    ia.psx = dps;
    ia.xstride = (long)kInvNB * kInvNB;
    ia.tile = kInvNB;
    invert_tiles<P>(cx, ia, n / kInvNB);
    InvBlkArgs ib;
    ib.U = R;
    ib.ldu = ldr;
    ib.psu = psr;
    ib.Xd = Xd;
    ib.dps = dps;
    ib.X = Xinv;
    ib.psx = xips;
    ib.tile = tile;
    ib.skip = nullptr;
    constexpr int NCB = inv_blk_cols<P>();
    const int nbt = tile / kInvNB;
    double work = 0.0;  // md multiply-adds: per block column K, sum over I < K of (K - I) + 1 blocks
    for (int K = 1; K < nbt; ++K) work += (double)(K * (K + 1) / 2 + K) * kInvNB * kInvNB * kInvNB;
    MDLS_LAUNCH("k_inv_blocks", P, work * N, (k_inv_blocks<P>), dim3(kInvNB / NCB, nbt - 1, N), dim3(kThreads), cx.s,
                ib);
}

// Stage 2 (Algorithm 1): for i = N-1 .. 0, x_i := U_i^-1 y_i, then y_j -= R_{j,i} x_i for every
// j < i; y (P planes of n) is overwritten.  Every kernel returns at once while *skip is set.
template <int P>
void backsub_sweep(const Ctx<P> &cx, int n, int tile, const double *R, long ldr, long psr, const double *Xinv,
                   double *y, double *x, long xps, const int *skip)
{
    const int N = n / tile;
    const long xips = (long)tile * n;
    const long yps = n;
    for (int i = N - 1; i >= 0; --i) {
        const long it = (long)i * tile;
        MDLS_LAUNCH("k_bs_xi", P, 0.5 * tile * tile, (k_bs_xi<P>), dim3((tile + 3) / 4), dim3(kThreads), cx.s,
                    Xinv + (long)i * tile * tile, (long)tile, xips, y + it, yps, x + it, xps, tile, skip);
        if (i > 0) {
            const int rows = i * tile;
            if (tile % (4 * kBsSlices) == 0) {
                // the update split over column slices; partial sums in the trailing-update scratch
                double *part = cx.apart();
                MDLS_LAUNCH("k_bs_upd", P, (double)rows * tile, (k_bs_upd_part<P>), dim3((rows + 63) / 64, kBsSlices),
                            dim3(kThreads), cx.s, R + it * ldr, ldr, psr, x + it, xps, part, (long)kBsSlices * rows,
                            rows, tile, skip);
                MDLS_LAUNCH("k_bs_comb", P, 0, (k_bs_comb<P>), dim3((rows + kThreads - 1) / kThreads), dim3(kThreads), cx.s,
                            part, (long)kBsSlices * rows, y, yps, rows, skip);
            } else {
                MDLS_LAUNCH("k_bs_upd", P, (double)rows * tile, (k_bs_upd<P>), dim3((rows + 63) / 64), dim3(kThreads),
                            cx.s, R + it * ldr, ldr, psr, x + it, xps, y, yps, rows, tile, skip);
            }
        }
    }
}

// More row blocks than this and k_trsv works ahead of the chain (AH = 2).  AH = 2 against AH = 0, us: double n = 704
// (22 blocks) 54 / 54, 1024 65 / 72; dd 640 89 / 85, 704 92 / 91, 768 95 / 96, 1024 107 / 124; qd 640 234 / 227, 704
// 243 / 242, 768 252 / 259, 1024 287 / 324; od 768 1089 / 980, 1024 1216 / 1147, 1280 (40 blocks) 1361 / 1358, 1408
// 1432 / 1471.
template <int P>
constexpr int trsv_ahead()
{
    return P <= 4 ? 22 : 40;
}

// Whether the back substitution runs by the caller's tiles (k_invert, k_inv_blocks, k_bs_*) and not in one launch.
// k_trsv inverts its block on one compute unit, 32 steps of up to four od multiply-adds a lane (qd 70, od 290 us
// alone), which the tile kernels spread over several and, for tiles below 32, shorten; they take 30 us a tile in
// return.  One launch / tiles, us: qd n = 8, 16, 24, 32 in one tile 33 / 31, 45 / 39, 56 / 49, 71 / 58, 64 with
// tile 32 79 / 76, tile 16 79 / 81; od one tile of 1, 8, 32 45 / 33, 84 / 70, 290 / 185; tile 8 n = 64 317 / 276,
// 128 373 / 501; tile 16 n = 128 372 / 329, 256 480 / 552; tile 32 n = 256 482 / 414, 1024 1147 / 1157, 1280 1358 /
// 1452; tile 48 n = 1152 1253 / 1075, 1440 1447 / 1274; tile 50 n = 500 680 / 804; tile 64 n = 192 425 / 425, 256 479 /
// 456, 1024 1147 / 871, 4096 3167 / 3050, 5120 3625 / 4019; tile 96 n = 960 1088 / 937, 3072 2387 / 2295; tile 128 n = 896
// 1031 / 1121, 1024 1147 / 1170 (1231 on the card that gave 1170), 2048 1872 / 1736, 2560 2089 / 2055, 3584 2702 / 2959.
template <int P>
constexpr bool backsub_by_tiles(int n, int tile)
{
    if (P < 4) return false;
    if (P == 4) return tile <= 32 && n <= 64 && (n == tile || (tile >= 8 && n <= 4 * tile));
    if (tile < 32) return n == tile || (tile >= 4 && n <= 8 * tile);
    if (tile <= 48) return n <= 26 * tile;
    return (tile == 64 || tile == 96 || tile == 128) && n >= tile * tile / 16 && n <= 262144 / tile;
}

// Back substitution R x = y (y: P planes yps apart, may be x).  In one launch: the words of x lie in the
// trailing update's partial sums.  *d_info: the first exactly zero R(k,k), -1 for a time-out.
template <int P>
void backsub_solve(const Ctx<P> &cx, int n, int tile, const double *R, long ldr, long psr, const double *y, long yps,
                   double *x, long xps, int *d_info, bool clear_err)
{
    if constexpr (P >= 4) {
        if (backsub_by_tiles<P>(n, tile)) {
            if (y != cx.yw())
                MDLS_LAUNCH("k_copy", P, 0, k_copy, dim3((n + 255) / 256), dim3(256), cx.s, y, yps, cx.yw(), (long)n, n, P);
            backsub_prep<P>(cx, n, tile, R, ldr, psr, cx.big(), d_info);
            backsub_sweep<P>(cx, n, tile, R, ldr, psr, cx.big(), cx.yw(), x, xps, nullptr);
            if (!clear_err) MDLS_LAUNCH("k_fold_err", P, 0, k_fold_err, dim3(1), dim3(64), cx.s, cx.err(), d_info);
            return;
        }
    }
    unsigned long long *xw = (unsigned long long *)cx.apart();
    const long nw = (long)P * n;
    const int nblk = (n + kTrB - 1) / kTrB;
    const int grid = (int)std::min<long>(256, (nw + kThreads - 1) / kThreads);
    MDLS_LAUNCH("k_trsv_init", P, 0, k_trsv_init, dim3(grid), dim3(kThreads), cx.s, xw, nw, cx.err(), clear_err ? 1 : 0, R,
                ldr, psr, n, P, d_info);
    const TrsvArgs ta{R, ldr, psr, y, yps, x, xps, xw, n, nblk, cx.err(), d_info, tuning().spin_limit};
    const double work = 0.5 * n * n + (double)nblk * kTrB * kTrB * kTrB / 6.0;
    if (nblk > trsv_ahead<P>())
        MDLS_LAUNCH("k_trsv", P, work, (k_trsv<P, 2>), dim3(nblk), dim3(kTrNT), cx.s, ta);
    else
        MDLS_LAUNCH("k_trsv", P, work, (k_trsv<P, 0>), dim3(nblk), dim3(kTrNT), cx.s, ta);
}

template <int P>
int solve_t(int m, int n, int tile, double *A, int lda, double *b, double *x, void *ws, int *d_info, hipStream_t s)
{
    Ctx<P> cx{(char *)ws, layout(P, m, n, tile), s};
    const long psa = (long)lda * n;
    if (qr_panels<P>(cx, m, n, A, lda, psa, b, m, m, 1) != 0) return MDLS_EHIP;
    // a workgroup of the back substitution reads its rows of y only and writes its rows of x, so y may be x;
    // where x lies over other elements of b (x == b with m > n), y is taken out first
    const double *y = b;
    long yps = m;
    if (x < b + (size_t)P * m && b < x + (size_t)P * n && !(x == b && (m == n || P == 1))) {
        MDLS_LAUNCH("k_copy", P, 0, k_copy, dim3((n + 255) / 256), dim3(256), s, b, (long)m, cx.yw(), (long)n, n, P);
        y = cx.yw();
        yps = n;
    }
    backsub_solve<P>(cx, n, tile, A, lda, psa, y, yps, x, n, d_info, false);
    return hipGetLastError() == hipSuccess ? 0 : MDLS_EHIP;
}

// Whether the tiles' Gram blocks are formed in blocks of sums (k_gemm) or a wave each (k_gram).  2048 rows, k_gram
// against k_gemm, one to eight tiles: dd 117-127 / 365 us at tile 32, 220-239 / 362 at 64, 386-469 / 363 at 128,
// 806-1138 / 370-425 at 256; qd 183-196 / 645, 345-418 / 650, 681-1156 / 653-898, 1256-3296 / 675-2429; od
// 633 / 4070, 1270-2101 / 4080, 2433-4103 / 4100-4425, 4639-7748 / 4272-7462.
constexpr bool gram_blocks(int P, int tile) { return P <= 4 && tile >= 96; }

template <int P>
int qr_impl(int m, int n, int tile, double *A, int lda, double *beta, double *T, int ldt, void *ws, int *d_info,
            hipStream_t s, double *split)
{
    Ctx<P> cx{(char *)ws, layout(P, m, n, tile), s};
    cx.split = split;
    const long psa = (long)lda * n;
    if (qr_panels<P>(cx, m, n, A, lda, psa, nullptr, 0, 0, 0) != 0) return MDLS_EHIP;
    if (beta)
        MDLS_LAUNCH("k_copy", P, 0, k_copy, dim3((n + 255) / 256), dim3(256), s, cx.beta(), (long)n, beta, (long)n, n,
                    P);
    if (d_info) MDLS_LAUNCH("k_set_info", P, 0, k_set_info, dim3(1), dim3(64), s, cx.err(), d_info);
    if (T) {
        const int N = n / tile;
        double *G = cx.big();
        const long gps = (long)tile * n;
        if constexpr (gram_blocks(P, 256)) {
            constexpr int BT = 16 * gemm_rb<P>();
            const int nb = (tile + BT - 1) / BT;
            const GemmArgs ga{A, (long)lda, psa, nullptr, 0, 0, G, (long)tile, gps, m, tile, tile, (long)tile * (lda + 1),
                              (long)tile * tile, nullptr};
            if (gram_blocks(P, tile))
                MDLS_LAUNCH("k_gram", P, 0, (k_gemm<P, kGram>), dim3(nb, nb, N), dim3(kThreads), s, ga);
        }
        if (!gram_blocks(P, tile))
            MDLS_LAUNCH("k_gram", P, 0, (k_gram<P>), dim3(tile, N), dim3(kThreads), s, A, (long)lda, psa, m, tile, G, gps);
        InvArgs ia;
        ia.U = G;
        ia.ldu = tile;
        ia.psu = gps;
        ia.ustride = (long)tile * tile;
        ia.dsup = cx.beta();
        ia.dps = n;
        ia.X = T;
        ia.ldx = ldt;
        ia.psx = (long)ldt * n;
        ia.xstride = (long)tile * ldt;
        ia.tile = tile;
        invert_tiles<P>(cx, ia, N);
    }
    return hipGetLastError() == hipSuccess ? 0 : MDLS_EHIP;
}

template <int P>
int qr_t(int m, int n, int tile, double *A, int lda, double *beta, double *T, int ldt, void *ws, int *d_info,
         hipStream_t s)
{
    return qr_impl<P>(m, n, tile, A, lda, beta, T, ldt, ws, d_info, s, nullptr);
}

// The double-double QR with its trailing-update products Y^T C on the matrix cores (split ->
// split_scratch_bytes(n) bytes); the refined solve's factorisation.
template <int P>
int qr_split_t(int m, int n, int tile, double *A, int lda, double *T, int ldt, void *ws, double *split, hipStream_t s)
{
    return qr_impl<P>(m, n, tile, A, lda, nullptr, T, ldt, ws, nullptr, s, split);
}

// The form of each of a tile block's three products.  A thread of k_gemm forms its outputs' whole sums, so a
// launch lasts as long as one sum while its blocks are fewer than the chip takes at once, and its waste is
// the part of the blocks that hold no output; a wave (k_tn, k_trmm_v, k_nn_sub_v) forms one output, or 64 rows of
// them, with the sum split, at more instructions per multiply-add (dd and double: up to three times, qd 1.2, od
// 1.05).  So k_gemm takes over from a number of full blocks on, whatever the length of the sums, where enough of
// them is output.  Measured for 16 to 2048 columns, tiles of 8 to 256 and 256 to 2048 rows, time of the wave
// form over k_gemm's with the blocks of the launch: Y^T B dd 0.5 at 32, 0.8 at 64, 1.4 at 128, 2.6 at 256;
// qd 0.7-1.1 at 128, 1.2 at 256; od 0.5-0.7 at 128, 1.0-1.2 at 256.  B -= Y U dd 0.8-1.0 at 128, 1.1-1.4 at
// 256; qd 0.8-1.1 at 256, 1.0-1.3 at 512; od 0.9-1.05 up to 4096: never k_gemm.  op(T) S, tile 32, 64, 128,
// 256: qd 1 at 16, 32, 64, 120 blocks; od 34, 64, 125, 200; dd 20, 30, 55, 90.  (k_gemm for every call of 16
// columns or more: dd 1000 x 32, tile 32, 16 columns 187 us and not 24, od 2150 and not 102.)
enum { kRowForm, kWaveForm, kBlockForm };

template <int P>
int gemm_or(double need, int rows, int nc, int else_form)
{
    constexpr int BT = 16 * gemm_rb<P>();
    constexpr double useful = P <= 2 ? 0.5 : (P == 4 ? 0.8 : 0.9);
    const double out = (double)rows * nc;
    const double full = out / (BT * BT), launched = (double)((rows + BT - 1) / BT) * ((nc + BT - 1) / BT);
    return full >= need && full >= useful * launched ? kBlockForm : else_form;
}

template <int P>
int tn_form(int tile, int nc)
{
    return gemm_or<P>(P <= 2 ? 96 : (P == 4 ? 192 : 256), tile, nc, kWaveForm);
}

template <int P>
int trmm_form(int tile, int nc)
{
    if (tile <= 4) return kRowForm;
    return gemm_or<P>(P <= 2 ? 16 + tile / 4 : (P == 4 ? std::max(12, tile / 2) : std::max(24, tile)), tile, nc, kWaveForm);
}

template <int P>
int nn_form(int h, int tile, int nc)
{
    constexpr int BT = 16 * gemm_rb<P>();
    if (tile <= 2 || (tile <= (P < 8 ? 8 : 16) && (double)h * nc >= 192.0 * BT * BT)) return kRowForm;
    return P < 8 ? gemm_or<P>(P <= 2 ? 160 : 256, h, nc, kWaveForm) : kWaveForm;
}

// One tile block on nc columns of B: S = Y^T B, U = op(T) S, B -= Y U (op(T) = T^T for Q^T, T for Q);
// h rows from the block's diagonal.
template <int P, bool TRANS>
void apply_block(const double *Y, long lda, long psa, int h, int tile, const double *Tk, long ldt, long tps, double *B,
                 long ldb, long bps, int nc, double *S, double *U, long sps, const int *skip, hipStream_t s)
{
    const double tri = 0.5 * tile * tile * nc, full = (double)h * tile * nc;
    constexpr int BT = 16 * gemm_rb<P>();
    const unsigned bt = (tile + BT - 1) / BT, bh = (h + BT - 1) / BT, bc = (nc + BT - 1) / BT;
    if (tn_form<P>(tile, nc) == kBlockForm) {
        const GemmArgs ga{Y, lda, psa, B, ldb, bps, S, (long)tile, sps, h, tile, nc, 0, 0, skip};
        MDLS_LAUNCH("k_tn", P, full, (k_gemm<P, kTN>), dim3(bt, bc), dim3(kThreads), s, ga);
    } else {
        MDLS_LAUNCH("k_tn", P, full, (k_tn<P>), dim3((tile + 3) / 4, nc), dim3(kThreads), s, Y, lda, psa, h, tile, B, ldb,
                    bps, nc, S, sps, skip);
    }
    switch (trmm_form<P>(tile, nc)) {
    case kBlockForm: {
        const GemmArgs ga{Tk, ldt, tps, S, (long)tile, sps, U, (long)tile, sps, h, tile, nc, 0, 0, skip};
        MDLS_LAUNCH("k_trmm", P, tri, (k_gemm<P, TRANS ? kTT : kTNo>), dim3(bt, bc), dim3(kThreads), s, ga);
        break;
    }
    case kRowForm:
        MDLS_LAUNCH("k_trmm", P, tri, (k_trmm<P, TRANS>), dim3((tile + kThreads - 1) / kThreads, nc), dim3(kThreads), s, Tk,
                    ldt, tps, S, sps, U, tile, nc, skip);
        break;
    default:
        MDLS_LAUNCH("k_trmm", P, tri, (k_trmm_v<P, TRANS>), dim3((tile + 3) / 4, nc), dim3(kThreads), s, Tk, ldt, tps, S,
                    sps, U, tile, nc, skip);
    }
    const int nf = nn_form<P>(h, tile, nc);
    if constexpr (P < 8) {
        if (nf == kBlockForm) {
            const GemmArgs ga{Y, lda, psa, U, (long)tile, sps, B, ldb, bps, h, tile, nc, 0, 0, skip};
            MDLS_LAUNCH("k_nn_sub", P, full, (k_gemm<P, kNN>), dim3(bh, bc), dim3(kThreads), s, ga);
            return;
        }
    }
    if (nf == kRowForm)
        MDLS_LAUNCH("k_nn_sub", P, full, (k_nn_sub<P>), dim3((h + kThreads - 1) / kThreads, nc), dim3(kThreads), s, Y, lda,
                    psa, h, tile, U, sps, B, ldb, bps, skip);
    else
        MDLS_LAUNCH("k_nn_sub", P, full, (k_nn_sub_v<P>), dim3((h + 63) / 64, nc), dim3(kThreads), s, Y, lda, psa, h, tile,
                    U, sps, B, ldb, bps, skip);
}

// B := Q^T B (TRANS: the tile blocks in order, B := (I - Y_k T_k^T Y_k^T) B) or B := Q B (the blocks
// in reverse, T untransposed; the paper forms Q itself, Algorithm 2: with B = I this is that Q), cols
// columns of B at a time; S and U are scratch of P tile cols doubles each.  Every kernel returns at
// once while *skip is set (skip may be null).
template <int P, bool TRANS>
void apply_blocks(int m, int n, int tile, const double *A, int lda, const double *T, int ldt, double *B, int ldb,
                  int nrhs, double *S, double *U, int cols, const int *skip, hipStream_t s)
{
    const long psa = (long)lda * n, tps = (long)ldt * n, bps = (long)ldb * nrhs;
    const long sps = (long)tile * cols;
    const int N = n / tile;
    for (int c0 = 0; c0 < nrhs; c0 += cols) {
        const int nc = (nrhs - c0 < cols) ? nrhs - c0 : cols;
        double *Bc = B + (long)c0 * ldb;
        for (int q = 0; q < N; ++q) {
            const long kt = (long)(TRANS ? q : N - 1 - q) * tile;
            apply_block<P, TRANS>(A + kt * lda + kt, (long)lda, psa, m - (int)kt, tile, T + kt * ldt, (long)ldt, tps,
                                  Bc + kt, (long)ldb, bps, nc, S, U, sps, skip, s);
        }
    }
}

// The same with S and U in the workspace: S in the trailing update's partial sums and U in the tile
// inverses' place where each holds 64 columns or more, else both in the latter, 64 columns each.
// The more columns a launch has, the more blocks of outputs: qd, m = n = 1024, 1024 columns in chunks
// of 64 leave 32 blocks for Y^T B.
template <int P, bool TRANS>
int apply_ws(int m, int n, int tile, const double *A, int lda, const double *T, int ldt, double *B, int ldb, int nrhs,
             void *ws, hipStream_t s)
{
    Ctx<P> cx{(char *)ws, layout(P, m, n, tile), s};
    const size_t col = sizeof(double) * P * tile;
    const size_t cols = std::min((cx.L.anu - cx.L.apart) / col, (cx.L.total - cx.L.big) / col);
    if (cols >= 64)
        apply_blocks<P, TRANS>(m, n, tile, A, lda, T, ldt, B, ldb, nrhs, cx.apart(), cx.big(),
                               (int)std::min(cols, (size_t)nrhs), nullptr, s);
    else
        apply_blocks<P, TRANS>(m, n, tile, A, lda, T, ldt, B, ldb, nrhs, cx.big(), cx.big() + (size_t)P * tile * 64, 64,
                               nullptr, s);
    return hipGetLastError() == hipSuccess ? 0 : MDLS_EHIP;
}

template <int P>
int apply_qt_t(int m, int n, int tile, const double *A, int lda, const double *T, int ldt, double *B, int ldb, int nrhs,
               void *ws, hipStream_t s)
{
    return apply_ws<P, true>(m, n, tile, A, lda, T, ldt, B, ldb, nrhs, ws, s);
}

template <int P>
int apply_q_t(int m, int n, int tile, const double *A, int lda, const double *T, int ldt, double *B, int ldb, int nrhs,
              void *ws, hipStream_t s)
{
    return apply_ws<P, false>(m, n, tile, A, lda, T, ldt, B, ldb, nrhs, ws, s);
}

// Q(:, 0:ncols) := the first ncols columns of Q (m x m orthogonal factor), ld ldq
template <int P>
int form_q_t(int m, int n, int tile, const double *A, int lda, const double *T, int ldt, double *Q, int ldq, int ncols,
             void *ws, hipStream_t s)
{
    const long qps = (long)ldq * ncols;
    MDLS_LAUNCH("k_identity", P, 0, k_identity, dim3((m + 255) / 256, ncols), dim3(256), s, Q, (long)ldq, qps, m, ncols,
                P);
    return apply_q_t<P>(m, n, tile, A, lda, T, ldt, Q, ldq, ncols, ws, s);
}

template <int P>
int form_w_t(int m, int n, int tile, const double *A, int lda, const double *T, int ldt, double *W, int ldw,
             hipStream_t s)
{
    MDLS_LAUNCH("k_form_w", P, 0, (k_form_w<P>), dim3((m + kThreads - 1) / kThreads, n), dim3(kThreads), s, A, (long)lda,
                       (long)lda * n, T, (long)ldt, (long)ldt * n, W, (long)ldw, (long)ldw * n, m, tile);
    return hipGetLastError() == hipSuccess ? 0 : MDLS_EHIP;
}

template <int P>
int backsub_t(int n, int tile, const double *R, int ldr, double *x, void *ws, int *d_info, hipStream_t s)
{
    Ctx<P> cx{(char *)ws, layout(P, n, n, tile), s};
    backsub_solve<P>(cx, n, tile, R, ldr, (long)ldr * n, x, n, x, n, d_info, true);
    return hipGetLastError() == hipSuccess ? 0 : MDLS_EHIP;
}

// ---------------------------------------------------------------- batched solves (host)
// Kernel variants (threads, panel width, rows per thread) tried by the autotuner; each holds
// kBatchRows rows per panel.
constexpr int kBatchVariants = 3;
constexpr int kBatchWMax = 16;

inline int batch_variants(int P) { return (P == 2 || P == 4) ? kBatchVariants : 0; }

struct BatchLayout {
    size_t plan, slots, nslots, ctr, tctr, xch, scratch, total;
    int maxgrid;
};

inline BatchLayout batch_layout(int P, int count)
{
    BatchLayout L{};
    size_t off = 0;
    auto take = [&](size_t bytes) {
        size_t at = off;
        off += align256(bytes);
        return at;
    };
    const size_t cnt = (size_t)(count > 0 ? count : 1);
    const size_t xchp = ((size_t)kBatchWMax * kBatchWMax + 2 * (size_t)kTeamMax * (kBatchWMax * kBatchWMax + 2 * kBatchWMax)) * P;
    L.maxgrid = 8 * kCUs;
    L.plan = take(sizeof(BatchDesc) * cnt);
    L.slots = take(sizeof(int) * cnt * kTeamMax);
    L.nslots = take(sizeof(int));
    L.ctr = take(sizeof(unsigned) * 64);  // [0] slot counter, [1] barrier time-out flag
    L.tctr = take(sizeof(unsigned) * cnt * kTeamCtrs);
    L.xch = take(sizeof(double) * cnt * xchp);
    L.scratch = take(sizeof(double) * (size_t)L.maxgrid * kBatchRows * P);
    L.total = off;
    return L;
}

// Predicted milliseconds of one m x n problem on a team of T workgroups (one per CU): a column's
// serial chain (longer where a team meets) plus the multiply-adds shared by the team.  The constants
// were fitted to single problems and to 256 and 512 equal ones of 64 x 64 to 512 x 512, T = 1 and 16, on MI355X
// (dd 512 x 512: 28.7 ms on one workgroup, 5.0 on 16; qd 128 and 14.9).  Predicted over measured on the present
// kernels, variant 1, T = 1, 2, 4, 8, 16, 16 x 16 to 512 x 512 and 512 x 64, 200 x 20, 384 x 300: a problem alone
// 0.81 to 1.28, a device full of equal ones 0.63 to 1.18 (tall problems and those below 64 x 64 on large teams
// take the longest); variants 0 and 2 take up to 60 and 150 % longer than variant 1.  (Constants fitted to the full
// device instead gave slower plans where it is not full: qd, 200 problems of up to 96 x 96 1292 -> 1414 us, dd, 16 of
// up to 512 x 512 4623 -> 4753, and the two large batches above within 1 %.)
struct BatchCost {
    double one, chain, shared;  // T = 1; T > 1: chain + shared / T
};

inline BatchCost batch_cost(int P, const BatchDesc &d)
{
    const double m = d.m, n = d.n;
    const double fmas = m * n * n - n * n * n / 3.0 + 2.0 * m * n + n * n / 2.0;
    const double shared = (P == 2 ? 0.30e-6 : 1.35e-6) * fmas;
    return BatchCost{(P == 2 ? 4.0e-3 : 14e-3) * n + shared, (P == 2 ? 6.3e-3 : 14e-3) * n, shared};
}

// Order and teams of a batch.  For a deadline D every problem gets the smallest team (at most
// kTeamMax workgroups) that is predicted to finish within D, the problems are listed longest first,
// and the list is played through on kCUs workgroups (the members of a team take consecutive slots,
// and the team starts with its last member).  Of a falling sequence of deadlines, from every problem
// alone to every problem on its largest team, the plan with the shortest predicted end is kept; the
// first one where no other ends 2.5 % earlier (the prediction is no better than that: qd, 64 problems of 16 x 16,
// predicted 2 % earlier in teams: 257 us in teams, 193 alone; dd, 64 of 128 x 128, predicted 3 %: 990 and 1061), and
// at once where none can: single workgroups
// balance, or no team ends before the longest problem alone.  A fixed cap on
// the workgroups in teams, in place of this, left the problems past the first eight of a batch of
// 160 on one workgroup each: qd, 160 problems of up to 512 x 512, 61.3 ms against 16.2 ms now; dd, 512
// problems, 15.3 against 9.6 ms.
// Teams may stand anywhere in the list: slots are taken in order, so at any time at most one team
// is incomplete, its waiting members are fewer than the resident workgroups, and every complete
// team finishes without waiting for a later slot.  The members that come first wait until a running
// problem ends, which the limit on the waits inside a team does not count (kTeamPolls).
// Returns the slot list (problem index in the sorted plan * kTeamMax + member).
inline std::vector<int> batch_schedule(int P, std::vector<BatchDesc> &plan)
{
    constexpr int kDeadlines = 16;
    const size_t cnt = plan.size();
    std::vector<int> team(cnt), best_team, order(cnt), best_order;
    std::vector<double> t(cnt);
    std::vector<BatchCost> cost(cnt);
    double hi = 0.0, lo = 0.0, area = 0.0, best = 0.0, alone = 0.0;
    for (size_t q = 0; q < cnt; ++q) {
        cost[q] = batch_cost(P, plan[q]);
        hi = std::max(hi, cost[q].one);
        lo = std::max(lo, cost[q].chain + cost[q].shared / kTeamMax);
        area += cost[q].one;
    }
    for (int k = 0; k < kDeadlines; ++k) {
        const double D = hi * std::pow(lo / hi, (double)k / (kDeadlines - 1));
        double busy = 0.0;
        for (size_t q = 0; q < cnt; ++q) {
            const BatchCost &c = cost[q];
            team[q] = 1;
            t[q] = c.one;
            if (c.one > D) {
                const double T = (D > c.chain) ? std::ceil(c.shared / (D - c.chain)) : (double)kTeamMax;
                team[q] = (int)std::min((double)kTeamMax, std::max(2.0, T));
                t[q] = c.chain + c.shared / team[q];
            }
            order[q] = (int)q;
            busy += t[q] * team[q];
        }
        // no plan ends before its workgroups' time is spent, and shorter deadlines only add to it
        if (k > 0 && busy >= best * kCUs) break;
        std::stable_sort(order.begin(), order.end(), [&](int x, int y) { return t[x] > t[y]; });
        // the workgroups' times at which they come free, earliest on top
        std::priority_queue<double, std::vector<double>, std::greater<double>> free_at;
        for (int w = 0; w < kCUs; ++w) free_at.push(0.0);
        double end = 0.0;
        for (int q : order) {
            double start = 0.0;
            for (int w = 0; w < team[q]; ++w) {
                start = free_at.top();
                free_at.pop();
            }
            for (int w = 0; w < team[q]; ++w) free_at.push(start + t[q]);
            end = std::max(end, start + t[q]);
            if (k > 0 && end >= best) break;  // no better than the plan kept so far
        }
        if (k == 0) alone = end;
        if (k == 0 || (end < best && end < 0.975 * alone)) {
            best = end;
            best_team = team;
            best_order = order;
        }
        if (k == 0 && std::max(area / kCUs, lo) >= 0.975 * alone) break;
    }
    std::vector<BatchDesc> sorted;
    std::vector<int> slots;
    sorted.reserve(cnt);
    for (size_t q = 0; q < cnt; ++q) {
        sorted.push_back(plan[best_order[q]]);
        sorted.back().team = best_team[best_order[q]];
        for (int w = 0; w < sorted.back().team; ++w) slots.push_back((int)q * kTeamMax + w);
    }
    plan.swap(sorted);
    return slots;
}

template <int P, int W, int R, int NT>
int launch_batch(BatchArgs a, int count, int maxgrid, hipStream_t s)
{
    int per_cu = 0, cus = 0, dev = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, k_batch<P, W, R, NT>, NT, 0) != hipSuccess || per_cu < 1)
        per_cu = 1;
    if (hipGetDevice(&dev) != hipSuccess || hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) !=
                                                hipSuccess || cus < 1)
        cus = kCUs;
    // every workgroup of the grid is resident at once, so the members of every team meet
    int grid = per_cu * cus;
    if (grid > maxgrid) grid = maxgrid;
    if (grid > count * kTeamMax) grid = count * kTeamMax;
    const int nz = count * kTeamCtrs;
    MDLS_LAUNCH("k_zero", P, 0, k_zero_u32, dim3(1), dim3(64), s, a.counter, 64);
    MDLS_LAUNCH("k_zero", P, 0, k_zero_u32, dim3((nz + 255) / 256), dim3(256), s, a.tctr, nz);
    MDLS_LAUNCH("k_batch", P, 0, (k_batch<P, W, R, NT>), dim3(grid), dim3(NT), s, a);
    return hipGetLastError() == hipSuccess ? 0 : MDLS_EHIP;
}

template <int P>
int batch_solve_t(int count, double *A, double *b, double *x, int variant, void *ws, int *d_info, long long *d_times,
                  hipStream_t s)
{
    const BatchLayout L = batch_layout(P, count);
    char *w = (char *)ws;
    BatchArgs a;
    a.desc = (const BatchDesc *)(w + L.plan);
    a.slots = (const int *)(w + L.slots);
    a.nslots = (const int *)(w + L.nslots);
    a.A = A;
    a.b = b;
    a.x = x;
    a.scratch = (double *)(w + L.scratch);
    a.counter = (unsigned *)(w + L.ctr);
    a.err = (int *)(w + L.ctr) + 1;
    a.spin = tuning().spin_limit;
    a.tctr = (unsigned *)(w + L.tctr);
    a.xch = (double *)(w + L.xch);
    a.info = d_info;
    a.times = d_times;
    if constexpr (P == 2) {
        switch (variant) {
        case 0: return launch_batch<2, 8, 16, 256>(a, count, L.maxgrid, s);
        case 1: return launch_batch<2, 8, 8, 512>(a, count, L.maxgrid, s);
        case 2: return launch_batch<2, 4, 8, 256>(a, count, L.maxgrid, s);
        }
    } else if constexpr (P == 4) {
        switch (variant) {
        case 0: return launch_batch<4, 4, 8, 256>(a, count, L.maxgrid, s);
        case 1: return launch_batch<4, 4, 4, 512>(a, count, L.maxgrid, s);
        case 2: return launch_batch<4, 8, 16, 256>(a, count, L.maxgrid, s);
        }
    }
    return MDLS_EUNSUPPORTED;
}

#define MDLS_BATCH_FOR_PRECISION(X, P) \
    X template int batch_solve_t<P>(int, double *, double *, double *, int, void *, int *, long long *, hipStream_t);

// ---------------------------------------------------------------- refined solve (host)
// Least squares to PX limbs from a double-double factorisation: F := A, QR of F in dd (with
// the tile T factors), the inverses of R's diagonal tiles (once), then at most `iters` steps,
// stopping on the device once the correction norms show convergence (k_refine_check; the
// remaining steps' kernels return at once, so the call stays asynchronous).
//  * m == n (a square system is consistent): x := 0, r := b; each step d := R^-1 (Q^T r) in dd
//    (r rounded to dd), x += d, r := b - A x in PX limbs.
//  * m > n: refinement of the augmented system [I A; A^T 0][r; x] = [b; 0] (Bjorck 1967), which
//    refines the residual with x, so that a nonzero residual does not limit the accuracy:
//    x := 0, r := 0; each step f := b - r - A x and g := -A^T r in PX limbs, rounded to dd;
//    h := R^-T g (forward substitution with the transposed tile inverses), d := Q^T f,
//    dx := R^-1 (d(0:n) - h), dr := Q [h; d(n:m)], x += dx, r += dr.
// Converges when kappa(A) 2^-105 << 1; norms[2 it], norms[2 it + 1] receive max |dx| and max |x|
// of step it, -1 for steps not taken.
inline size_t refine_extra_bytes(int px, int m, int n, int tile)
{
    const size_t nch = (size_t)(n + kResidCols - 1) / kResidCols;
    return sizeof(double) * (2 * (size_t)n * tile + 2 * (size_t)px * m + 2 * (size_t)m + 6 * (size_t)n +
                             nch * px * m + 4 * (size_t)tile * 64) +
           10 * 256 + split_scratch_bytes(n);
}

template <int PX>
int refine_t(int m, int n, int tile, const double *A, int lda, const double *b, double *x, int iters, double *F,
             void *ws, int *d_info, double *norms, hipStream_t s)
{
    const Layout L = layout(2, m, n, tile);
    Ctx<2> cx{(char *)ws, L, s};
    char *e = (char *)ws + align256(L.total);
    auto take = [&](size_t bytes) {
        char *p = e;
        e += align256(bytes);
        return p;
    };
    const int nch = (n + kResidCols - 1) / kResidCols;
    const bool aug = m > n;
    double *T = (double *)take(sizeof(double) * 2 * (size_t)n * tile);
    double *r = (double *)take(sizeof(double) * (size_t)PX * m);    // residual b - A x, or f
    double *rr = (double *)take(sizeof(double) * (size_t)PX * m);   // augmented form: the residual iterate
    double *rdd = (double *)take(sizeof(double) * 2 * (size_t)m);
    double *dd = (double *)take(sizeof(double) * 2 * (size_t)n);
    double *gdd = (double *)take(sizeof(double) * 2 * (size_t)n);
    double *hdd = (double *)take(sizeof(double) * 2 * (size_t)n);
    double *part = (double *)take(sizeof(double) * (size_t)nch * PX * m);
    double *S = (double *)take(sizeof(double) * 4 * (size_t)tile * 64);
    int *done = (int *)take(sizeof(int) * 4);
    double *split = (double *)take(split_scratch_bytes(n));
    double *U = S + 2 * (size_t)tile * 64;
    const long psa = (long)lda * n;
    const int N = n / tile;
    MDLS_LAUNCH("k_copy", PX, 0, k_copy, dim3((unsigned)((psa + 255) / 256)), dim3(256), s, A, psa, F, psa, (int)psa, 2);
    MDLS_LAUNCH("k_copy", PX, 0, k_copy, dim3((m + 255) / 256), dim3(256), s, b, (long)m, r, (long)m, m, PX);
    MDLS_LAUNCH("k_zero", PX, 0, k_zero_f64, dim3((PX * n + 255) / 256), dim3(256), s, x, (long)PX * n);
    if (aug) {
        MDLS_LAUNCH("k_zero", PX, 0, k_zero_f64, dim3((PX * m + 255) / 256), dim3(256), s, rr, (long)PX * m);
        MDLS_LAUNCH("k_zero", PX, 0, k_zero_f64, dim3((2 * n + 255) / 256), dim3(256), s, gdd, 2L * n);
    }
    MDLS_LAUNCH("k_refine_init", PX, 0, k_refine_init, dim3((2 * iters + 255) / 256), dim3(256), s, norms, iters, done);
    // with MDLS_TUNE_SPLIT_UPDATE the factorisation's trailing-update products Y^T C run on the
    // FP64 matrix cores (split limbs); by default on the vector units
    int rc = qr_split_t<2>(m, n, tile, F, lda, T, tile, ws, tuning().split_update ? split : nullptr, s);
    if (rc != 0) return rc;
    double *Xinv = cx.big();
    const long xips = (long)tile * n;
    backsub_prep<2>(cx, n, tile, F, lda, psa, Xinv, d_info);
    for (int it = 0; it < iters; ++it) {
        if (it > 0) {
            // r := b - A x (square), f := b - r - A x and g := -A^T r (augmented), in PX limbs
            MDLS_LAUNCH("k_resid_part", PX, (double)m * n, (k_resid_part<2, PX>), dim3((m + kThreads - 1) / kThreads, nch),
                        dim3(kThreads), s, A, (long)lda, psa, m, n, x, (long)n, part, done);
            MDLS_LAUNCH("k_resid_fin", PX, 0, (k_resid_fin<PX>), dim3((m + kThreads - 1) / kThreads), dim3(kThreads), s, b,
                        (long)m, aug ? rr : nullptr, (long)m, part, m, nch, r, (long)m, done);
            if (aug)
                MDLS_LAUNCH("k_resid_t", PX, (double)m * n, (k_resid_t<2, PX, 2>), dim3((n + 3) / 4), dim3(kThreads), s, A,
                            (long)lda, psa, m, n, rr, (long)m, gdd, (long)n, done);
        }
        MDLS_LAUNCH("k_copy", PX, 0, k_copy_if, dim3((m + 255) / 256), dim3(256), s, r, (long)m, rdd, (long)m, m, 2, done);
        if (aug) {
            // h := R^-T g: for each tile from the top, h_i = Xinv_i^T g_i, then g_j -= R_ij^T h_i
            for (int i = 0; i < N; ++i) {
                const long it0 = (long)i * tile;
                MDLS_LAUNCH("k_bs_xi_t", PX, 0.5 * tile * tile, (k_bs_xi_t<2>), dim3((tile + 3) / 4), dim3(kThreads), s,
                            Xinv + (long)i * tile * tile, (long)tile, xips, gdd + it0, (long)n, hdd + it0, (long)n, tile,
                            done);
                const int rest = n - (int)it0 - tile;
                if (rest > 0)
                    MDLS_LAUNCH("k_bs_upd_t", PX, (double)rest * tile, (k_bs_upd_t<2>), dim3((rest + 3) / 4),
                                dim3(kThreads), s, F + (it0 + tile) * lda + it0, (long)lda, psa, hdd + it0, (long)n,
                                gdd + it0 + tile, (long)n, rest, tile, done);
            }
        }
        apply_blocks<2, true>(m, n, tile, F, lda, T, tile, rdd, m, 1, S, U, 1, done, s);
        if (aug)
            MDLS_LAUNCH("k_aug_split", PX, 0, (k_aug_split<2>), dim3((n + kThreads - 1) / kThreads), dim3(kThreads), s,
                        rdd, (long)m, hdd, (long)n, cx.yw(), (long)n, n, done);
        else
            MDLS_LAUNCH("k_copy", PX, 0, k_copy_if, dim3((n + 255) / 256), dim3(256), s, rdd, (long)m, cx.yw(), (long)n,
                        n, 2, done);
        backsub_sweep<2>(cx, n, tile, F, lda, psa, Xinv, cx.yw(), dd, n, done);
        MDLS_LAUNCH("k_refine_add", PX, 0, (k_refine_add<PX, 2>), dim3((n + kThreads - 1) / kThreads), dim3(kThreads), s,
                    x, (long)n, dd, (long)n, n, (unsigned long long *)(norms + 2 * it), done);
        if (aug) {
            apply_blocks<2, false>(m, n, tile, F, lda, T, tile, rdd, m, 1, S, U, 1, done, s);
            MDLS_LAUNCH("k_md_add", PX, 0, (k_md_add<PX, 2>), dim3((m + kThreads - 1) / kThreads), dim3(kThreads), s, rr,
                        (long)m, rdd, (long)m, m, done);
        }
        MDLS_LAUNCH("k_refine_check", PX, 0, (k_refine_check<PX>), dim3(1), dim3(64), s, it, iters, norms, done);
    }
    MDLS_LAUNCH("k_fold_err", PX, 0, k_fold_err, dim3(1), dim3(64), s, cx.err(), d_info);
    return hipGetLastError() == hipSuccess ? 0 : MDLS_EHIP;
}

#define MDLS_REFINE_FOR_PRECISION(X, P) \
    X template int refine_t<P>(int, int, int, const double *, int, const double *, double *, int, double *, void *, \
                               int *, double *, hipStream_t);

#define MDLS_FOR_PRECISION(X, P)                                                                        \
    X template int solve_t<P>(int, int, int, double *, int, double *, double *, void *, int *, hipStream_t);     \
    X template int qr_t<P>(int, int, int, double *, int, double *, double *, int, void *, int *, hipStream_t); \
    X template int qr_split_t<P>(int, int, int, double *, int, double *, int, void *, double *, hipStream_t); \
    X template int apply_qt_t<P>(int, int, int, const double *, int, const double *, int, double *, int, int,   \
                                 void *, hipStream_t);                                                         \
    X template int form_w_t<P>(int, int, int, const double *, int, const double *, int, double *, int,         \
                               hipStream_t);                                                                   \
    X template int backsub_t<P>(int, int, const double *, int, double *, void *, int *, hipStream_t);          \
    X template int apply_q_t<P>(int, int, int, const double *, int, const double *, int, double *, int, int,    \
                                void *, hipStream_t);                                                          \
    X template int form_q_t<P>(int, int, int, const double *, int, const double *, int, double *, int, int,     \
                               void *, hipStream_t);                                                          \
    X template int panel_occupancy_t<P>(PanelCfg);                                                         \
    X template int step_occupancy_t<P>();

}  // namespace mdls_impl
