// The differentiable unrolled map x_K(c, b) and its hand-written adjoint.
//
// Forward: exactly K PDHG iterations per instance from (0, 0), with the same
// scaling, step and restart rule as the solve but no termination test.  The
// restart iterations and the (tau, sigma) of every epoch are recorded on a
// tape, together with a checkpoint of the state (x, y, x0, y0, k, epoch)
// every `ckpt` iterations.  x_K is the projected primal point of iteration K,
// unscaled.  The schedule and the steps are constants of the map (they are not
// differentiated), so x_K is piecewise linear in (c, b).
//
// Backward: for each checkpoint segment, last to first, the segment is
// recomputed from its checkpoint (bitwise identical to the forward pass),
// keeping the projection masks 1[x - tau g > 0] as one bit per column
// (wavefront ballots) plus k, tau and sigma of every iteration; then the
// segment is swept backwards.  One reverse step is the transpose of the
// iteration's linearisation:
//   Halpern / restart:  adjoints of x_hat, y_hat from the adjoints of the new
//                       state and anchor (a restart sends both to x_hat, y_hat)
//   dual step:          lam_y += lam_yhat, lam_b~ += sigma lam_yhat,
//                       lam_xbar = -sigma A~^T lam_yhat
//   extrapolation:      lam_xhat += 2 lam_xbar, lam_x -= lam_xbar
//   projection:         lam_v = mask * lam_xhat
//   primal step:        lam_x += lam_v, lam_g = -tau lam_v, lam_c~ += lam_g,
//                       lam_y -= A~ lam_g
// with the seed D_c * grad(x_K) on the last x_hat.  dL/dc = D_c lam_c~ and
// dL/db = D_r lam_b~.  Both passes run one workgroup per instance in one
// persistent launch, with the two gathered vectors in LDS and, between the
// iterations that checkpoint or may restart, the matrices and the state in
// the threads' registers as in the batched solve: an iteration is bound by the
// latency of its gathers and two barriers (the reverse sweep: three).
// Measured at 256 instances of 500 x 1,500, 5 entries a column, FP32, K = 400:
// with 256 threads reading the matrices and the state from L2, 4.9 ms forward
// and 9.3 ms backward; so, 0.80 (set-up) + 1.72 and 3.50 ms.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstring>
#include <numeric>
#include <vector>

#include "common.h"
#include "inst_common.h"
#include "plain.h"

namespace mip {

template <typename T, typename V>
struct UArgs {
    int32_t B, K, ckpt, E, nseg, nep, W;
    int32_t lds, replay;  // lds: bytes of dynamic LDS per workgroup
    int32_t N, Mrows;
    const int32_t *row_off, *col_off, *word_off;
    InstMat M;
    // tape: scaling, scaled values, schedule, checkpoints; the instance
    // vectors, masks and checkpoints by position (see Side)
    double *d_row, *d_col, *pu, *pav;
    InstStore<V> S;
    int32_t* levels;  // per instance: the matrices' layout
    T *bt, *ct;
    double *eta, *omega0, *taus, *sigmas;
    int8_t* restart;
    T *cp_x, *cp_x0, *cp_y, *cp_y0;
    int32_t *cp_k, *cp_ep;
    // working state
    T *x, *x0, *y0, *xhat, *yhat;
    // backward
    uint64_t* masks;
    int32_t* kbuf;
    double *tbuf, *sbuf;
    T *lx, *lx0, *ly, *ly0;
    double *lct, *lbt;
    const double* gx;
    double *xK, *gc, *gb;
    int32_t* counter;
    double step_safety, rho, beta_suff, beta_nec, beta_art, theta;
    int32_t ruiz, pc, power_iters, halpern, restarts;
};

// One forward iteration of instance I (number i) with step (tau, sig) and
// Halpern weight from k.  want_q: the sums' entries x - x^, x^ - x0 (by column)
// and y - y^, y^ - y0 (by row) go to pu, xK and pav, lbt; keep_hat: x^, y^ are
// kept; last: x_K is written; maskrow (or NULL): the projection masks.
template <typename T, typename V, typename Acc, int BS, bool LONG>
__device__ __forceinline__ void u_iterate(const UArgs<T, V>& a, const Inst<T, V>& I, const unsigned char* lds, int64_t k,
                                          double tau, double sig, bool want_q, bool keep_hat, bool last,
                                          uint64_t* maskrow) {
    typedef RegShape<V> RS;
    const int tid = opaque(threadIdx.x);
    const int n = I.n, m = I.m, c0 = I.c0, r0 = I.r0;
    const double w = a.halpern ? (double)(k + 1) / (double)(k + 2) : 1.0;
    const double omw = 1.0 - w, rho = a.rho, opr = 1.0 + a.rho;
    for (int p = tid; p < n; p += BS) {
        const int g = c0 + p;
        const double o = (double)a.x[g], an = (double)a.x0[g], ctg = (double)a.ct[g];
        const Acc s = side_dot<LONG, Acc>(I.AT, lds, I.yl, p, RS::RC * BS, RS::KC);
        const double v = o - tau * (ctg - (double)s);
        const double hh = v < 0.0 ? 0.0 : v;
        if (maskrow) {
            const unsigned long long bits = __ballot(v > 0.0);
            if ((tid & (kWave - 1)) == 0) maskrow[p >> 6] = bits;
        }
        I.xl[p] = (T)(2.0 * hh - o);
        a.x[g] = (T)(w * (opr * hh - rho * o) + omw * an);
        if (want_q || last) {
            const int j = I.column(p);
            if (last) a.xK[j] = a.d_col[j] * hh;
            if (want_q) {
                a.pu[j] = o - hh;
                a.xK[j] = hh - an;  // (the last iteration wants no sums)
            }
        }
        if (keep_hat) a.xhat[g] = (T)hh;
    }
    __syncthreads();
    for (int p = tid; p < m; p += BS) {
        const int g = r0 + p;
        const double an = (double)a.y0[g], btg = (double)a.bt[g];
        const Acc s = side_dot<LONG, Acc>(I.A, lds, I.xl, p, RS::RR * BS, RS::KR);
        const double o = (double)I.yl[p];
        const double hh = o + sig * (btg - (double)s);
        I.yl[p] = (T)(w * (opr * hh - rho * o) + omw * an);
        if (want_q) {
            const int i = I.row(p);
            a.pav[i] = o - hh;
            a.lbt[i] = hh - an;
        }
        if (keep_hat) a.yhat[g] = (T)hh;
    }
    __syncthreads();
}

// `count` such iterations with none of these extras (but the masks, W words
// from one iteration's to the next), from iteration k of the epoch on: the
// threads' rows and their vectors' entries stay in registers.
template <typename T, typename V, typename Acc, int BS, bool LONG>
__device__ __forceinline__ void u_plain(const UArgs<T, V>& a, const Inst<T, V>& I, const unsigned char* lds, int count,
                                        int64_t k, double tau, double sig, uint64_t* maskrow) {
    typedef RegShape<V> RS;
    const int tid = opaque(threadIdx.x);
    const int m = I.m, n = I.n, c0 = I.c0, r0 = I.r0, W = a.W;
    T *const yL = I.yl, *const xbL = I.xl;
    const double rho = a.rho, opr = 1.0 + a.rho;
    RegSide<V, RS::RC, RS::KC, LONG> gt;
    RegSide<V, RS::RR, RS::KR, LONG> ga;
    reg_load<BS, T>(gt, I.AT, lds, n, m);
    reg_load<BS, T>(ga, I.A, lds, m, n);
    T xr[RS::RC], x0r[RS::RC], ctr[RS::RC], y0r[RS::RR], btr[RS::RR];
#pragma unroll
    for (int r = 0; r < RS::RC; ++r) {
        const int g = c0 + min(tid + r * BS, n - 1);
        xr[r] = a.x[g];
        x0r[r] = a.x0[g];
        ctr[r] = a.ct[g];
    }
#pragma unroll
    for (int r = 0; r < RS::RR; ++r) {
        const int g = r0 + min(tid + r * BS, m - 1);
        y0r[r] = a.y0[g];
        btr[r] = a.bt[g];
    }
    double wl = 1.0;  // lane l: the Halpern weight of iteration l of each 64
    for (int it = 0; it < count; ++it) {
        if (a.halpern && (it & (kWave - 1)) == 0) {
            const double kl = (double)(k + it + (tid & (kWave - 1)));
            wl = (kl + 1.0) / (kl + 2.0);
        }
        const double w = lane_value(wl, it & (kWave - 1)), omw = 1.0 - w;
        gt.pin();
        ga.pin();
        inst_rows<BS, RS::RC, Acc>(I.levels, n, gt, I.AT, lds, yL, [&](int p, int r, Acc s) {
            const int g = c0 + p;
            const double o = (double)(r >= 0 ? xr[r] : a.x[g]), an = (double)(r >= 0 ? x0r[r] : a.x0[g]);
            const double ctg = (double)(r >= 0 ? ctr[r] : a.ct[g]);
            const double v = o - tau * (ctg - (double)s);
            const double hh = v < 0.0 ? 0.0 : v;
            if (maskrow) {
                const unsigned long long bits = __ballot(v > 0.0);
                if ((tid & (kWave - 1)) == 0) maskrow[p >> 6] = bits;
            }
            xbL[p] = (T)(2.0 * hh - o);
            const T xn = (T)(w * (opr * hh - rho * o) + omw * an);
            if (r >= 0) xr[r] = xn;
            else a.x[g] = xn;
        });
        __syncthreads();
        inst_rows<BS, RS::RR, Acc>(I.levels, m, ga, I.A, lds, xbL, [&](int p, int r, Acc s) {
            const int g = r0 + p;
            const double an = (double)(r >= 0 ? y0r[r] : a.y0[g]), btg = (double)(r >= 0 ? btr[r] : a.bt[g]);
            const double o = (double)yL[p];
            const double hh = o + sig * (btg - (double)s);
            yL[p] = (T)(w * (opr * hh - rho * o) + omw * an);
        });
        __syncthreads();
        if (maskrow) maskrow += W;
    }
    if (I.levels)
#pragma unroll
        for (int r = 0; r < RS::RC; ++r)
            if (tid + r * BS < n) a.x[c0 + tid + r * BS] = xr[r];
}

// state and anchor <- projected point (a restart)
template <typename T, typename V, int BS>
__device__ __forceinline__ void u_restart(const UArgs<T, V>& a, const Inst<T, V>& I) {
    for (int p = opaque(threadIdx.x); p < I.n; p += BS) {
        const T v = a.xhat[I.c0 + p];
        a.x[I.c0 + p] = v;
        a.x0[I.c0 + p] = v;
    }
    for (int p = opaque(threadIdx.x); p < I.m; p += BS) {
        const T v = a.yhat[I.r0 + p];
        I.yl[p] = v;
        a.y0[I.r0 + p] = v;
    }
    __syncthreads();
}

// Set-up of instance i: layout, scaling, scaled matrices and (if no schedule is
// replayed) the first step sizes.  A kernel of its own, so that the registers
// it wants are not taken from the iterations.
template <typename T, typename V, int BS>
__device__ void prepare_instance(const UArgs<T, V>& a, Inst<T, V>& I, int i, unsigned char* lds, double* sh) {
    const InstSetup su = inst_setup<T, V, BS>(I, a.M, a.S, a.d_row, a.d_col, a.pu, a.pav, a.bt, a.ct, a.ruiz, a.pc,
                                              a.power_iters, a.step_safety, lds, a.lds, sh);
    if (threadIdx.x != 0) return;
    a.levels[i] = I.levels;
    if (a.replay) return;
    a.eta[i] = su.eta;
    a.omega0[i] = su.omega0;
    a.taus[i] = su.eta / su.omega0;
    a.sigmas[i] = su.eta * su.omega0;
}

// the layout and the matrices that prepare_instance left
template <typename T, typename V, int BS>
__device__ __forceinline__ void reload_instance(const UArgs<T, V>& a, Inst<T, V>& I, int i, unsigned char* lds) {
    I.levels = uniform(a.levels[i]) != 0;
    I.perm_r = a.S.perm_r + I.r0;
    I.perm_c = a.S.perm_c + I.c0;
    inst_load<T, V, BS>(I, a.M, a.S, lds, a.lds, true);
}

template <typename T, typename V, typename Acc, int BS, bool LONG>
__device__ void forward_instance(const UArgs<T, V>& a, Inst<T, V>& I, int i, unsigned char* lds, double* sh) {
    const int tid = threadIdx.x, B = a.B;
    const int m = I.m, n = I.n, r0 = I.r0, c0 = I.c0;
    reload_instance<T, V, BS>(a, I, i, lds);
    const double eta = uniform(a.eta[i]);  // (unused in a replay)
    double omega = uniform(a.omega0[i]);
    int epoch = 0;
    double tau = uniform(a.taus[i]), sig = uniform(a.sigmas[i]);
    for (int p = tid; p < n; p += BS) {
        a.x[c0 + p] = (T)0;
        a.x0[c0 + p] = (T)0;
    }
    for (int p = tid; p < m; p += BS) {
        I.yl[p] = (T)0;
        a.y0[r0 + p] = (T)0;
    }
    __syncthreads();
    int64_t k = 0;
    double R0 = NAN, R_prev = INFINITY;
    for (int t = 1; t <= a.K;) {
        if ((t - 1) % a.ckpt == 0) {  // checkpoint of the state before iteration t
            const int seg = (t - 1) / a.ckpt;
            for (int p = opaque(tid); p < n; p += BS) {
                a.cp_x[(int64_t)seg * a.N + c0 + p] = a.x[c0 + p];
                a.cp_x0[(int64_t)seg * a.N + c0 + p] = a.x0[c0 + p];
            }
            for (int p = opaque(tid); p < m; p += BS) {
                a.cp_y[(int64_t)seg * a.Mrows + r0 + p] = I.yl[p];
                a.cp_y0[(int64_t)seg * a.Mrows + r0 + p] = a.y0[r0 + p];
            }
            if (tid == 0) {
                a.cp_k[seg * B + i] = (int32_t)k;
                a.cp_ep[seg * B + i] = epoch;
            }
        }
        // plain iterations up to the next checkpoint, evaluation or the end
        if (k != 0 || a.replay) {
            const int to_cp = a.ckpt - (t - 1) % a.ckpt, to_ev = a.E - (t - 1) % a.E - 1, to_end = a.K - t;
            const int plain = min(to_cp, min(to_ev, to_end));
            if (plain > 0) {
                u_plain<T, V, Acc, BS, LONG>(a, I, lds, plain, k, tau, sig, nullptr);
                t += plain;
                k += plain;
                if (plain == to_cp) continue;
            }
        }
        const bool at_eval = (t % a.E == 0) && t < a.K;
        const bool first = k == 0;
        const bool need_q = !a.replay && (first || at_eval) && t < a.K;
        u_iterate<T, V, Acc, BS, LONG>(a, I, lds, k, tau, sig, need_q, at_eval, t == a.K, nullptr);
        double qx[2] = {0.0, 0.0}, qy[2] = {0.0, 0.0};  // ||x - x^||^2, ||x^ - x0||^2 and the same of y
        if (need_q) {
            inst_sums<BS, 2>(n, sh, qx, [&](int j, double(&s)[2]) {
                const double d = a.pu[c0 + j], e = a.xK[c0 + j];
                s[0] += d * d;
                s[1] += e * e;
            });
            inst_sums<BS, 2>(m, sh, qy, [&](int r, double(&s)[2]) {
                const double d = a.pav[r0 + r], e = a.lbt[r0 + r];
                s[0] += d * d;
                s[1] += e * e;
            });
            __syncthreads();
        }
        if (!a.replay && first) R0 = uniform(sqrt(omega * qx[0] + qy[0] / omega));
        ++k;
        const int te = t++;
        if (!at_eval) continue;
        bool restart;
        if (a.replay) {
            restart = a.restart[(int64_t)(te - 1) * B + i] != 0;
        } else {
            const double R = uniform(sqrt(omega * qx[0] + qy[0] / omega));
            restart = a.restarts && ((R <= a.beta_suff * R0) || (R <= a.beta_nec * R0 && R > R_prev) ||
                                     ((double)k >= a.beta_art * (double)te));
            if (restart) {
                const double dx = sqrt(qx[1]), dy = sqrt(qy[1]);
                if (dx > 1e-10 && dy > 1e-10)
                    omega = uniform(exp(a.theta * log(dy / dx) + (1.0 - a.theta) * log(omega)));
                R_prev = INFINITY;
            } else {
                R_prev = R;
            }
        }
        if (restart) {
            ++epoch;
            if (a.replay) {
                tau = uniform(a.taus[(int64_t)epoch * B + i]);
                sig = uniform(a.sigmas[(int64_t)epoch * B + i]);
            } else {
                tau = uniform(eta / omega);
                sig = uniform(eta * omega);
                if (tid == 0) {
                    a.restart[(int64_t)(te - 1) * B + i] = 1;
                    a.taus[(int64_t)epoch * B + i] = tau;
                    a.sigmas[(int64_t)epoch * B + i] = sig;
                }
            }
            u_restart<T, V, BS>(a, I);
            k = 0;
        }
    }
}

// The reverse sweep over iterations te, ..., tb + 1 of a segment, its adjoint
// state in the workspace before and after, in the threads' registers between;
// yL holds lam_yhat, xbL holds lam_g.  The iterations' numbers (k, tau, sigma,
// restart) are loaded 64 at a time, one to a lane.
template <typename T, typename V, typename Acc, int BS, bool LONG>
__device__ __forceinline__ void u_reverse(const UArgs<T, V>& a, const Inst<T, V>& I, const unsigned char* lds, int i,
                                          int tb, int te) {
    typedef RegShape<V> RS;
    const int tid = opaque(threadIdx.x), lane = tid & (kWave - 1);
    const int m = I.m, n = I.n, c0 = I.c0, r0 = I.r0, B = a.B;
    T *const lyhL = I.yl, *const lgL = I.xl;
    const double rho = a.rho, opr = 1.0 + a.rho;
    RegSide<V, RS::RC, RS::KC, LONG> gt;
    RegSide<V, RS::RR, RS::KR, LONG> ga;
    reg_load<BS, T>(gt, I.AT, lds, n, m);
    reg_load<BS, T>(ga, I.A, lds, m, n);
    T lxr[RS::RC], lx0r[RS::RC], lyr[RS::RR], ly0r[RS::RR];
    double lcr[RS::RC], lbr[RS::RR];
#pragma unroll
    for (int r = 0; r < RS::RC; ++r) {
        const int g = c0 + min(tid + r * BS, n - 1);
        lxr[r] = a.lx[g];
        lx0r[r] = a.lx0[g];
        lcr[r] = a.lct[g];
    }
#pragma unroll
    for (int r = 0; r < RS::RR; ++r) {
        const int g = r0 + min(tid + r * BS, m - 1);
        lyr[r] = a.ly[g];
        ly0r[r] = a.ly0[g];
        lbr[r] = a.lbt[g];
    }
    int kl = 0, rl = 0;
    double wl = 1.0, tl = 0.0, sl = 0.0;
    for (int t = te; t > tb; --t) {
        const int back = te - t;
        if ((back & (kWave - 1)) == 0) {
            const int it = max(t - tb - 1 - lane, 0);
            kl = a.kbuf[(int64_t)it * B + i];
            tl = a.tbuf[(int64_t)it * B + i];
            sl = a.sbuf[(int64_t)it * B + i];
            rl = a.restart[(int64_t)(tb + it) * B + i];
            wl = a.halpern ? ((double)kl + 1.0) / ((double)kl + 2.0) : 1.0;
        }
        const int src = back & (kWave - 1);
        const bool rs = __builtin_amdgcn_readlane(rl, src) != 0;
        const double w = lane_value(wl, src), omw = 1.0 - w;
        const double tau = lane_value(tl, src), sig = lane_value(sl, src);
        gt.pin();
        ga.pin();
        // (R1) rows: adjoint of y_hat, of the previous y (partial) and anchor
        auto rows1 = [&](int p, T& lyT, T& ly0T, double& lb) {
            const double ly = (double)lyT, ly0 = (double)ly0T;
            const double lyh = rs ? ly + ly0 : w * opr * ly;
            lyhL[p] = (T)lyh;
            lyT = (T)((rs ? 0.0 : -w * rho * ly) + lyh);
            ly0T = (T)(rs ? 0.0 : ly0 + omw * ly);
            lb += sig * lyh;
        };
        int p = opaque(tid);
        if (I.levels) {
#pragma unroll
            for (int r = 0; r < RS::RR; ++r)
                if (tid + r * BS < m) rows1(tid + r * BS, lyr[r], ly0r[r], lbr[r]);
            p += RS::RR * BS;
        }
        for (; p < m; p += BS) rows1(p, a.ly[r0 + p], a.ly0[r0 + p], a.lbt[r0 + p]);
        __syncthreads();
        // (C) columns: lam_xbar = -sigma A~^T lam_yhat, then extrapolation,
        // projection and primal step
        const uint64_t* mrow = a.masks + (int64_t)(t - tb - 1) * a.W + a.word_off[i];
        inst_rows<BS, RS::RC, Acc>(I.levels, n, gt, I.AT, lds, lyhL, [&](int p, int r, Acc s) {
            const int g = c0 + p;
            const double lxbar = -sig * (double)s;
            const double lx = (double)(r >= 0 ? lxr[r] : a.lx[g]), lx0 = (double)(r >= 0 ? lx0r[r] : a.lx0[g]);
            double lxh = (rs ? lx + lx0 : w * opr * lx) + 2.0 * lxbar;
            if (t == a.K) {
                const int j = I.column(p);
                lxh += a.d_col[j] * a.gx[j];
            }
            const bool on = (mrow[p >> 6] >> (p & 63)) & 1ull;
            const double lv = on ? lxh : 0.0;
            const double lg = -tau * lv;
            const T nx = (T)((rs ? 0.0 : -w * rho * lx) - lxbar + lv), nx0 = (T)(rs ? 0.0 : lx0 + omw * lx);
            if (r >= 0) {
                lxr[r] = nx;
                lx0r[r] = nx0;
                lcr[r] += lg;
            } else {
                a.lx[g] = nx;
                a.lx0[g] = nx0;
                a.lct[g] += lg;
            }
            lgL[p] = (T)lg;
        });
        __syncthreads();
        // (R2) rows: lam_y -= A~ lam_g
        inst_rows<BS, RS::RR, Acc>(I.levels, m, ga, I.A, lds, lgL, [&](int p, int r, Acc s) {
            if (r >= 0) lyr[r] = (T)((double)lyr[r] - (double)s);
            else a.ly[r0 + p] = (T)((double)a.ly[r0 + p] - (double)s);
        });
        // (the next iteration's rows write lyhL, read by nobody since the last
        // barrier, and its columns lgL only after the next one)
    }
    __syncthreads();
    if (I.levels) {
#pragma unroll
        for (int r = 0; r < RS::RC; ++r)
            if (tid + r * BS < n) {
                const int g = c0 + tid + r * BS;
                a.lx[g] = lxr[r];
                a.lx0[g] = lx0r[r];
                a.lct[g] = lcr[r];
            }
#pragma unroll
        for (int r = 0; r < RS::RR; ++r)
            if (tid + r * BS < m) {
                const int g = r0 + tid + r * BS;
                a.ly[g] = lyr[r];
                a.ly0[g] = ly0r[r];
                a.lbt[g] = lbr[r];
            }
    }
}

template <typename T, typename V, typename Acc, int BS, bool LONG>
__device__ void backward_instance(const UArgs<T, V>& a, Inst<T, V>& I, int i, unsigned char* lds) {
    const int tid = threadIdx.x, B = a.B;
    const int m = I.m, n = I.n, r0 = I.r0, c0 = I.c0;
    reload_instance<T, V, BS>(a, I, i, lds);
    for (int p = tid; p < n; p += BS) {
        const int g = c0 + p;
        a.lx[g] = (T)0;
        a.lx0[g] = (T)0;
        a.lct[g] = 0.0;
    }
    for (int p = tid; p < m; p += BS) {
        const int g = r0 + p;
        a.ly[g] = (T)0;
        a.ly0[g] = (T)0;
        a.lbt[g] = 0.0;
    }
    for (int seg = a.nseg - 1; seg >= 0; --seg) {
        const int tb = seg * a.ckpt, te = min(a.K, tb + a.ckpt);
        // restore the checkpoint and recompute the segment, keeping masks
        for (int p = opaque(tid); p < n; p += BS) {
            a.x[c0 + p] = a.cp_x[(int64_t)seg * a.N + c0 + p];
            a.x0[c0 + p] = a.cp_x0[(int64_t)seg * a.N + c0 + p];
        }
        for (int p = opaque(tid); p < m; p += BS) {
            I.yl[p] = a.cp_y[(int64_t)seg * a.Mrows + r0 + p];
            a.y0[r0 + p] = a.cp_y0[(int64_t)seg * a.Mrows + r0 + p];
        }
        int64_t k = uniform(a.cp_k[seg * B + i]);
        int epoch = uniform(a.cp_ep[seg * B + i]);
        __syncthreads();
        for (int t = tb + 1; t <= te;) {
            const double tau = uniform(a.taus[(int64_t)epoch * B + i]), sig = uniform(a.sigmas[(int64_t)epoch * B + i]);
            // the iterations up to the next one that may restart, or te
            const int to_ev = a.E - (t - 1) % a.E - 1;
            const int plain = min(to_ev, te - t + 1);
            auto note = [&](int it0, int cnt) {
                for (int q = tid; q < cnt; q += BS) {
                    a.kbuf[(int64_t)(it0 + q) * B + i] = (int32_t)(k + q);
                    a.tbuf[(int64_t)(it0 + q) * B + i] = tau;
                    a.sbuf[(int64_t)(it0 + q) * B + i] = sig;
                }
            };
            uint64_t* const masks = a.masks + (int64_t)(t - tb - 1) * a.W + a.word_off[i];
            if (plain > 0) {
                note(t - tb - 1, plain);
                u_plain<T, V, Acc, BS, LONG>(a, I, lds, plain, k, tau, sig, masks);
                t += plain;
                k += plain;
                continue;
            }
            note(t - tb - 1, 1);
            const bool rs = a.restart[(int64_t)(t - 1) * B + i] != 0;
            u_iterate<T, V, Acc, BS, LONG>(a, I, lds, k, tau, sig, false, rs, false, masks);
            ++t;
            ++k;
            if (rs) {
                u_restart<T, V, BS>(a, I);
                k = 0;
                ++epoch;
            }
        }
        __syncthreads();  // the iterations' numbers and masks are read by all
        u_reverse<T, V, Acc, BS, LONG>(a, I, lds, i, tb, te);
        __syncthreads();
    }
    for (int p = opaque(tid); p < n; p += BS) {
        const int j = I.column(p);
        a.gc[j] = a.d_col[j] * a.lct[c0 + p];
    }
    for (int p = opaque(tid); p < m; p += BS) {
        const int r = I.row(p);
        a.gb[r] = a.d_row[r] * a.lbt[r0 + p];
    }
    __syncthreads();
}

enum { kPrepare = 0, kForward = 1, kBackward = 2 };

template <typename T, typename V, typename Acc, int BS, int PHASE, bool LONG>
__global__ __launch_bounds__(BS, 4) void k_unrolled(UArgs<T, V> a) {
    extern __shared__ __align__(16) unsigned char lds[];
    __shared__ double sh[BS / kWave > 12 ? BS / kWave : 12];
    __shared__ int next;
    while (true) {
        if (threadIdx.x == 0) next = atomicAdd(a.counter + PHASE, 1);
        __syncthreads();
        const int qi = __builtin_amdgcn_readfirstlane(next);
        __syncthreads();
        if (qi >= a.B) break;
        Inst<T, V> I;
        I.r0 = uniform(a.row_off[qi]);
        I.c0 = uniform(a.col_off[qi]);
        I.m = uniform(a.row_off[qi + 1]) - I.r0;
        I.n = uniform(a.col_off[qi + 1]) - I.c0;
        I.z0 = uniform(a.M.a_rowptr[I.r0]);
        I.nnz = uniform(a.M.a_rowptr[I.r0 + I.m]) - I.z0;
        I.yl = (T*)lds;
        I.xl = (T*)(lds + inst_align((I.m + 1) * (int)sizeof(T)));
        if (PHASE == kPrepare) prepare_instance<T, V, BS>(a, I, qi, lds, sh);
        else if (PHASE == kBackward) backward_instance<T, V, Acc, BS, LONG>(a, I, qi, lds);
        else forward_instance<T, V, Acc, BS, LONG>(a, I, qi, lds, sh);
        __syncthreads();  // the next instance takes over the LDS
    }
}

__global__ void k_zero_bytes(uint8_t* p, int64_t n) {
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        p[i] = 0;
}

// ---------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------
struct TapeLayout {
    int32_t *row_off, *col_off, *word_off, *counter;
    double *d_row, *d_col, *pu, *pav, *eta, *omega0, *taus, *sigmas;
    void *a_vs, *at_vs, *bt, *ct;
    uint16_t *a_cl, *at_cl, *perm_r, *perm_c;
    int32_t* levels;
    int8_t* restart;
    void *cp_x, *cp_x0, *cp_y, *cp_y0;
    int32_t *cp_k, *cp_ep;
    void *x, *x0, *y0, *xhat, *yhat;
    uint64_t* masks;
    int32_t* kbuf;
    double *tbuf, *sbuf;
    void *lx, *lx0, *ly, *ly0;
    double *lct, *lbt;
    int64_t* nnz_off;  // input validation (forward)
    int32_t* vflags;
    double* vpartials;
    int32_t W, nseg, nep;
    size_t bytes;
};

static TapeLayout carve_tape(void* base, size_t cap, const mipdhg_batch& bt, int prec, int K, int ckpt, int E) {
    Carver cv(base, cap);
    TapeLayout t;
    const int64_t B = bt.count, m = bt.whole.m, n = bt.whole.n, nnz = bt.whole.nnz;
    const size_t vs = prec == MIPDHG_FP64 ? 8 : (prec == MIPDHG_FP32_BF16A ? 2 : 4);
    const size_t ts = prec == MIPDHG_FP64 ? 8 : 4;
    int64_t W = 0;
    for (int64_t i = 0; i < B; ++i) W += (bt.col_off[i + 1] - bt.col_off[i] + 63) / 64;
    t.W = (int32_t)W;
    t.nseg = (K + ckpt - 1) / ckpt;
    t.nep = (K - 1) / E + 2;
    t.row_off = cv.take<int32_t>(B + 1);
    t.col_off = cv.take<int32_t>(B + 1);
    t.word_off = cv.take<int32_t>(B + 1);
    t.counter = cv.take<int32_t>(64);
    t.d_row = cv.take<double>(m);
    t.d_col = cv.take<double>(n);
    t.pu = cv.take<double>(n);
    t.pav = cv.take<double>(m);
    t.eta = cv.take<double>(B);
    t.omega0 = cv.take<double>(B);
    t.taus = cv.take<double>((size_t)t.nep * B);
    t.sigmas = cv.take<double>((size_t)t.nep * B);
    t.a_vs = cv.take<char>(nnz * vs);
    t.at_vs = cv.take<char>(nnz * vs);
    t.a_cl = cv.take<uint16_t>(nnz);
    t.at_cl = cv.take<uint16_t>(nnz);
    t.perm_r = cv.take<uint16_t>(m);
    t.perm_c = cv.take<uint16_t>(n);
    t.levels = cv.take<int32_t>(B);
    t.bt = cv.take<char>(m * ts);
    t.ct = cv.take<char>(n * ts);
    t.restart = cv.take<int8_t>((size_t)K * B);
    t.cp_x = cv.take<char>((size_t)t.nseg * n * ts);
    t.cp_x0 = cv.take<char>((size_t)t.nseg * n * ts);
    t.cp_y = cv.take<char>((size_t)t.nseg * m * ts);
    t.cp_y0 = cv.take<char>((size_t)t.nseg * m * ts);
    t.cp_k = cv.take<int32_t>((size_t)t.nseg * B);
    t.cp_ep = cv.take<int32_t>((size_t)t.nseg * B);
    t.x = cv.take<char>(n * ts);
    t.x0 = cv.take<char>(n * ts);
    t.y0 = cv.take<char>(m * ts);
    t.xhat = cv.take<char>(n * ts);
    t.yhat = cv.take<char>(m * ts);
    t.masks = cv.take<uint64_t>((size_t)ckpt * W);
    t.kbuf = cv.take<int32_t>((size_t)ckpt * B);
    t.tbuf = cv.take<double>((size_t)ckpt * B);
    t.sbuf = cv.take<double>((size_t)ckpt * B);
    t.lx = cv.take<char>(n * ts);
    t.lx0 = cv.take<char>(n * ts);
    t.ly = cv.take<char>(m * ts);
    t.ly0 = cv.take<char>(m * ts);
    t.lct = cv.take<double>(n);
    t.lbt = cv.take<double>(m);
    t.nnz_off = cv.take<int64_t>(B + 1);
    t.vflags = cv.take<int32_t>(64);
    t.vpartials = cv.take<double>(4 * kCheckGrid);
    t.bytes = (cv.off + 255) & ~size_t(255);
    return t;
}

static int check_unrolled(const mipdhg_batch* bt, const mipdhg_options* o, int K, int ckpt) {
    if (!bt || !o) return set_error("NULL argument"), MIPDHG_ERR_INVALID_ARG;
    if (bt->count < 1 || !bt->row_off || !bt->col_off || !bt->nnz_off)
        return set_error("batch count >= 1 and host offsets are required"), MIPDHG_ERR_INVALID_ARG;
    int rc = check_lp(&bt->whole);
    if (rc) return rc;
    if ((rc = check_options(o))) return rc;
    if (K < 1 || ckpt < 1) return set_error("K >= 1 and ckpt_every >= 1 required"), MIPDHG_ERR_INVALID_ARG;
    if (o->resume) return set_error("the unrolled map has no state to resume"), MIPDHG_ERR_UNSUPPORTED;
    if (is_general(bt->whole))
        return set_error("the general form (bounds, inequality rows) is a single-LP option"), MIPDHG_ERR_UNSUPPORTED;
    if (o->pw_ki != 0.0 || o->pw_kd != 0.0 || o->restart_avg || o->step_rule)
        return set_error("the PID primal weight, restart to average and the adaptive step are single-LP options"),
               MIPDHG_ERR_UNSUPPORTED;
    const int B = bt->count;
    if (bt->row_off[0] != 0 || bt->col_off[0] != 0 || bt->nnz_off[0] != 0 || bt->row_off[B] != bt->whole.m ||
        bt->col_off[B] != bt->whole.n || bt->nnz_off[B] != bt->whole.nnz)
        return set_error("instance offsets must start at 0 and end at m, n, nnz"), MIPDHG_ERR_INVALID_ARG;
    for (int i = 0; i < B; ++i)
        if (bt->row_off[i + 1] <= bt->row_off[i] || bt->col_off[i + 1] <= bt->col_off[i])
            return set_error("instance %d is empty", i), MIPDHG_ERR_INVALID_ARG;
    return 0;
}

template <typename T, typename V, typename Acc, int BS, int PHASE>
static int launch_phase(const UArgs<T, V>& a, bool rests, int cus, hipStream_t s) {
    auto* k = rests ? k_unrolled<T, V, Acc, BS, PHASE, LongRows<V>::ok && PHASE != kPrepare>
                    : k_unrolled<T, V, Acc, BS, PHASE, false>;
    int per_cu = 1;
    MIP_HIP(hipFuncSetAttribute((const void*)k, hipFuncAttributeMaxDynamicSharedMemorySize, 162000));
    MIP_HIP(hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, k, BS, a.lds));
    const int grid = std::max(1, std::min(a.B, cus * std::max(per_cu, 1)));
    hipLaunchKernelGGL(k, dim3(grid), dim3(BS), a.lds, s, a);
    MIP_LAUNCH_CHECK();
    return 0;
}
template <typename T, typename V, typename Acc, int BS>
static int launch_unrolled(const UArgs<T, V>& a, bool rests, int cus, bool backward, hipStream_t s) {
    if (backward) return launch_phase<T, V, Acc, BS, kBackward>(a, rests, cus, s);
    if (int rc = launch_phase<T, V, Acc, BS, kPrepare>(a, rests, cus, s)) return rc;
    return launch_phase<T, V, Acc, BS, kForward>(a, rests, cus, s);
}

template <typename T, typename V, typename Acc>
static int unrolled_impl(const mipdhg_batch& bt, const mipdhg_options& o, int K, int ckpt, void* tape,
                         size_t tape_bytes, hipStream_t stream, bool backward, int replay, const double* gx,
                         double* out1, double* out2) {
    TapeLayout t = carve_tape(tape, tape_bytes, bt, o.precision, K, ckpt, o.eval_every);
    if (t.bytes > tape_bytes)
        return set_error("tape too small: %zu bytes given, %zu needed", tape_bytes, t.bytes), MIPDHG_ERR_WORKSPACE;
    if (((uintptr_t)tape & 255) != 0) return set_error("tape must be 256-byte aligned"), MIPDHG_ERR_INVALID_ARG;
    const int B = bt.count;
    int max_m = 0, max_n = 0;
    for (int i = 0; i < B; ++i) {
        max_m = std::max(max_m, bt.row_off[i + 1] - bt.row_off[i]);
        max_n = std::max(max_n, bt.col_off[i + 1] - bt.col_off[i]);
    }
    const int lds = (int)(((size_t)max_m + (size_t)max_n) * sizeof(T) + 16);  // the vectors'
    if (lds > 150 * 1024 || max_m > kInstMaxDim || max_n > kInstMaxDim)
        return set_error("instance too large for LDS (%d bytes)", lds), MIPDHG_ERR_UNSUPPORTED;
    StreamDrain drain{stream};
    const mipdhg_lp& lp = bt.whole;
    if (!backward) {
        std::vector<int32_t> wo(B + 1, 0);
        for (int i = 0; i < B; ++i) wo[i + 1] = wo[i] + (bt.col_off[i + 1] - bt.col_off[i] + 63) / 64;
        MIP_HIP(hipMemcpyAsync(t.row_off, bt.row_off, (B + 1) * 4, hipMemcpyHostToDevice, stream));
        MIP_HIP(hipMemcpyAsync(t.col_off, bt.col_off, (B + 1) * 4, hipMemcpyHostToDevice, stream));
        MIP_HIP(hipMemcpyAsync(t.word_off, wo.data(), (B + 1) * 4, hipMemcpyHostToDevice, stream));
        // row pointers, column ranges, finiteness, A^T against A, and the block-diagonal
        // structure, before any kernel indexes with the columns
        if (int rc = check_blocks(bt, o.validate, t.row_off, t.col_off, t.nnz_off, t.vflags, t.vpartials, stream))
            return rc;
        if (!replay)
            hipLaunchKernelGGL(k_zero_bytes, dim3(grid_for((int64_t)K * B)), dim3(kBlock), 0, stream,
                               (uint8_t*)t.restart, (int64_t)K * B);
        MIP_HIP(hipStreamSynchronize(stream));  // host vectors go out of scope
    }
    UArgs<T, V> a;
    memset(&a, 0, sizeof(a));
    a.B = B;
    a.K = K;
    a.ckpt = ckpt;
    a.E = o.eval_every;
    a.nseg = t.nseg;
    a.nep = t.nep;
    a.W = t.W;
    a.replay = replay;
    a.N = lp.n;
    a.Mrows = lp.m;
    a.row_off = t.row_off;
    a.col_off = t.col_off;
    a.word_off = t.word_off;
    a.M = InstMat{lp.a_rowptr, lp.a_col, lp.a_val, lp.at_rowptr, lp.at_col, lp.at_val, lp.b, lp.c};
    a.d_row = t.d_row;
    a.d_col = t.d_col;
    a.pu = t.pu;
    a.pav = t.pav;
    a.S = InstStore<V>{(V*)t.a_vs, (V*)t.at_vs, t.a_cl, t.at_cl, t.perm_r, t.perm_c};
    a.levels = t.levels;
    a.bt = (T*)t.bt;
    a.ct = (T*)t.ct;
    a.eta = t.eta;
    a.omega0 = t.omega0;
    a.taus = t.taus;
    a.sigmas = t.sigmas;
    a.restart = t.restart;
    a.cp_x = (T*)t.cp_x;
    a.cp_x0 = (T*)t.cp_x0;
    a.cp_y = (T*)t.cp_y;
    a.cp_y0 = (T*)t.cp_y0;
    a.cp_k = t.cp_k;
    a.cp_ep = t.cp_ep;
    a.x = (T*)t.x;
    a.x0 = (T*)t.x0;
    a.y0 = (T*)t.y0;
    a.xhat = (T*)t.xhat;
    a.yhat = (T*)t.yhat;
    a.masks = t.masks;
    a.kbuf = t.kbuf;
    a.tbuf = t.tbuf;
    a.sbuf = t.sbuf;
    a.lx = (T*)t.lx;
    a.lx0 = (T*)t.lx0;
    a.ly = (T*)t.ly;
    a.ly0 = (T*)t.ly0;
    a.lct = t.lct;
    a.lbt = t.lbt;
    a.gx = gx;
    a.xK = backward ? nullptr : out1;
    a.gc = backward ? out1 : nullptr;
    a.gb = backward ? out2 : nullptr;
    a.counter = t.counter;
    a.step_safety = o.step_safety;
    a.rho = o.reflect_rho;
    a.beta_suff = o.beta_suff;
    a.beta_nec = o.beta_nec;
    a.beta_art = o.beta_art;
    a.theta = o.pw_theta;
    a.ruiz = o.ruiz_iters;
    a.pc = o.pock_chambolle;
    a.power_iters = o.power_iters;
    a.halpern = o.halpern;
    a.restarts = o.restarts;
    int dev = 0, cus = 256;
    MIP_HIP(hipGetDevice(&dev));
    MIP_HIP(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev));
    // One launch of workgroups shaped for the largest instance: with no more
    // instances than compute units about one thread per column and all the
    // LDS the instance can use; with more, as many waves as keep 16 on a
    // compute unit (see kClassBs in batched.hip, and one_wave).  48 maps, FP32,
    // K = 200, forward and backward: at 100 columns 64 threads 1.99 ms, 256 1.77; at
    // 200 256 threads 1.83, 1,024 1.95; at 375 2.13 and 2.04; at 750 3.31 and 2.35.
    int64_t full[3] = {0, 0, 0};
    const int bs[3] = {1024, 256, 64};
    const int64_t share[3] = {162000, 40400, 9700};
    for (int c = 0; c < 3; ++c)
        for (int i = 0; i < B; ++i) {
            typedef RegShape<V> RS;
            const int mi = bt.row_off[i + 1] - bt.row_off[i], ni = bt.col_off[i + 1] - bt.col_off[i];
            const int64_t zi = bt.nnz_off[i + 1] - bt.nnz_off[i];
            const int64_t nreg = std::min(ni, RS::RC * bs[c]) * std::min<int64_t>(zi / ni, RS::KC) +
                                 std::min(mi, RS::RR * bs[c]) * std::min<int64_t>(zi / mi, RS::KR);
            full[c] = std::max(full[c], inst_full_bytes(mi, ni, zi, sizeof(T), sizeof(V), nreg));
        }
    int c;
    if (B <= cus) c = std::max(max_m, max_n) <= 64 ? 2 : max_n <= 256 ? 1 : 0;
    else c = full[2] <= share[2] && one_wave(B, cus, max_m, max_n) ? 2 : full[1] <= share[1] ? 1 : 0;
    a.lds = (int)std::max<int64_t>(inst_vec_bytes(max_m, max_n, sizeof(T)),
                                   std::min(full[c], B <= cus ? share[0] : share[c]));
    hipLaunchKernelGGL(k_zero_bytes, dim3(1), dim3(64), 0, stream, (uint8_t*)t.counter, (int64_t)256);
    const bool rests = LongRows<V>::pays(lp.m, lp.nnz);
    int rc;
    if (c == 0) rc = launch_unrolled<T, V, Acc, 1024>(a, rests, cus, backward, stream);
    else if (c == 1) rc = launch_unrolled<T, V, Acc, 256>(a, rests, cus, backward, stream);
    else rc = launch_unrolled<T, V, Acc, 64>(a, rests, cus, backward, stream);
    if (rc) return rc;
    MIP_LAUNCH_CHECK();
    MIP_HIP(hipStreamSynchronize(stream));
    drain.armed = false;
    return 0;
}

}  // namespace mip

using namespace mip;

extern "C" int mipdhg_unrolled_tape_size(const mipdhg_batch* bt, const mipdhg_options* opt, int32_t K,
                                         int32_t ckpt_every, size_t* bytes) {
    clear_error();
    int rc = check_unrolled(bt, opt, K, ckpt_every);
    if (rc) return rc;
    if (!bytes) return set_error("bytes is NULL"), MIPDHG_ERR_INVALID_ARG;
    *bytes = carve_tape(nullptr, 0, *bt, opt->precision, K, ckpt_every, opt->eval_every).bytes;
    return 0;
}

extern "C" int mipdhg_unrolled_forward(const mipdhg_batch* bt, const mipdhg_options* opt, int32_t K,
                                       int32_t ckpt_every, int32_t replay, void* tape, size_t tape_bytes,
                                       void* stream, double* x_K) {
    clear_error();
    int rc = check_unrolled(bt, opt, K, ckpt_every);
    if (rc) return rc;
    if (!tape || !x_K) return set_error("tape and x_K are required"), MIPDHG_ERR_INVALID_ARG;
    hipStream_t s = (hipStream_t)stream;
    if (opt->precision == MIPDHG_FP32_A)
        return set_error("FP32_A is a single-LP precision mode"), MIPDHG_ERR_UNSUPPORTED;
    switch (opt->precision) {
        case MIPDHG_FP64:
            return unrolled_impl<double, double, double>(*bt, *opt, K, ckpt_every, tape, tape_bytes, s, false, replay,
                                                         nullptr, x_K, nullptr);
        case MIPDHG_FP32:
            return unrolled_impl<float, float, double>(*bt, *opt, K, ckpt_every, tape, tape_bytes, s, false, replay,
                                                       nullptr, x_K, nullptr);
        case MIPDHG_FP32_BF16A:
            return unrolled_impl<float, uint16_t, double>(*bt, *opt, K, ckpt_every, tape, tape_bytes, s, false,
                                                          replay, nullptr, x_K, nullptr);
        default:
            return unrolled_impl<float, float, float>(*bt, *opt, K, ckpt_every, tape, tape_bytes, s, false, replay,
                                                      nullptr, x_K, nullptr);
    }
}

extern "C" int mipdhg_unrolled_backward(const mipdhg_batch* bt, const mipdhg_options* opt, int32_t K,
                                        int32_t ckpt_every, void* tape, size_t tape_bytes, const double* grad_xK,
                                        void* stream, double* grad_c, double* grad_b) {
    clear_error();
    int rc = check_unrolled(bt, opt, K, ckpt_every);
    if (rc) return rc;
    if (!tape || !grad_xK || !grad_c || !grad_b)
        return set_error("tape, grad_xK, grad_c and grad_b are required"), MIPDHG_ERR_INVALID_ARG;
    hipStream_t s = (hipStream_t)stream;
    if (opt->precision == MIPDHG_FP32_A)
        return set_error("FP32_A is a single-LP precision mode"), MIPDHG_ERR_UNSUPPORTED;
    switch (opt->precision) {
        case MIPDHG_FP64:
            return unrolled_impl<double, double, double>(*bt, *opt, K, ckpt_every, tape, tape_bytes, s, true, 1,
                                                         grad_xK, grad_c, grad_b);
        case MIPDHG_FP32:
            return unrolled_impl<float, float, double>(*bt, *opt, K, ckpt_every, tape, tape_bytes, s, true, 1, grad_xK,
                                                       grad_c, grad_b);
        case MIPDHG_FP32_BF16A:
            return unrolled_impl<float, uint16_t, double>(*bt, *opt, K, ckpt_every, tape, tape_bytes, s, true, 1,
                                                          grad_xK, grad_c, grad_b);
        default:
            return unrolled_impl<float, float, float>(*bt, *opt, K, ckpt_every, tape, tape_bytes, s, true, 1, grad_xK,
                                                      grad_c, grad_b);
    }
}

extern "C" int mipdhg_unrolled_schedule(const mipdhg_batch* bt, const mipdhg_options* opt, int32_t K,
                                        int32_t ckpt_every, const void* tape, size_t tape_bytes, int32_t inst,
                                        void* stream, int32_t capacity, int32_t* restart_at, double* taus,
                                        double* sigmas, int32_t* n_restarts) {
    clear_error();
    int rc = check_unrolled(bt, opt, K, ckpt_every);
    if (rc) return rc;
    if (!tape || !restart_at || !taus || !sigmas || !n_restarts)
        return set_error("tape and the four outputs are required"), MIPDHG_ERR_INVALID_ARG;
    if (inst < 0 || inst >= bt->count) return set_error("inst must be in [0, count)"), MIPDHG_ERR_INVALID_ARG;
    const TapeLayout t = carve_tape(const_cast<void*>(tape), tape_bytes, *bt, opt->precision, K, ckpt_every,
                                    opt->eval_every);
    if (t.bytes > tape_bytes)
        return set_error("tape too small: %zu bytes given, %zu needed", tape_bytes, t.bytes), MIPDHG_ERR_WORKSPACE;
    const int B = bt->count;
    hipStream_t s = (hipStream_t)stream;
    std::vector<int8_t> flags((size_t)K * B);
    std::vector<double> tv((size_t)t.nep * B), sv((size_t)t.nep * B);
    MIP_HIP(hipMemcpyAsync(flags.data(), t.restart, flags.size(), hipMemcpyDeviceToHost, s));
    MIP_HIP(hipMemcpyAsync(tv.data(), t.taus, tv.size() * 8, hipMemcpyDeviceToHost, s));
    MIP_HIP(hipMemcpyAsync(sv.data(), t.sigmas, sv.size() * 8, hipMemcpyDeviceToHost, s));
    MIP_HIP(hipStreamSynchronize(s));
    int32_t nr = 0;
    for (int32_t it = 1; it <= K; ++it)
        if (flags[(size_t)(it - 1) * B + inst]) {
            if (nr + 1 >= capacity)
                return set_error("capacity %d holds fewer epochs than the schedule's", capacity),
                       MIPDHG_ERR_INVALID_ARG;
            restart_at[nr++] = it;
        }
    if (nr + 1 > capacity || nr + 1 > t.nep)
        return set_error("capacity %d holds fewer epochs than the schedule's", capacity), MIPDHG_ERR_INVALID_ARG;
    for (int32_t e = 0; e <= nr; ++e) {
        taus[e] = tv[(size_t)e * B + inst];
        sigmas[e] = sv[(size_t)e * B + inst];
    }
    *n_restarts = nr;
    return 0;
}
