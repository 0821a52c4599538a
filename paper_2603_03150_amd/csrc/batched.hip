// Many independent LPs in one persistent launch.
//
// The instances are the diagonal blocks of one block-diagonal CSR pair.  Each
// workgroup takes instances from an atomic queue (largest first) and runs the
// whole method of the single solve on its instance: scaling, power iteration,
// the PDHG iterations, float64 evaluations on the original block and the
// restart / primal-weight rule, with __syncthreads() as the only phase barrier.
// The dual iterate y and the extrapolated primal x_bar, the two vectors the
// SpMVs gather from, live in LDS; between evaluations each thread holds the
// entries of its rows and columns and their vectors' entries in registers, and
// LDS takes what they leave of the matrices (see Side and RegSide).  An
// iteration is then two barriers and, for each row, a few gathers in LDS: it
// is bound by their latency and by the instructions a wave issues.  Every
// reduction is a fixed-order workgroup reduction whose result every thread
// holds, so all threads take the same decisions without a broadcast and the
// results do not depend on which workgroup ran the instance.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <chrono>
#include <cstring>
#include <numeric>
#include <vector>

#include "common.h"
#include "inst_common.h"
#include "plain.h"

namespace mip {

constexpr int kClasses = 4;  // launch classes (see kClassBs)

struct BInst {  // per-instance result, device side
    int32_t status, restarts;
    int64_t iters;
    double rp2, rd2, pobj, dobj, xz, rp_inf, rd_inf;
    double b_norm, c_norm, sigma_hat, eta, omega0, omega;
};

struct BState {  // an instance's solve state between resumable calls
    int64_t t, k;
    double omega, tau, sig, R0, R_prev;
    int32_t restarts, phase;  // phase: 1 suspended, 2 finished
    int32_t levels, pad;      // the matrices' layout (see Side)
};

template <typename T, typename V>
struct BArgs {
    int32_t B;
    int32_t lds;  // bytes of dynamic LDS per workgroup
    const int32_t* order;
    const int32_t* row_off;
    const int32_t* col_off;
    InstMat M;
    InstStore<V> S;
    // the state relative to the epoch's anchor (x0, y0): x holds u = x - x0
    // (y's v = y - y0 is in LDS), ct and bt the anchor's residuals
    // c~ - A~^T y0 and b~ - A~ x0; all by position (see Side)
    T *x, *x0, *xhat, *ct, *y0, *yhat, *bt;
    double *d_row, *d_col, *pu, *pav;
    double *xo, *yo, *zo, *rpo, *rdo;
    BInst* info;
    BState* state;
    T* ysave;  // y of suspended instances
    int32_t* counter;
    const double* eps;  // per-instance eps_rel
    int32_t resume, block_iters;
    double step_safety, rho, beta_suff, beta_nec, beta_art, theta;
    int64_t max_iter;
    int32_t ruiz, pc, power_iters, eval_every, halpern, restarts;
};

// The instance's sizes and its vectors in LDS
template <typename T, typename V>
__device__ __forceinline__ Inst<T, V> inst_of(const BArgs<T, V>& a, int inst, unsigned char* lds) {
    Inst<T, V> I;
    I.r0 = uniform(a.row_off[inst]);
    I.c0 = uniform(a.col_off[inst]);
    I.m = uniform(a.row_off[inst + 1]) - I.r0;
    I.n = uniform(a.col_off[inst + 1]) - I.c0;
    I.z0 = uniform(a.M.a_rowptr[I.r0]);
    I.nnz = uniform(a.M.a_rowptr[I.r0 + I.m]) - I.z0;
    I.yl = (T*)lds;
    I.xl = (T*)(lds + inst_align((I.m + 1) * (int)sizeof(T)));
    return I;
}

// The instance's set-up, and its state before the first iteration
template <typename T, typename V, int BS>
__device__ void setup_instance(const BArgs<T, V>& a, int inst, unsigned char* lds, double* sh) {
    Inst<T, V> I = inst_of(a, inst, lds);
    const InstSetup su = inst_setup<T, V, BS>(I, a.M, a.S, a.d_row, a.d_col, a.pu, a.pav, a.bt, a.ct, a.ruiz, a.pc,
                                              a.power_iters, a.step_safety, lds, a.lds, sh);
    if (threadIdx.x == 0) {
        BInst& r = a.info[inst];
        r.b_norm = su.b_norm;
        r.c_norm = su.c_norm;
        r.sigma_hat = su.sigma_hat;
        r.eta = su.eta;
        r.omega0 = su.omega0;
        BState& st = a.state[inst];
        st.phase = 1;
        st.levels = I.levels;
        st.t = 0;
        st.k = 0;
        st.omega = su.omega0;
        st.tau = su.eta / su.omega0;
        st.sig = su.eta * su.omega0;
        st.R0 = NAN;
        st.R_prev = INFINITY;
        st.restarts = 0;
    }
    // initial point (0, 0)
    for (int p = threadIdx.x; p < I.n; p += BS) {
        a.x[I.c0 + p] = (T)0;
        a.x0[I.c0 + p] = (T)0;
    }
    for (int p = threadIdx.x; p < I.m; p += BS) {
        a.ysave[I.r0 + p] = (T)0;
        a.y0[I.r0 + p] = (T)0;
    }
}

// `count` iterations of an instance with no sums, from iteration k of the
// epoch on.  Each thread loads its register rows first (a loop of their own,
// so that nothing else competes for the registers: they are read again after
// each evaluation, a few us in about 60 us).  Float64 arithmetic, stored in
// T: u = x - x0, v = y - y0 (in LDS), rc = c~ - A~^T y0, rb = b~ - A~ x0:
// x_hat = x0 + max(u - tau (rc - A~^T v), -x0),
// y_hat = y0 + v + sigma (rb - A~ (x_bar - x0)).
template <typename T, typename V, typename Acc, int BS, bool LONG>
__device__ __forceinline__ void plain_iterations(const BArgs<T, V>& a, const Inst<T, V>& I, unsigned char* lds, int count,
                                                 int64_t k, double tau, double sig) {
    typedef RegShape<V> RS;
    const int tid = opaque(threadIdx.x);
    const int m = I.m, n = I.n, c0 = I.c0, r0 = I.r0;
    T *const yL = I.yl, *const xbL = I.xl;
    const double rho = a.rho, opr = 1.0 + a.rho;
    RegSide<V, RS::RC, RS::KC, LONG> gt;
    RegSide<V, RS::RR, RS::KR, LONG> ga;
    reg_load<BS, T>(gt, I.AT, lds, n, m);
    reg_load<BS, T>(ga, I.A, lds, m, n);
    T ur[RS::RC], x0r[RS::RC], rcr[RS::RC], rbr[RS::RR];
#pragma unroll
    for (int r = 0; r < RS::RC; ++r) {
        const int g = c0 + min(tid + r * BS, n - 1);
        ur[r] = a.x[g];
        x0r[r] = a.x0[g];
        rcr[r] = a.ct[g];
    }
#pragma unroll
    for (int r = 0; r < RS::RR; ++r) rbr[r] = a.bt[r0 + min(tid + r * BS, m - 1)];
    double wl = 1.0;  // lane l: the Halpern weight of iteration l of each 64
    for (int it = 0; it < count; ++it) {
        if (a.halpern && (it & (kWave - 1)) == 0) {
            const double kl = (double)(k + it + (tid & (kWave - 1)));
            wl = (kl + 1.0) / (kl + 2.0);
        }
        const double w = lane_value(wl, it & (kWave - 1));
        gt.pin();
        ga.pin();
        inst_rows<BS, RS::RC, Acc>(I.levels, n, gt, I.AT, lds, yL, [&](int p, int r, Acc s) {
            const int g = c0 + p;
            const double u = (double)(r >= 0 ? ur[r] : a.x[g]), x0 = (double)(r >= 0 ? x0r[r] : a.x0[g]);
            const double rc = (double)(r >= 0 ? rcr[r] : a.ct[g]);
            double uh = u - tau * (rc - (double)s);
            uh = uh < -x0 ? -x0 : uh;
            xbL[p] = (T)(2.0 * uh - u);  // x_bar - x0
            const T un = (T)(w * (opr * uh - rho * u));
            if (r >= 0) ur[r] = un;
            else a.x[g] = un;
        });
        __syncthreads();
        inst_rows<BS, RS::RR, Acc>(I.levels, m, ga, I.A, lds, xbL, [&](int p, int r, Acc s) {
            const double rb = (double)(r >= 0 ? rbr[r] : a.bt[r0 + p]);
            const double v = (double)yL[p];
            const double vh = v + sig * (rb - (double)s);
            yL[p] = (T)(w * (opr * vh - rho * v));
        });
        __syncthreads();
    }
    if (I.levels)
#pragma unroll
        for (int r = 0; r < RS::RC; ++r)
            if (tid + r * BS < n) a.x[c0 + tid + r * BS] = ur[r];
}

// The iterations of an instance from the state in the workspace (set up, or
// suspended at the end of a block): the scaled matrix, b~, c~, the scaling, x,
// the anchors and the report's set-up fields, y and the scalars.
template <typename T, typename V, typename Acc, int BS, bool LONG>
__device__ void solve_instance(const BArgs<T, V>& a, int inst, unsigned char* lds, double* sh) {
    const int tid = threadIdx.x;
    BState& st = a.state[inst];
    if (uniform(st.phase) == 2) return;  // finished in an earlier call: its outputs and report stand
    Inst<T, V> I = inst_of(a, inst, lds);
    const int r0 = I.r0, c0 = I.c0, m = I.m, n = I.n;
    T *const yL = I.yl, *const xbL = I.xl;
    const double eps = uniform(a.eps[inst]);
    const BInst& in = a.info[inst];
    const double eta = uniform(in.eta), tol_p = uniform(eps * (1.0 + in.b_norm)),
                 tol_d = uniform(eps * (1.0 + in.c_norm));
    double omega = uniform(st.omega), tau = uniform(st.tau), sig = uniform(st.sig), R0 = uniform(st.R0),
           R_prev = uniform(st.R_prev);
    int64_t k = uniform64(st.k), t = uniform64(st.t);
    int restarts = uniform(st.restarts);
    I.levels = uniform(st.levels) != 0;
    I.perm_r = a.S.perm_r + r0;
    I.perm_c = a.S.perm_c + c0;
    inst_load<T, V, BS>(I, a.M, a.S, lds, a.lds, true);
    for (int p = tid; p < m; p += BS) yL[p] = a.ysave[r0 + p];
    __syncthreads();

    typedef RegShape<V> RS;
    const double rho = a.rho, opr = 1.0 + a.rho;
    const int E = a.eval_every;
    const int32_t *arp = a.M.a_rowptr + r0, *trp = a.M.at_rowptr + c0;
    const int64_t t_begin = t;
    int to_eval = (int)(E - t % E);  // iterations up to and with the next evaluation
    if (a.max_iter > t && a.max_iter - t < to_eval) to_eval = (int)(a.max_iter - t);
    bool suspended = false;
    int status = -1;
    while (status < 0) {
        // the iterations that nothing is summed over: all but an epoch's
        // first and the evaluated one
        const int plain = k == 0 ? 0 : to_eval - 1;
        if (plain > 0) {
            plain_iterations<T, V, Acc, BS, LONG>(a, I, lds, plain, k, tau, sig);
            t += plain;
            k += plain;
            to_eval -= plain;
        }
        ++t;
        const bool is_eval = --to_eval <= 0;
        const bool first = (k == 0);
        const double w = a.halpern ? (double)(k + 1) / (double)(k + 2) : 1.0;
        // the primal and the dual step of plain_iterations, with the sums'
        // entries stored by column and row
        const int et = opaque(tid);
        for (int p = et; p < n; p += BS) {
            const int g = c0 + p, j = I.column(p);
            const double u = (double)a.x[g], x0 = (double)a.x0[g], rc = (double)a.ct[g];
            const Acc s = side_dot<LONG, Acc>(I.AT, lds, yL, p, RS::RC * BS, RS::KC);
            double uh = u - tau * (rc - (double)s);
            uh = uh < -x0 ? -x0 : uh;
            xbL[p] = (T)(2.0 * uh - u);
            a.x[g] = (T)(w * (opr * uh - rho * u));
            a.pu[j] = u - uh;
            if (is_eval) {
                a.rdo[j] = uh;
                const double xh = x0 + uh;
                a.xhat[g] = (T)xh;
                a.xo[j] = a.d_col[j] * xh;
            }
        }
        __syncthreads();
        for (int p = et; p < m; p += BS) {
            const int g = r0 + p, i = I.row(p);
            const double rb = (double)a.bt[g];
            const Acc s = side_dot<LONG, Acc>(I.A, lds, xbL, p, RS::RR * BS, RS::KR);
            const double v = (double)yL[p];
            const double vh = v + sig * (rb - (double)s);
            yL[p] = (T)(w * (opr * vh - rho * v));
            a.pav[i] = v - vh;
            if (is_eval) {
                a.rpo[i] = vh;
                const double yh = (double)a.y0[g] + vh;
                a.yhat[g] = (T)yh;
                a.yo[i] = a.d_row[i] * yh;
            }
        }
        __syncthreads();
        double qx[2], qy[2];  // ||u - uh||^2, ||uh||^2 and the same of v
        inst_sums<BS, 2>(n, sh, qx, [&](int j, double(&s)[2]) {
            const double d = a.pu[c0 + j];
            s[0] += d * d;
            if (is_eval) {
                const double e = a.rdo[c0 + j];
                s[1] += e * e;
            }
        });
        inst_sums<BS, 2>(m, sh, qy, [&](int i, double(&s)[2]) {
            const double d = a.pav[r0 + i];
            s[0] += d * d;
            if (is_eval) {
                const double e = a.rpo[r0 + i];
                s[1] += e * e;
            }
        });
        if (first) R0 = uniform(sqrt(omega * qx[0] + qy[0] / omega));
        ++k;
        if (!is_eval) continue;
        const double R = uniform(sqrt(omega * qx[0] + qy[0] / omega));
        // evaluation on the original block, float64
        double rp_inf = 0.0, rd_inf = 0.0;
        for (int i = et; i < m; i += BS) {
            const int g = r0 + i;
            const double rp = a.M.b[g] - row_f64<0>(a.M.a_val, a.M.a_col, a.xo, arp[i], arp[i + 1]);
            a.rpo[g] = rp;
            rp_inf = fmax(rp_inf, fabs(rp));
        }
        for (int j = et; j < n; j += BS) {
            const int g = c0 + j;
            const double gg = a.M.c[g] - row_f64<0>(a.M.at_val, a.M.at_col, a.yo, trp[j], trp[j + 1]);
            const double z = gg > 0.0 ? gg : 0.0;
            const double rd = gg - z;
            a.zo[g] = z;
            a.rdo[g] = rd;
            rd_inf = fmax(rd_inf, fabs(rd));
        }
        rp_inf = inst_max<BS>(rp_inf, sh);
        rd_inf = inst_max<BS>(rd_inf, sh);
        double ep[2], ed[3];
        inst_sums<BS, 2>(m, sh, ep, [&](int i, double(&s)[2]) {
            const double rp = a.rpo[r0 + i];
            s[0] += rp * rp;
            s[1] += a.M.b[r0 + i] * a.yo[r0 + i];
        });
        inst_sums<BS, 3>(n, sh, ed, [&](int j, double(&s)[3]) {
            const double rd = a.rdo[c0 + j], xv = a.xo[c0 + j];
            s[0] += rd * rd;
            s[1] += a.M.c[c0 + j] * xv;
            s[2] += xv * a.zo[c0 + j];
        });
        const double rp = sqrt(ep[0]), rd = sqrt(ed[0]), pobj = ed[1], dobj = ep[1];
        const double gap = fabs(pobj - dobj);
        if (!(isfinite(ep[0]) && isfinite(ed[0]) && isfinite(pobj) && isfinite(dobj))) status = MIPDHG_NUMERICAL;
        else if (rp <= tol_p && rd <= tol_d && gap <= eps * (1.0 + fabs(pobj) + fabs(dobj)))
            status = MIPDHG_OPTIMAL;
        else if (t >= a.max_iter) status = MIPDHG_ITER_LIMIT;
        if (tid == 0) {  // the latest evaluation's measures
            BInst& r = a.info[inst];
            r.rp2 = ep[0];
            r.rd2 = ed[0];
            r.pobj = pobj;
            r.dobj = dobj;
            r.xz = ed[2];
            r.rp_inf = rp_inf;
            r.rd_inf = rd_inf;
        }
        if (status >= 0) break;
        bool restart = false;
        if (a.restarts)
            restart = (R <= a.beta_suff * R0) || (R <= a.beta_nec * R0 && R > R_prev) ||
                      ((double)k >= a.beta_art * (double)t);
        to_eval = E;
        if (a.max_iter - t < to_eval) to_eval = (int)(a.max_iter - t);
        if (restart) {
            const double dx = sqrt(qx[1]), dy = sqrt(qy[1]);
            if (dx > 1e-10 && dy > 1e-10) {
                omega = uniform(exp(a.theta * log(dy / dx) + (1.0 - a.theta) * log(omega)));
                tau = uniform(eta / omega);
                sig = uniform(eta * omega);
            }
            // the anchor moves to (x_hat, y_hat), the state to 0, and the new
            // anchor's residuals are formed in float64 on the caller's
            // matrix: rb = D_r (b - A D_c x0), rc = D_c (c - A^T D_r y0)
            // (pu, pav: D_c x0 and D_r y0)
            for (int p = et; p < n; p += BS) {
                const T v = a.xhat[c0 + p];
                a.x0[c0 + p] = v;
                a.x[c0 + p] = (T)0;
                const int j = I.column(p);
                a.pu[j] = a.d_col[j] * (double)v;
            }
            for (int p = et; p < m; p += BS) {
                const T v = a.yhat[r0 + p];
                a.y0[r0 + p] = v;
                yL[p] = (T)0;
                const int i = I.row(p);
                a.pav[i] = a.d_row[i] * (double)v;
            }
            __syncthreads();
            for (int p = et; p < m; p += BS) {
                const int g = I.row(p), i = g - r0;
                const double sa = row_f64<0>(a.M.a_val, a.M.a_col, a.pu, arp[i], arp[i + 1]);
                a.bt[r0 + p] = (T)(a.d_row[g] * (a.M.b[g] - sa));
            }
            for (int p = et; p < n; p += BS) {
                const int g = I.column(p), j = g - c0;
                const double sa = row_f64<0>(a.M.at_val, a.M.at_col, a.pav, trp[j], trp[j + 1]);
                a.ct[c0 + p] = (T)(a.d_col[g] * (a.M.c[g] - sa));
            }
            k = 0;
            R_prev = INFINITY;
            ++restarts;
            __syncthreads();
        } else {
            R_prev = R;
        }
        // end of this call's block: the state after an evaluation and its
        // restart decision is what the next iteration starts from
        if (a.block_iters > 0 && t - t_begin >= a.block_iters) {
            suspended = true;
            break;
        }
    }
    if (suspended) {
        for (int p = tid; p < m; p += BS) a.ysave[r0 + p] = yL[p];
        status = MIPDHG_IN_PROGRESS;
    }
    if (tid == 0) {
        st.phase = suspended ? 1 : 2;
        st.t = t;
        st.k = k;
        st.omega = omega;
        st.tau = tau;
        st.sig = sig;
        st.R0 = R0;
        st.R_prev = R_prev;
        st.restarts = restarts;
        BInst& r = a.info[inst];
        r.status = status;
        r.restarts = restarts;
        r.iters = t;
        r.omega = omega;
    }
    __syncthreads();
}

// Four waves to a SIMD in every class of launch: at most 128 registers.  The
// set-up is a launch of its own, so that its code takes no registers from the
// iterations.
template <typename T, typename V, typename Acc, int BS, bool SETUP, bool LONG = false>
__global__ __launch_bounds__(BS, 4) void k_batched(BArgs<T, V> a) {
    extern __shared__ __align__(16) unsigned char lds[];
    __shared__ double sh[BS / kWave > 12 ? BS / kWave : 12];
    __shared__ int next;
    while (true) {
        if (threadIdx.x == 0) next = atomicAdd(a.counter + (SETUP ? 0 : kClasses), 1);
        __syncthreads();
        const int qi = __builtin_amdgcn_readfirstlane(next);  // uniform: scalar loads of the offsets
        __syncthreads();
        if (qi >= a.B) break;  // uniform: every wave leaves once the queue is empty
        const int inst = __builtin_amdgcn_readfirstlane(a.order[qi]);
        if constexpr (SETUP) setup_instance<T, V, BS>(a, inst, lds, sh);
        else solve_instance<T, V, Acc, BS, LONG>(a, inst, lds, sh);
        __syncthreads();  // the next instance takes over the LDS
    }
}

__global__ void k_zero_i32(int32_t* p, int n) {
    for (int i = threadIdx.x; i < n; i += blockDim.x) p[i] = 0;
}

struct BatchWs {
    uint64_t* hdr;  // {marker, fingerprint} of the state the workspace holds
    int32_t *order, *row_off, *col_off, *counter, *flags;
    int64_t* nnz_off;
    BInst* info;
    BState* state;
    double *d_row, *d_col, *pu, *pav, *partials, *eps;
    void *a_vs, *at_vs, *x, *x0, *xhat, *ct, *y0, *yhat, *bt, *ysave;
    uint16_t *a_cl, *at_cl, *perm_r, *perm_c;
    size_t bytes;
};

static BatchWs carve_batch(void* base, size_t cap, int64_t B, int64_t m, int64_t n, int64_t nnz, int prec) {
    Carver cv(base, cap);
    BatchWs w;
    const size_t vs = prec == MIPDHG_FP64 ? 8 : (prec == MIPDHG_FP32_BF16A ? 2 : 4);
    const size_t ts = prec == MIPDHG_FP64 ? 8 : 4;
    w.hdr = cv.take<uint64_t>(4);
    w.order = cv.take<int32_t>(B);
    w.row_off = cv.take<int32_t>(B + 1);
    w.col_off = cv.take<int32_t>(B + 1);
    w.counter = cv.take<int32_t>(64);
    w.flags = cv.take<int32_t>(64);
    w.nnz_off = cv.take<int64_t>(B + 1);
    w.info = cv.take<BInst>(B);
    w.state = cv.take<BState>(B);
    w.eps = cv.take<double>(B);
    w.d_row = cv.take<double>(m);
    w.d_col = cv.take<double>(n);
    w.pu = cv.take<double>(n);
    w.pav = cv.take<double>(m);
    w.partials = cv.take<double>(4 * kCheckGrid);
    w.a_vs = cv.take<char>(nnz * vs);
    w.at_vs = cv.take<char>(nnz * vs);
    w.a_cl = cv.take<uint16_t>(nnz);
    w.at_cl = cv.take<uint16_t>(nnz);
    w.perm_r = cv.take<uint16_t>(m);
    w.perm_c = cv.take<uint16_t>(n);
    w.x = cv.take<char>(n * ts);
    w.x0 = cv.take<char>(n * ts);
    w.xhat = cv.take<char>(n * ts);
    w.ct = cv.take<char>(n * ts);
    w.y0 = cv.take<char>(m * ts);
    w.yhat = cv.take<char>(m * ts);
    w.bt = cv.take<char>(m * ts);
    w.ysave = cv.take<char>(m * ts);
    w.bytes = (cv.off + 255) & ~size_t(255);
    return w;
}

// Identity of a batched solve's state in its workspace: the batch's sizes
// and offsets and every option the iterations depend on (not eps_rel,
// max_iter, batch_block_iters, validate or resume).  FNV-1a over the fields.
static uint64_t batch_fingerprint(const mipdhg_batch& bt, const mipdhg_options& o) {
    uint64_t h = 1469598103934665603ull;
    auto mix = [&](const void* p, size_t nb) {
        const unsigned char* c = (const unsigned char*)p;
        for (size_t i = 0; i < nb; ++i) h = (h ^ c[i]) * 1099511628211ull;
    };
    const int64_t sz[4] = {bt.count, bt.whole.m, bt.whole.n, bt.whole.nnz};
    mix(sz, sizeof(sz));
    mix(bt.row_off, ((size_t)bt.count + 1) * sizeof(int32_t));
    mix(bt.col_off, ((size_t)bt.count + 1) * sizeof(int32_t));
    mix(bt.nnz_off, ((size_t)bt.count + 1) * sizeof(int64_t));
    const int32_t iv[8] = {o.precision, o.ruiz_iters, o.pock_chambolle, o.power_iters,
                           o.eval_every, o.halpern, o.restarts, o.batch_split};
    mix(iv, sizeof(iv));
    const double dv[6] = {o.step_safety, o.reflect_rho, o.beta_suff, o.beta_nec, o.beta_art, o.pw_theta};
    mix(dv, sizeof(dv));
    return h;
}

// What the header says of the state's layout: another value for each (this one
// has the vectors by position, with the positions kept; a workspace that was
// kept from a library with another layout is refused)
constexpr uint64_t kBatchStateMarker = 0x6d69706468672d63ull;

static int check_batch(const mipdhg_batch* bt) {
    if (!bt) return set_error("batch is NULL"), MIPDHG_ERR_INVALID_ARG;
    if (bt->count < 1) return set_error("batch count must be >= 1"), MIPDHG_ERR_INVALID_ARG;
    if (!bt->row_off || !bt->col_off || !bt->nnz_off)
        return set_error("row_off, col_off and nnz_off are required"), MIPDHG_ERR_INVALID_ARG;
    int rc = check_lp(&bt->whole);
    if (rc) return rc;
    const int B = bt->count;
    if (bt->row_off[0] != 0 || bt->col_off[0] != 0 || bt->nnz_off[0] != 0 || bt->row_off[B] != bt->whole.m ||
        bt->col_off[B] != bt->whole.n || bt->nnz_off[B] != bt->whole.nnz)
        return set_error("instance offsets must start at 0 and end at m, n, nnz"), MIPDHG_ERR_INVALID_ARG;
    for (int i = 0; i < B; ++i)
        if (bt->row_off[i + 1] <= bt->row_off[i] || bt->col_off[i + 1] <= bt->col_off[i] ||
            bt->nnz_off[i + 1] < bt->nnz_off[i])
            return set_error("instance %d is empty or its offsets decrease", i), MIPDHG_ERR_INVALID_ARG;
    return 0;
}

static int lds_bytes_for(int max_m, int max_n, size_t ts) {
    return (int)(((size_t)max_m + (size_t)max_n) * ts + 16);
}

// Launch classes: workgroups of kClassBs threads.  An instance's results do
// not depend on its class.  With more instances than compute units the class
// follows from the LDS the instance needs with both matrices in it, so that
// every class keeps 16 waves on a compute unit: up to a sixteenth of its LDS
// one wave (but see one_wave), up to a quarter 256 threads, up to a half 512,
// else 1,024 threads and the whole LDS, from which the matrices' last levels
// are left out when they do not fit.  With no more instances than compute
// units nothing is gained by leaving room for others: about one thread per
// column (a thread holds three).  48 LPs, 256 iterations, FP32: at 62 columns 64
// threads 0.95 ms, 256 0.92; at 80 1.04 and 0.92; at 255 256 threads 1.01, 512
// 1.01; at 400 1.24 and 1.15; at 900 512 threads 1.40, 1,024 1.42; at 1,300 1.88 and
// 1.58.
// Measured on 4,096 LPs of 20 to 2,000 rows, 2.5 times the columns, 4 entries
// a column (FP32, 256 iterations, call with its host part): one launch of 256
// threads sized by the largest instance, the matrices in L2, 32.3 ms; these
// classes 22.9 ms (15.7 ms with the inputs checked on the device).  48 LPs of
// 20 to 500 rows in FP64: 256 threads each 2.37 ms, by the columns 1.56 ms
// (1.46 ms).
constexpr int kClassBs[kClasses] = {1024, 512, 256, 64};
constexpr int kClassLds[kClasses] = {162000, 81000, 40400, 9700};  // shares of 160 KB, less the static part

// Whether work on other streams may use the compute units that work on this
// one may (a stream can be made with a mask of them)
static bool unmasked(hipStream_t s) {
    if (!s) return true;
    uint32_t own[64] = {}, all[64] = {};
    if (hipExtStreamGetCUMask(s, 64, own) != hipSuccess || hipExtStreamGetCUMask(nullptr, 64, all) != hipSuccess) {
        (void)hipGetLastError();
        return false;
    }
    return memcmp(own, all, sizeof(own)) == 0;
}

// One class's launches: as many workgroups as fit, never more than instances
template <typename T, typename V, typename Acc, int BS>
static int launch_class(const BArgs<T, V>& a, bool rests, int cus, hipStream_t s) {
    auto* ks = k_batched<T, V, Acc, BS, true>;
    auto* k = rests ? k_batched<T, V, Acc, BS, false, LongRows<V>::ok> : k_batched<T, V, Acc, BS, false, false>;
    // (the largest class's bytes whatever this launch's: the attribute is the process's)
    MIP_HIP(hipFuncSetAttribute((const void*)ks, hipFuncAttributeMaxDynamicSharedMemorySize, kClassLds[0]));
    MIP_HIP(hipFuncSetAttribute((const void*)k, hipFuncAttributeMaxDynamicSharedMemorySize, kClassLds[0]));
    int per_cu = 1;
    MIP_HIP(hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, k, BS, a.lds));
    const int grid = std::max(1, std::min(a.B, cus * std::max(per_cu, 1)));
    if (!a.resume) hipLaunchKernelGGL(ks, dim3(grid), dim3(BS), a.lds, s, a);
    hipLaunchKernelGGL(k, dim3(grid), dim3(BS), a.lds, s, a);
    MIP_LAUNCH_CHECK();
    return 0;
}

template <typename T, typename V, typename Acc>
static int batched_impl(const mipdhg_batch& bt, const mipdhg_options& o, const double* eps, void* ws, size_t ws_bytes,
                        hipStream_t stream, double* x, double* y, double* z, double* r_p, double* r_d,
                        mipdhg_info* info) {
    using clk = std::chrono::steady_clock;
    const auto t0 = clk::now();
    const mipdhg_lp& lp = bt.whole;
    const int B = bt.count;
    BatchWs w = carve_batch(ws, ws_bytes, B, lp.m, lp.n, lp.nnz, o.precision);
    if (w.bytes > ws_bytes)
        return set_error("workspace too small: %zu bytes given, %zu needed", ws_bytes, w.bytes), MIPDHG_ERR_WORKSPACE;
    if (((uintptr_t)ws & 255) != 0) return set_error("workspace must be 256-byte aligned"), MIPDHG_ERR_INVALID_ARG;
    // a resume continues only the state of this batch under these options;
    // the header is invalid while a call runs and valid once it returns
    const uint64_t fp = batch_fingerprint(bt, o);
    uint64_t hdr_in[2] = {0, 0};
    const uint64_t hdr_running[2] = {0, 0}, hdr_done[2] = {kBatchStateMarker, fp};
    if (o.resume) {
        MIP_HIP(hipMemcpyAsync(hdr_in, w.hdr, sizeof(hdr_in), hipMemcpyDeviceToHost, stream));
        MIP_HIP(hipStreamSynchronize(stream));
        if (hdr_in[0] != kBatchStateMarker || hdr_in[1] != fp)
            return set_error("resume: the workspace does not hold the state of this batch with these options"),
                   MIPDHG_ERR_INVALID_ARG;
    }
    int max_m = 0, max_n = 0;
    for (int i = 0; i < B; ++i) {
        max_m = std::max(max_m, bt.row_off[i + 1] - bt.row_off[i]);
        max_n = std::max(max_n, bt.col_off[i + 1] - bt.col_off[i]);
    }
    const int lds = lds_bytes_for(max_m, max_n, sizeof(T));
    if (lds > 150 * 1024 || max_m > kInstMaxDim || max_n > kInstMaxDim)
        return set_error("largest instance needs %d bytes of LDS (limit 150 KiB): m + n too large", lds),
               MIPDHG_ERR_UNSUPPORTED;
    StreamDrain drain{stream};
    int dev = 0, cus = 256;
    MIP_HIP(hipGetDevice(&dev));
    MIP_HIP(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev));
    // the classes' instances one after the other in the order array, each
    // class largest first; batch_split sends the instances whose vectors fit
    // its bytes to 256 threads and the others to 1,024
    std::vector<uint8_t> cls(B);
    int cl_count[kClasses] = {0, 0, 0, 0}, cl_lds[kClasses] = {0, 0, 0, 0};
    int64_t cl_m[kClasses] = {}, cl_nnz[kClasses] = {};
    auto rows = [&](int i) { return bt.row_off[i + 1] - bt.row_off[i]; };
    auto columns = [&](int i) { return bt.col_off[i + 1] - bt.col_off[i]; };
    auto full = [&](int i, int k) {  // LDS that holds all of it beside the registers of class k's threads
        typedef RegShape<V> RS;
        const int mi = rows(i), ni = columns(i);
        const int64_t zi = bt.nnz_off[i + 1] - bt.nnz_off[i], zc = zi / std::max(ni, 1), zr = zi / std::max(mi, 1);
        const int64_t nreg = std::min(ni, RS::RC * kClassBs[k]) * std::min<int64_t>(zc, RS::KC) +
                             std::min(mi, RS::RR * kClassBs[k]) * std::min<int64_t>(zr, RS::KR);
        return inst_full_bytes(mi, ni, zi, sizeof(T), sizeof(V), nreg);
    };
    int quarter = 0;  // instances that a quarter of a compute unit's LDS holds
    for (int i = 0; i < B; ++i) {
        const int ni = columns(i);
        int c;
        if (o.batch_split > 0) c = lds_bytes_for(rows(i), ni, sizeof(T)) <= o.batch_split ? 2 : 0;
        else if (B <= cus) c = std::max(rows(i), ni) <= 64 ? 3 : ni <= 256 ? 2 : ni <= 1024 ? 1 : 0;
        else c = full(i, 3) <= kClassLds[3] ? 3 : full(i, 2) <= kClassLds[2] ? 2 : full(i, 1) <= kClassLds[1] ? 1 : 0;
        quarter += c >= 2;
        cls[i] = (uint8_t)c;
    }
    for (int i = 0; i < B; ++i) {
        if (cls[i] == 3 && !one_wave(quarter, cus, rows(i), columns(i))) cls[i] = 2;
        const int c = cls[i];
        const int64_t cap = B <= cus && o.batch_split == 0 ? kClassLds[0] : kClassLds[c];
        const int need = (int)std::max<int64_t>(inst_vec_bytes(rows(i), columns(i), sizeof(T)), std::min(full(i, c), cap));
        ++cl_count[c];
        cl_m[c] += rows(i);
        cl_nnz[c] += bt.nnz_off[i + 1] - bt.nnz_off[i];
        cl_lds[c] = std::max(cl_lds[c], need);
    }
    std::vector<int32_t> order(B);
    std::iota(order.begin(), order.end(), 0);
    std::stable_sort(order.begin(), order.end(), [&](int p, int q) {
        if (cls[p] != cls[q]) return cls[p] < cls[q];
        return bt.nnz_off[p + 1] - bt.nnz_off[p] > bt.nnz_off[q + 1] - bt.nnz_off[q];
    });
    MIP_HIP(hipMemcpyAsync(w.hdr, hdr_running, sizeof(hdr_running), hipMemcpyHostToDevice, stream));
    MIP_HIP(hipMemcpyAsync(w.order, order.data(), B * 4, hipMemcpyHostToDevice, stream));
    MIP_HIP(hipMemcpyAsync(w.row_off, bt.row_off, (B + 1) * 4, hipMemcpyHostToDevice, stream));
    MIP_HIP(hipMemcpyAsync(w.eps, eps, (size_t)B * 8, hipMemcpyHostToDevice, stream));
    MIP_HIP(hipMemcpyAsync(w.col_off, bt.col_off, (B + 1) * 4, hipMemcpyHostToDevice, stream));
    // the row pointers against the instance offsets and, unless this resumes
    // a validated call's state, the entries
    if (int rc = check_blocks(bt, o.validate && !o.resume, w.row_off, w.col_off, w.nnz_off, w.flags, w.partials, stream))
        return rc;
    BArgs<T, V> a;
    a.B = B;
    a.lds = 0;
    a.order = w.order;
    a.row_off = w.row_off;
    a.col_off = w.col_off;
    a.M = InstMat{lp.a_rowptr, lp.a_col, lp.a_val, lp.at_rowptr, lp.at_col, lp.at_val, lp.b, lp.c};
    a.S = InstStore<V>{(V*)w.a_vs, (V*)w.at_vs, w.a_cl, w.at_cl, w.perm_r, w.perm_c};
    a.x = (T*)w.x;
    a.x0 = (T*)w.x0;
    a.xhat = (T*)w.xhat;
    a.ct = (T*)w.ct;
    a.y0 = (T*)w.y0;
    a.yhat = (T*)w.yhat;
    a.bt = (T*)w.bt;
    a.d_row = w.d_row;
    a.d_col = w.d_col;
    a.pu = w.pu;
    a.pav = w.pav;
    a.xo = x;
    a.yo = y;
    a.zo = z;
    a.rpo = r_p;
    a.rdo = r_d;
    a.info = w.info;
    a.state = w.state;
    a.ysave = (T*)w.ysave;
    a.resume = o.resume;
    a.block_iters = o.batch_block_iters;
    a.counter = w.counter;
    a.eps = w.eps;
    a.step_safety = o.step_safety;
    a.rho = o.reflect_rho;
    a.beta_suff = o.beta_suff;
    a.beta_nec = o.beta_nec;
    a.beta_art = o.beta_art;
    a.theta = o.pw_theta;
    a.max_iter = o.max_iter;
    a.ruiz = o.ruiz_iters;
    a.pc = o.pock_chambolle;
    a.power_iters = o.power_iters;
    a.eval_every = o.eval_every;
    a.halpern = o.halpern;
    a.restarts = o.restarts;
    // one persistent launch per class with instances, all at once: the first
    // on the caller's stream, the others on side streams joined to it
    // (neither waits on another; each takes the compute units the others
    // leave); one after the other where the caller's stream is held to some of
    // the compute units
    struct Sides {
        hipStream_t s[kClasses] = {};
        hipEvent_t fork = nullptr, join[kClasses] = {};
        hipEvent_t e0 = nullptr, e1 = nullptr;
        ~Sides() {
            for (int c = 0; c < kClasses; ++c) {
                if (s[c]) {
                    (void)hipStreamSynchronize(s[c]);
                    (void)hipStreamDestroy(s[c]);
                }
                if (join[c]) (void)hipEventDestroy(join[c]);
            }
            if (fork) (void)hipEventDestroy(fork);
            if (e0) (void)hipEventDestroy(e0);
            if (e1) (void)hipEventDestroy(e1);
        }
    } side;
    hipLaunchKernelGGL(k_zero_i32, dim3(1), dim3(64), 0, stream, w.counter, 64);
    const auto t1 = clk::now();
    MIP_HIP(hipEventCreate(&side.e0));
    MIP_HIP(hipEventCreate(&side.e1));
    const hipEvent_t e0 = side.e0, e1 = side.e1;
    MIP_HIP(hipEventRecord(e0, stream));
    const bool spread = unmasked(stream);
    int first = -1, begin = 0;
    for (int c = 0; c < kClasses; ++c) {
        if (!cl_count[c]) continue;
        hipStream_t cs = stream;
        if (first < 0) {
            first = c;
            if (spread && cl_count[c] < B) {
                MIP_HIP(hipEventCreateWithFlags(&side.fork, hipEventDisableTiming));
                MIP_HIP(hipEventRecord(side.fork, stream));
            }
        } else if (spread) {
            MIP_HIP(hipStreamCreateWithFlags(&side.s[c], hipStreamNonBlocking));
            MIP_HIP(hipEventCreateWithFlags(&side.join[c], hipEventDisableTiming));
            cs = side.s[c];
            MIP_HIP(hipStreamWaitEvent(cs, side.fork, 0));
        }
        BArgs<T, V> ac = a;
        ac.B = cl_count[c];
        ac.order = w.order + begin;
        ac.counter = w.counter + c;
        ac.lds = cl_lds[c];
        begin += cl_count[c];
        const bool rests = LongRows<V>::pays(cl_m[c], cl_nnz[c]);
        int rc;
        if (c == 0) rc = launch_class<T, V, Acc, kClassBs[0]>(ac, rests, cus, cs);
        else if (c == 1) rc = launch_class<T, V, Acc, kClassBs[1]>(ac, rests, cus, cs);
        else if (c == 2) rc = launch_class<T, V, Acc, kClassBs[2]>(ac, rests, cus, cs);
        else rc = launch_class<T, V, Acc, kClassBs[3]>(ac, rests, cus, cs);
        if (rc) return rc;
    }
    for (int c = 0; c < kClasses; ++c)
        if (side.s[c]) {
            MIP_HIP(hipEventRecord(side.join[c], side.s[c]));
            MIP_HIP(hipStreamWaitEvent(stream, side.join[c], 0));
        }
    MIP_HIP(hipEventRecord(e1, stream));
    MIP_HIP(hipMemcpyAsync(w.hdr, hdr_done, sizeof(hdr_done), hipMemcpyHostToDevice, stream));
    std::vector<BInst> res(B);
    MIP_HIP(hipMemcpyAsync(res.data(), w.info, sizeof(BInst) * B, hipMemcpyDeviceToHost, stream));
    MIP_HIP(hipStreamSynchronize(stream));
    drain.armed = false;
    float kms = 0.f;
    MIP_HIP(hipEventElapsedTime(&kms, e0, e1));
    const auto t2 = clk::now();
    int worst = MIPDHG_OPTIMAL;
    for (int i = 0; i < B; ++i) worst = std::max(worst, res[i].status);
    if (info) {
        for (int i = 0; i < B; ++i) {
            const BInst& r = res[i];
            mipdhg_info& f = info[i];
            memset(&f, 0, sizeof(f));
            f.status = r.status;
            f.restarts = r.restarts;
            f.iters = r.iters;
            f.rp_norm = sqrt(r.rp2);
            f.rd_norm = sqrt(r.rd2);
            f.pobj = r.pobj;
            f.dobj = r.dobj;
            f.gap = fabs(r.pobj - r.dobj);
            f.b_norm = r.b_norm;
            f.c_norm = r.c_norm;
            f.rel_rp = f.rp_norm / (1.0 + r.b_norm);
            f.rel_rd = f.rd_norm / (1.0 + r.c_norm);
            f.rel_gap = f.gap / (1.0 + fabs(r.pobj) + fabs(r.dobj));
            f.rp_inf = r.rp_inf;
            f.rd_inf = r.rd_inf;
            f.xz = r.xz;
            f.max_violation = std::max(std::max(r.rp_inf, r.rd_inf), r.xz / (1.0 + fabs(r.pobj)));
            f.sigma_hat = r.sigma_hat;
            f.eta = r.eta;
            f.omega0 = r.omega0;
            f.omega = r.omega;
            f.ms_setup = std::chrono::duration<double, std::milli>(t1 - t0).count();
            f.ms_iter = kms;
            f.ms_total = std::chrono::duration<double, std::milli>(t2 - t0).count();
        }
    }
    return worst;
}

}  // namespace mip

using namespace mip;

extern "C" int mipdhg_batch_workspace_size(const mipdhg_batch* bt, const mipdhg_options* opt, size_t* bytes) {
    clear_error();
    if (!bytes || !opt) return set_error("NULL argument"), MIPDHG_ERR_INVALID_ARG;
    int rc = check_batch(bt);
    if (rc) return rc;
    if ((rc = check_options(opt))) return rc;
    *bytes = carve_batch(nullptr, 0, bt->count, bt->whole.m, bt->whole.n, bt->whole.nnz, opt->precision).bytes;
    return 0;
}

extern "C" int mipdhg_solve_batched(const mipdhg_batch* bt, const mipdhg_options* opt, const double* eps_rel,
                                    void* workspace, size_t workspace_bytes, void* stream, double* x, double* y,
                                    double* z, double* r_p, double* r_d, mipdhg_info* info) {
    clear_error();
    int rc = check_batch(bt);
    if (rc) return rc;
    if (!opt) return set_error("options are NULL"), MIPDHG_ERR_INVALID_ARG;
    if ((rc = check_options(opt))) return rc;
    if (!eps_rel) return set_error("eps_rel (one per instance) is NULL"), MIPDHG_ERR_INVALID_ARG;
    for (int i = 0; i < bt->count; ++i)
        if (!(eps_rel[i] >= 0.0) || !std::isfinite(eps_rel[i]))
            return set_error("eps_rel[%d] must be finite and >= 0", i), MIPDHG_ERR_INVALID_ARG;
    if (!workspace || !x || !y || !z || !r_p || !r_d)
        return set_error("workspace and all five outputs are required"), MIPDHG_ERR_INVALID_ARG;
    if (is_general(bt->whole))
        return set_error("the general form (bounds, inequality rows) is a single-LP option"), MIPDHG_ERR_UNSUPPORTED;
    if (opt->pw_ki != 0.0 || opt->pw_kd != 0.0 || opt->restart_avg || opt->step_rule)
        return set_error("the PID primal weight, restart to average and the adaptive step are single-LP options"),
               MIPDHG_ERR_UNSUPPORTED;
    if (opt->trace_iters || opt->x_init || opt->y_init || opt->kernel_timing)
        return set_error("tracing, warm starts and kernel timing are single-LP options"), MIPDHG_ERR_UNSUPPORTED;
    if (opt->precision == MIPDHG_FP32_A)
        return set_error("FP32_A is a single-LP precision mode"), MIPDHG_ERR_UNSUPPORTED;
    hipStream_t s = (hipStream_t)stream;
    switch (opt->precision) {
        case MIPDHG_FP64:
            return batched_impl<double, double, double>(*bt, *opt, eps_rel, workspace, workspace_bytes, s, x, y, z,
                                                        r_p, r_d, info);
        case MIPDHG_FP32:
            return batched_impl<float, float, double>(*bt, *opt, eps_rel, workspace, workspace_bytes, s, x, y, z, r_p,
                                                      r_d, info);
        case MIPDHG_FP32_BF16A:
            return batched_impl<float, uint16_t, double>(*bt, *opt, eps_rel, workspace, workspace_bytes, s, x, y, z,
                                                         r_p, r_d, info);
        default:
            return batched_impl<float, float, float>(*bt, *opt, eps_rel, workspace, workspace_bytes, s, x, y, z, r_p,
                                                     r_d, info);
    }
}

extern "C" int mipdhg_autotune_batched(const mipdhg_batch* bt, mipdhg_options* opt, const double* eps_rel,
                                       void* workspace, size_t workspace_bytes, void* stream, double* x, double* y,
                                       double* z, double* r_p, double* r_d, double* best_ms) {
    clear_error();
    int rc = check_batch(bt);
    if (rc) return rc;
    if (!opt) return set_error("options are NULL"), MIPDHG_ERR_INVALID_ARG;
    std::vector<mipdhg_info> info((size_t)bt->count);
    // LDS budgets of the narrow launch (0: one launch); the default stays
    // unless another is more than 3 % faster, so that the choice is stable
    const int32_t cands[] = {0, 2048, 4096, 8192, 16384, 32768};
    double best = 1e300, def = 1e300;
    int32_t pick = 0;
    for (int32_t c : cands) {
        mipdhg_options o = *opt;
        o.batch_split = c;
        o.resume = 0;  // whole solves from the start
        o.batch_block_iters = 0;
        const int r = mipdhg_solve_batched(bt, &o, eps_rel, workspace, workspace_bytes, stream, x, y, z, r_p, r_d,
                                           info.data());
        if (r < 0) return r;
        const double ms = info[0].ms_iter;  // the launches, timed by events on the stream
        if (c == 0) def = ms;
        if (ms < best) {
            best = ms;
            pick = c;
        }
    }
    if (best * 1.03 >= def) {
        pick = 0;
        best = def;
    }
    opt->batch_split = pick;
    if (best_ms) *best_ms = best;
    return 0;
}
