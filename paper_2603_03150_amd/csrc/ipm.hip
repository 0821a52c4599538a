// Interior-point consumer of the centered start (Section 3.1): the solver
// Algorithm 1 hands its point to, and the alpha_min recovery loop around it.
//
// Mehrotra's primal-dual predictor-corrector (Wright 1997, Chapter 10) on the
// scaled LP min c~^T x s.t. A~ x = b~, x >= 0 with A~ = D_r A D_c, b~ = D_r b,
// c~ = D_c c.  Every Newton system goes through the normal equations
// (A~ D A~^T) dy = r_b - A~ (Z^-1 r_xz - D r_c), D = X Z^-1: the m x m matrix
// is formed dense on the device (a wave per row, accumulated in LDS in a fixed
// order), factored by a blocked right-looking Cholesky on FP64 MFMAs (64 x 64
// blocks, one launch per block column), and each of the two triangular solves
// is one launch, a workgroup per 64 rows.
// The predictor and the corrector share the factor.  Scalars (norms, step
// lengths, mu) are fixed-order reductions read back by the host, which runs
// the iteration.  Dense factors bound m (kIpmMaxM): this consumer is for the
// modest LPs on which the paper's iteration-count ratio is measured, not for
// the large sparse models of Section 4, which need a sparse factorization.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <chrono>
#include <cmath>
#include <cstring>
#include <vector>

#include "common.h"
#include "mipdhg.h"
#include "plain.h"

namespace mip {
namespace {

constexpr int kNb = 64;           // Cholesky block
constexpr int kIpmMaxM = 16384;   // dense normal matrix: 2 GiB at this size
constexpr int kRedBlocks = 1024;  // partial slots of a reduction

// out[r] = (s0 ? s0[r] : 0) + sgn * sum_k a_rk v[col_k] - (s1 ? s1[r] : 0);
// one wave per row, the lanes' strided sums added by a butterfly
__global__ __launch_bounds__(kBlock) void k_ipm_spmv(const int32_t* rp, const int32_t* col, const double* val,
                                                     const double* v, int32_t nrows, const double* s0, double sgn,
                                                     const double* s1, double* out) {
    const int lane = threadIdx.x & (kWave - 1);
    const int64_t r = (int64_t)blockIdx.x * (kBlock / kWave) + threadIdx.x / kWave;
    if (r >= nrows) return;
    double acc = 0.0;
    for (int k = rp[r] + lane; k < rp[r + 1]; k += kWave) acc += val[k] * v[col[k]];
#pragma unroll
    for (int o = kWave / 2; o > 0; o >>= 1) acc += __shfl_xor(acc, o, kWave);
    if (lane == 0) out[r] = (s0 ? s0[r] : 0.0) + sgn * acc - (s1 ? s1[r] : 0.0);
}

// scaled values (d_row[i] a_ij) d_col[j] of A
// (a wave to a row: with one thread its longest row's entries came one after
// the other, 93 us on 1,000 x 4,000 and 203 us on 4,000 x 16,000 power-law LPs;
// so 4.8 and 9.8 us (the mean of A's and A^T's))
__global__ void k_ipm_scale_vals(const int32_t* rp, const int32_t* col, const double* val, int32_t nrows,
                                 const double* d_row, const double* d_col, double* out) {
    const int lane = threadIdx.x & (kWave - 1);
    const int64_t waves = (int64_t)gridDim.x * blockDim.x / kWave;
    for (int64_t r = (blockIdx.x * (int64_t)blockDim.x + threadIdx.x) / kWave; r < nrows; r += waves)
        for (int k = rp[r] + lane; k < rp[r + 1]; k += kWave) {
            const int32_t c = col[k];
            const double dr = d_row ? d_row[r] : 1.0, dc = d_col ? d_col[c] : 1.0;
            out[k] = (dr * val[k]) * dc;
        }
}

// out = d .* v (either may be NULL for ones), or v / d (div)
__global__ void k_ipm_vscale(const double* v, const double* d, int div, int64_t n, double* out) {
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
        const double s = d ? d[i] : 1.0;
        out[i] = div ? v[i] / s : v[i] * s;
    }
}

// What an infinite diagonal entry of M is stored as: an infinity among the B
// operands of the factorization's products makes a NaN of every zero that it
// meets.  Its row and column of the inverted factor, and with them the column of
// the factor, are made zero, what the division by an infinite pivot gives: the
// row decouples.
constexpr double kInfPivot = 1.79769313486231570e308;

// Lower triangle of M = A~ diag(w) A~^T (w NULL: ones), a workgroup of one
// wave per row i: the row is accumulated in LDS, column after column of A's
// row i in its order, the lanes over the entries of that column (a row of
// A~^T, whose rows k are distinct: the set-up has checked it).  Every entry
// (i, k) is the sum over the common columns of i and k in increasing order,
// whatever the launch.  Rows from m on (the padding up to ld) are those of the
// identity.
// What bounds it: the loads of a column's entries, a chain of two; four
// columns' loads are in flight together.  27 us at 1,000 x 4,000 (32,000
// nonzeros) and 150 us at 4,000 x 16,000 (128,000); one thread per entry
// merging the two sorted rows, the form before, walked both rows for every
// pair, mostly without a common column: 131 us and 2.0 ms.
__global__ __launch_bounds__(kWave) void k_ipm_normal(const int32_t* rp, const int32_t* col, const double* val,
                                                      const int32_t* trp, const int32_t* tcol, const double* tval,
                                                      const double* w, int32_t m, int32_t ld, double* M) {
    extern __shared__ __align__(16) double row[];
    const int lane = threadIdx.x;
    const int i = ld - 1 - (int)blockIdx.x;  // the longest rows of the triangle first
    for (int k = lane; k <= i; k += kWave) row[k] = (i >= m && k == i) ? 1.0 : 0.0;
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    const int p0 = i < m ? rp[i] : 0, p1 = i < m ? rp[i + 1] : 0;
    for (int base = p0; base < p1; base += kWave) {
        // lane l: column base + l of the row, its weighted value and its range in A~^T
        const int nc = min(kWave, p1 - base);
        double v = 0.0;
        int ts = 0, te = 0;
        if (lane < nc) {
            const int c = col[base + lane];
            v = val[base + lane] * (w ? w[c] : 1.0);
            ts = trp[c];
            te = trp[c + 1];
        }
        for (int q = 0; q < nc; q += 4) {
            int s[4], e[4], k[4];
            double vv[4], tv[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                s[u] = q + u < nc ? __shfl(ts, q + u, kWave) : 0;
                e[u] = q + u < nc ? __shfl(te, q + u, kWave) : 0;
                vv[u] = __shfl(v, (q + u) & (kWave - 1), kWave);
                k[u] = s[u] + lane < e[u] ? tcol[s[u] + lane] : -1;
                tv[u] = s[u] + lane < e[u] ? tval[s[u] + lane] : 0.0;
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                if (k[u] >= 0 && k[u] <= i) row[k[u]] += vv[u] * tv[u];
                for (int t = s[u] + kWave + lane; t < e[u]; t += kWave) {  // columns of more than 64 entries
                    const int kk = tcol[t];
                    if (kk >= 0 && kk <= i) row[kk] += vv[u] * tval[t];
                }
                __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
                __builtin_amdgcn_wave_barrier();  // the next column's entries may be other lanes'
                __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
            }
        }
    }
    for (int k = lane; k <= i; k += kWave) M[(int64_t)i * ld + k] = k == i && row[k] > kInfPivot ? kInfPivot : row[k];
}

// --- blocked Cholesky, lower triangle of a row-major ld x ld matrix in place,
// ld a multiple of 64 (rows and columns from m on are the identity's).  A
// pivot that is not positive (or underflows) is replaced by 1e128, which
// decouples that row (the usual treatment of a rank-deficient normal matrix);
// such replacements are counted in *flag.
//
// One launch per 64-column block s.  Every workgroup of the launch needs the
// panel of block s - 1 only, so the launches are the only synchronisation:
//  - the first nbk - s workgroups take the 64 x 64 blocks (i, s), i >= s:
//    panel s - 1 is applied to the block and, by each of them again, to the
//    diagonal block, which each factors for itself (a launch of its own would
//    cost a trip through memory more) and solves its rows with; (s, s) itself
//    stores the inverse of its factor, which the triangular solves use, and
//    L(s, s) is not stored;
//  - the others apply panel s - 1 to the blocks right of column s.
// The products are 16 x 16 x 4 FP64 MFMAs: a lane holds A[l % 16][l / 16],
// B[l / 16][l % 16] and, in register r, C[l / 16 + 4 r][l % 16], so a C block
// is its own B operand of the next product, and the row solves
// X^T <- L^-1 X^T keep X^T in registers throughout.
// What bounds it: the diagonal factors, a chain of 64 pivots and more than half
// of a launch, the rest the panel's loads and products before them and the row
// solve after; at m = 4,000 also the trailing update, which reads and writes
// 128 MB in the first launches.  A launch takes 21.5 us at m = 1,000 (27.8 us
// mean at 4,000), a factorization 0.34 and 1.75 ms.  The
// form before (a diagonal, a panel and an update launch per block, on vector
// FMAs, the diagonal one column at a time through LDS) took 2.2 and 10.2 ms.
// Measured beside it: the pivots of a block eliminated by lane reads in a row
// per lane, 24.6 us a launch; four pivots at a time through a 4 x 4 inverse,
// 25.1; the whole 64 x 64 factor by one wave, 25.5.
typedef double d4 __attribute__((ext_vector_type(4)));
typedef double d2 __attribute__((ext_vector_type(2)));
constexpr int kCholBlock = 320;  // 5 waves: one factors while four update
constexpr int kLs = kNb + 2;     // LDS row stride (doubles): fragments fall on distinct banks
constexpr int kTs = 18;          // the same for the 16 x 16 transposition

__device__ __forceinline__ d4 mfma16(double a, double b, d4 c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}

__device__ __forceinline__ double readlane_f64(double v, int l) {
    union {
        double d;
        int i[2];
    } u;
    u.d = v;
    u.i[0] = __builtin_amdgcn_readlane(u.i[0], l);
    u.i[1] = __builtin_amdgcn_readlane(u.i[1], l);
    return u.d;
}

// 1 / d for a finite positive d, to rounding: the hardware estimate and one
// third-order step (a shorter chain than the division's scaling)
__device__ __forceinline__ double recip(double d) {
    const double x = __builtin_amdgcn_rcp(d);
    const double e = fma(-d, x, 1.0);
    return fma(x, fma(e, e, e), x);
}

// A 64 x 64 block of M to LDS, rows of kLs doubles
__device__ __forceinline__ void block_to_lds(const double* src, int64_t ld, double* dst, int nthreads) {
    for (int e = threadIdx.x; e < kNb * kNb / 2; e += nthreads) {
        const int r = e / (kNb / 2), c = 2 * (e % (kNb / 2));
        *(d2*)(dst + r * kLs + c) = *(const d2*)(src + r * ld + c);
    }
}

// 1 / sqrt(d) for a finite positive d, to rounding
__device__ __forceinline__ double recip_sqrt(double d) {
    const double y = __builtin_amdgcn_rsq(d);
    const double e = fma(-d * y, y, 1.0);
    return fma(y * e, fma(0.375, e, 0.5), y);
}

// LDS writes of a wave before, reads after
__device__ __forceinline__ void wave_lds_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// a 16 x 16 block's four registers of every lane, [register][lane]
__device__ __forceinline__ d4 load_frag(const double* B, int t) {
    d4 v;
#pragma unroll
    for (int r = 0; r < 4; ++r) v[r] = B[t * 256 + r * 64 + (threadIdx.x & (kWave - 1))];
    return v;
}
__device__ __forceinline__ void store_frag(double* B, int t, d4 v) {
#pragma unroll
    for (int r = 0; r < 4; ++r) B[t * 256 + r * 64 + (threadIdx.x & (kWave - 1))] = v[r];
}

constexpr double kBadPivot = 1e128;

// Index of block (i, j), i <= j < 4, of an upper triangle of 16 x 16 blocks
__host__ __device__ constexpr int tri(int i, int j) { return i * 4 - i * (i - 1) / 2 + j - i; }

// Diagonal block b of a 64 x 64 block whose upper triangle of 16 x 16 blocks
// lies as fragments in B, factored by one wave: fragments 10 + b receive the A
// operands of the inverse of its Cholesky factor L(b, b) (the factor itself
// is not needed).  Eliminating with pivot j is one MFMA: row j of the block
// lies in register j / 4 of the lanes with l / 16 = j % 4, which is where both
// operands of a rank-1 product with k = j % 4 are read from, so the only data
// that moves is the pivot itself; the same product applied to the identity
// gives the inverse.  No square root is in the chain from pivot to pivot (the
// rows are scaled at the end).  tr: LDS of the wave for a transposition.
// Returns the number of pivots replaced.
__device__ __forceinline__ int factor16(double* B, int b, double* tr) {
    const int lane = threadIdx.x & (kWave - 1), l16 = lane & 15, lq = lane >> 4;
    d4 C = load_frag(B, tri(b, b)), E, piv;
#pragma unroll
    for (int r = 0; r < 4; ++r) E[r] = lq + 4 * r == l16 ? 1.0 : 0.0;
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int j = 4 * r + k;
            const double d = readlane_f64(C[r], 16 * k + j);
            const double f = d > 1e-300 ? -recip(d) : -1.0 / kBadPivot;
            const double a = lq == k && l16 > j ? C[r] * f : 0.0;
            if (j < 15) C = mfma16(a, C[r], C);
            if (j < 15) E = mfma16(a, E[r], E);
            piv[r] = k == 0 || lq == k ? d : piv[r];
            __builtin_amdgcn_sched_barrier(0);  // the second product fills the first one's latency
        }
    int bad = 0;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const bool ok = piv[r] > 1e-300;
        bad += __popcll(__ballot(!ok && l16 == 0));
        tr[(lq + 4 * r) * kTs + l16] = piv[r] >= kInfPivot ? 0.0 : E[r] * recip_sqrt(ok ? piv[r] : kBadPivot);
    }
    wave_lds_sync();
    d4 F;
#pragma unroll
    for (int r = 0; r < 4; ++r) F[r] = piv[r] >= kInfPivot ? 0.0 : tr[l16 * kTs + 4 * r + lq];
    store_frag(B, 10 + b, F);
    return bad;
}

// Fragment B(b, i) <- L(i, b)^T
__device__ __forceinline__ void solve16(double* B, int b, int i) {
    const d4 F = load_frag(B, 10 + b), t = load_frag(B, tri(b, i));
    d4 x = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int r = 0; r < 4; ++r) x = mfma16(F[r], t[r], x);
    store_frag(B, tri(b, i), x);
}

// Fragment B(i, j) -= L(i, b) L(j, b)^T
__device__ __forceinline__ void update16(double* B, int b, int i, int j) {
    const d4 u = load_frag(B, tri(b, i)), v = load_frag(B, tri(b, j));
    d4 x = load_frag(B, tri(i, j));
#pragma unroll
    for (int r = 0; r < 4; ++r) x = mfma16(-u[r], v[r], x);
    store_frag(B, tri(i, j), x);
}

// LDS: two 64 x 64 blocks; of the second, block column s uses the 10 + 4
// fragments of the diagonal block and the transposition's 16 rows
constexpr size_t kCholLds = sizeof(double) * 2 * kNb * kLs;
static_assert(14 * 256 + 16 * kTs <= kNb * kLs, "fragments fit the second block");

__global__ __launch_bounds__(kCholBlock, 3) void k_chol_step(double* M, int32_t ld, int32_t nbk, int32_t s, double* Linv,
                                                          int32_t* flag) {
    extern __shared__ __align__(16) double lds[];
    double* const P = lds;               // block (s, s - 1), or (j, s - 1)
    double* const D = lds + kNb * kLs;   // block (i, s - 1), or fragments: [block][register][lane]
    const int lane = threadIdx.x & (kWave - 1), wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int l16 = lane & 15, lq = lane >> 4;
    const int64_t L = ld;
    if ((int)blockIdx.x >= nbk - s) {  // block (i, j) right of column s: C -= P_i P_j^T
        const int64_t t = (int)blockIdx.x - (nbk - s);
        int64_t bi = (int64_t)((sqrt(8.0 * (double)t + 1.0) - 1.0) * 0.5);
        while ((bi + 1) * (bi + 2) / 2 <= t) ++bi;
        while (bi * (bi + 1) / 2 > t) --bi;
        const int64_t bj = t - bi * (bi + 1) / 2;
        const int64_t i = s + 1 + bi, j = s + 1 + bj;
        block_to_lds(M + i * kNb * L + (int64_t)(s - 1) * kNb, L, D, kCholBlock);
        block_to_lds(M + j * kNb * L + (int64_t)(s - 1) * kNb, L, P, kCholBlock);
        __syncthreads();
        if (wave >= 4) return;
        const int rw = 32 * (wave >> 1), cw = 32 * (wave & 1);  // the wave's 32 x 32 quarter
        double* C = M + (i * kNb + rw) * L + j * kNb + cw;
        d4 acc[2][2];
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
            for (int v = 0; v < 2; ++v)
#pragma unroll
                for (int r = 0; r < 4; ++r) acc[u][v][r] = C[(16 * u + lq + 4 * r) * L + 16 * v + l16];
#pragma unroll 4
        for (int k = 0; k < kNb; k += 4) {
            double a[2], b[2];
#pragma unroll
            for (int u = 0; u < 2; ++u) a[u] = -D[(rw + 16 * u + l16) * kLs + k + lq];
#pragma unroll
            for (int v = 0; v < 2; ++v) b[v] = P[(cw + 16 * v + l16) * kLs + k + lq];
#pragma unroll
            for (int u = 0; u < 2; ++u)
#pragma unroll
                for (int v = 0; v < 2; ++v) acc[u][v] = mfma16(a[u], b[v], acc[u][v]);
        }
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
            for (int v = 0; v < 2; ++v)
#pragma unroll
                for (int r = 0; r < 4; ++r) C[(16 * u + lq + 4 * r) * L + 16 * v + l16] = acc[u][v][r];
        return;
    }
    // block (i, s)
    const int i = s + (int)blockIdx.x;
    const bool diag = i == s;
    // the diagonal block with panel s - 1 applied: the upper triangle of its
    // ten 16 x 16 blocks (M holds the lower triangle), dealt so that no SIMD
    // has more than three (waves 0 and 4 share one)
    const int t0 = wave == 0 ? 0 : wave == 1 ? 1 : 2 * wave, nt = wave == 0 ? 1 : wave == 1 ? 3 : 2;
    d4 dd[3];
    int ti[3], tj[3];
#pragma unroll
    for (int u = 0; u < 3; ++u) {
        const int t = min(t0 + u, 9);
        ti[u] = t < 4 ? 0 : t < 7 ? 1 : t < 9 ? 2 : 3;
        tj[u] = t - tri(ti[u], ti[u]) + ti[u];
        if (u >= nt) continue;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int x = 16 * ti[u] + lq + 4 * r, y = 16 * tj[u] + l16;
            dd[u][r] = M[((int64_t)s * kNb + max(x, y)) * L + (int64_t)s * kNb + min(x, y)];
        }
    }
    if (s > 0) {
        block_to_lds(M + (int64_t)s * kNb * L + (int64_t)(s - 1) * kNb, L, P, kCholBlock);
        __syncthreads();
#pragma unroll 4
        for (int k = 0; k < kNb; k += 4)
#pragma unroll
            for (int u = 0; u < 3; ++u)
                if (u < nt)
                    dd[u] = mfma16(-P[(16 * ti[u] + l16) * kLs + k + lq], P[(16 * tj[u] + l16) * kLs + k + lq], dd[u]);
    }
#pragma unroll
    for (int u = 0; u < 3; ++u)
        if (u < nt) store_frag(D, t0 + u, dd[u]);
    __syncthreads();
    // wave 4 factors the diagonal block; the others apply panel s - 1 to X^T,
    // the wave's 16 rows of block (i, s) as columns (the identity's rows for
    // (s, s), whose solution is the inverse)
    d4 X[4];
    double* const Xg = M + ((int64_t)i * kNb + 16 * wave + l16) * L + (int64_t)s * kNb;
    int bad = 0;
    if (wave < 4) {
#pragma unroll
        for (int jb = 0; jb < 4; ++jb)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int c = 16 * jb + lq + 4 * r;
                X[jb][r] = diag ? (c == 16 * wave + l16 ? 1.0 : 0.0) : Xg[c];
            }
    }
    // the panel's 64 columns are applied to X^T 16 at a time, under the four
    // diagonal factors; the next diagonal block is brought up to date by wave
    // 4 alone, which goes on to factor it while the others update the rest
    const bool upd = s > 0 && !diag && wave < 4;
    const double* Pg = M + ((int64_t)i * kNb + 16 * (wave & 3) + l16) * L + (int64_t)(s - 1) * kNb + lq;
    double p[4], pn[4];
    if (upd)
#pragma unroll
        for (int k = 0; k < 4; ++k) pn[k] = Pg[4 * k];
#pragma unroll 1
    for (int b = 0; b < 4; ++b) {
        if (wave == 4) bad += factor16(D, b, D + 14 * 256);
        if (upd) {
            const double* Pf = P + l16 * kLs + lq + 16 * b;
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                p[k] = pn[k];
                pn[k] = Pg[16 * min(b + 1, 3) + 4 * k];
            }
#pragma unroll
            for (int k = 0; k < 4; ++k)
#pragma unroll
                for (int jb = 0; jb < 4; ++jb) X[jb] = mfma16(-Pf[16 * jb * kLs + 4 * k], p[k], X[jb]);
        }
        __syncthreads();
        if (b == 3) break;
        if (wave == 4) solve16(D, b, b + 1);
        else if (wave < 2 - b) solve16(D, b, b + 2 + wave);
        __syncthreads();
        if (wave == 4) update16(D, b, b + 1, b + 1);
        else if (b == 0) {
            if (wave == 0) update16(D, 0, 1, 2);
            else if (wave == 1) update16(D, 0, 1, 3);
            else if (wave == 2) update16(D, 0, 2, 2);
            else update16(D, 0, 2, 3);
            if (wave == 1) update16(D, 0, 3, 3);
        } else if (b == 1) {
            if (wave == 0) update16(D, 1, 2, 3);
            else if (wave == 1) update16(D, 1, 3, 3);
        }
    }
    if (wave == 4) {
        if (diag && lane == 0 && bad) atomicAdd(flag, bad);
        return;
    }
    // X^T <- L^-1 X^T, 16 rows at a time
#pragma unroll
    for (int jb = 0; jb < 4; ++jb) {
        d4 acc = X[jb];
#pragma unroll
        for (int l = 0; l < jb; ++l) {
            const d4 t = load_frag(D, tri(l, jb));
#pragma unroll
            for (int r = 0; r < 4; ++r) acc = mfma16(-t[r], X[l][r], acc);
        }
        const d4 t = load_frag(D, 10 + jb);
        d4 x = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int r = 0; r < 4; ++r) x = mfma16(t[r], acc[r], x);
        X[jb] = x;
    }
    if (diag) {  // X^T is L^-1
        double* Li = Linv + (int64_t)s * kNb * kNb + 16 * wave + l16;
#pragma unroll
        for (int jb = 0; jb < 4; ++jb)
#pragma unroll
            for (int r = 0; r < 4; ++r) Li[(16 * jb + lq + 4 * r) * kNb] = X[jb][r];
    } else {
#pragma unroll
        for (int jb = 0; jb < 4; ++jb)
#pragma unroll
            for (int r = 0; r < 4; ++r) Xg[16 * jb + lq + 4 * r] = X[jb][r];
    }
}

// --- triangular solves with the factor: one workgroup per 64 rows in one
// launch, each taking the solution blocks it depends on from the others as
// they are stored.  An entry not stored yet holds kUnset, a signalling NaN
// that no arithmetic produces (results that are NaN are quiet), so the value
// is its own flag: a block's step is one trip through memory and two
// 64 x 64 products, of the newest block and of the inverted diagonal factor.
// A workgroup waits only for workgroups that drew an earlier ticket, so they
// have started and wait for none later; a wait is bounded all the same
// (kMaxPolls): a value that did not come is used as the NaN it is, and the
// workgroup notes that in *late once it has passed its own values on (noted in
// the wait itself it was 0.5 to 0.9 us of a solve's chain); the call that
// launched this reports it as an error.
// What bounds it: the chain over the 64-row blocks, 1.2 to 1.4 us each: 22 us
// (lower) and 19 us (upper) at m = 1,000, 90 and 74 us at m = 4,000.  Before,
// one workgroup swept the whole factor, a compute unit's read rate: 0.52 and
// 0.62 ms, 5.8 and 10.0 ms.
constexpr unsigned long long kUnset = 0x7ff4a55a5aa5a55aull;
constexpr int kMaxPolls = 1 << 20;

__global__ __launch_bounds__(kBlock) void k_trsv_prepare(unsigned long long* y1, unsigned long long* y2, int32_t ld,
                                                         int32_t* ticket) {
    const int i = blockIdx.x * kBlock + threadIdx.x;
    if (i < 2) ticket[i] = 0;
    if (i < ld) {
        y1[i] = kUnset;
        y2[i] = kUnset;
    }
}

__device__ __forceinline__ double poll(const double* p) {
    const unsigned long long* q = (const unsigned long long*)p;
    unsigned long long v = kUnset;
    for (int k = 0; k < kMaxPolls; ++k) {
        v = __hip_atomic_load(q, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (v != kUnset) break;
    }
    return __longlong_as_double((long long)v);
}
__device__ __forceinline__ bool unset(double v) { return (unsigned long long)__double_as_longlong(v) == kUnset; }
__device__ __forceinline__ void publish(double* p, double v) {
    __hip_atomic_store((unsigned long long*)p, (unsigned long long)__double_as_longlong(v), __ATOMIC_RELAXED,
                       __HIP_MEMORY_SCOPE_AGENT);
}

// y <- L^-1 b.  Thread 4 r + q: row r of the block, its columns 16 q .. 16 q + 15.
__global__ __launch_bounds__(kBlock) void k_trsv_lower(const double* M, int32_t ld, const double* Linv, int32_t m,
                                                       const double* b, double* y, int32_t* ticket, int32_t* late) {
    __shared__ double xs[2][4 * 18];
    __shared__ int tk;
    if (threadIdx.x == 0) tk = atomicAdd(ticket, 1);
    __syncthreads();
    const int i = tk, r = threadIdx.x >> 2, q = threadIdx.x & 3;
    const int64_t L = ld;
    const double* Li = Linv + ((int64_t)i * kNb + r) * kNb + 16 * q;
    const double* A = M + ((int64_t)i * kNb + r) * L + 16 * q;
    d2 li[8], a[8], nx[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) li[k] = *(const d2*)(Li + 2 * k);
    const int row = i * kNb + r;
    const double bi = row < m ? b[row] : 0.0;
    if (i > 0)
#pragma unroll
        for (int k = 0; k < 8; ++k) nx[k] = *(const d2*)(A + 2 * k);
    double acc = 0.0;
    bool missed = false;
    for (int j = 0; j < i; ++j) {
#pragma unroll
        for (int k = 0; k < 8; ++k) a[k] = nx[k];
        if (j + 1 < i)
#pragma unroll
            for (int k = 0; k < 8; ++k) nx[k] = *(const d2*)(A + (int64_t)(j + 1) * kNb + 2 * k);
        double* x = xs[j & 1];
        double got = 0.0;
        if (threadIdx.x < kNb) {
            got = poll(y + (int64_t)j * kNb + threadIdx.x);
            x[18 * (threadIdx.x >> 4) + (threadIdx.x & 15)] = got;
        }
        __syncthreads();
        missed |= unset(got);
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            const d2 v = *(const d2*)(x + 18 * q + 2 * k);
            acc = fma(a[k][0], v[0], acc);
            acc = fma(a[k][1], v[1], acc);
        }
    }
    acc += __shfl_xor(acc, 1, kWave);
    acc += __shfl_xor(acc, 2, kWave);
    double* x = xs[i & 1];
    if (q == 0) x[18 * (r >> 4) + (r & 15)] = bi - acc;
    __syncthreads();
    acc = 0.0;
#pragma unroll
    for (int k = 0; k < 8; ++k) {
        const d2 v = *(const d2*)(x + 18 * q + 2 * k);
        acc = fma(li[k][0], v[0], acc);
        acc = fma(li[k][1], v[1], acc);
    }
    acc += __shfl_xor(acc, 1, kWave);
    acc += __shfl_xor(acc, 2, kWave);
    if (q == 0) publish(y + row, acc);
    if (missed) atomicOr(late, 1);
}

// x <- L^-T b (b, y of ld entries; x of m).  Thread 64 w + c: column c of the
// block, rows 16 w .. 16 w + 15.
__global__ __launch_bounds__(kBlock) void k_trsv_upper_t(const double* M, int32_t ld, const double* Linv, int32_t nbk,
                                                         int32_t m, const double* b, double* y, double* x_out,
                                                         int32_t* ticket, int32_t* late) {
    __shared__ double xs[2][kNb];
    __shared__ double part[4][kNb];
    __shared__ int tk;
    if (threadIdx.x == 0) tk = atomicAdd(ticket, 1);
    __syncthreads();
    const int i = nbk - 1 - tk, c = threadIdx.x & (kNb - 1), w = threadIdx.x >> 6;
    const int64_t L = ld;
    const double* Li = Linv + ((int64_t)i * kNb + 16 * w) * kNb + c;
    const double* A = M + (int64_t)16 * w * L + (int64_t)i * kNb + c;  // block (0, i), the thread's first row
    double li[16], a[16], nx[16];
#pragma unroll
    for (int k = 0; k < 16; ++k) li[k] = Li[k * kNb];
    if (i < nbk - 1)
#pragma unroll
        for (int k = 0; k < 16; ++k) nx[k] = A[((int64_t)(nbk - 1) * kNb + k) * L];
    double acc = 0.0;
    bool missed = false;
    for (int j = nbk - 1; j > i; --j) {
#pragma unroll
        for (int k = 0; k < 16; ++k) a[k] = nx[k];
        if (j - 1 > i)
#pragma unroll
            for (int k = 0; k < 16; ++k) nx[k] = A[((int64_t)(j - 1) * kNb + k) * L];
        double* x = xs[j & 1];
        double got = 0.0;
        if (w == 0) {
            got = poll(y + (int64_t)j * kNb + c);
            x[c] = got;
        }
        __syncthreads();
        missed |= unset(got);
#pragma unroll
        for (int k = 0; k < 16; ++k) acc = fma(a[k], x[16 * w + k], acc);
    }
    double* x = xs[i & 1];
    part[w][c] = acc;
    __syncthreads();
    if (w == 0) x[c] = b[(int64_t)i * kNb + c] - (((part[0][c] + part[1][c]) + part[2][c]) + part[3][c]);
    __syncthreads();
    acc = 0.0;
#pragma unroll
    for (int k = 0; k < 16; ++k) acc = fma(li[k], x[16 * w + k], acc);
    part[w][c] = acc;
    __syncthreads();
    if (w == 0) {
        const double v = ((part[0][c] + part[1][c]) + part[2][c]) + part[3][c];
        const int row = i * kNb + c;
        publish(y + row, v);
        if (row < m) x_out[row] = v;
        if (missed) atomicOr(late, 1);
    }
}

// --- per-iteration vector work
// d = x / z, r_xz (mode 0: -x z; 1: sigma_mu - x z - dxa dza), t = r_xz / z - d r_c
__global__ void k_ipm_t(const double* x, const double* z, const double* r_c, int mode, double sigma_mu,
                        const double* dxa, const double* dza, int64_t n, double* d, double* t) {
    for (int64_t j = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; j < n; j += (int64_t)gridDim.x * blockDim.x) {
        const double dj = x[j] / z[j];
        const double rxz = mode == 0 ? -x[j] * z[j] : sigma_mu - x[j] * z[j] - dxa[j] * dza[j];
        d[j] = dj;
        t[j] = rxz / z[j] - dj * r_c[j];
    }
}

// dx = d v + t, dz = r_c - v
__global__ void k_ipm_dir(const double* d, const double* v, const double* t, const double* r_c, int64_t n,
                          double* dx, double* dz) {
    for (int64_t j = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; j < n; j += (int64_t)gridDim.x * blockDim.x) {
        dx[j] = d[j] * v[j] + t[j];
        dz[j] = r_c[j] - v[j];
    }
}

// fixed-order block partials: W quantities per block, then one workgroup
// combines them (sum, or min for the ratio tests)
template <int W>
__device__ void block_partials(double (&v)[W], bool minimum, double* out) {
    __shared__ double sh[W][kBlock];
#pragma unroll
    for (int q = 0; q < W; ++q) sh[q][threadIdx.x] = v[q];
    __syncthreads();
    for (int st = kBlock / 2; st > 0; st >>= 1) {
        if (threadIdx.x < st)
#pragma unroll
            for (int q = 0; q < W; ++q)
                sh[q][threadIdx.x] = minimum ? fmin(sh[q][threadIdx.x], sh[q][threadIdx.x + st])
                                             : sh[q][threadIdx.x] + sh[q][threadIdx.x + st];
        __syncthreads();
    }
    if (threadIdx.x < W) out[(int64_t)blockIdx.x * W + threadIdx.x] = sh[threadIdx.x][0];
}

// step to the boundary: min over dv < 0 of -v / dv, for (x, dx) and (z, dz)
__global__ __launch_bounds__(kBlock) void k_ipm_ratio(const double* x, const double* dx, const double* z,
                                                      const double* dz, int64_t n, double* part) {
    double v[2] = {INFINITY, INFINITY};
    for (int64_t j = blockIdx.x * (int64_t)kBlock + threadIdx.x; j < n; j += (int64_t)gridDim.x * kBlock) {
        if (dx[j] < 0.0) v[0] = fmin(v[0], -x[j] / dx[j]);
        if (dz[j] < 0.0) v[1] = fmin(v[1], -z[j] / dz[j]);
    }
    block_partials<2>(v, true, part);
}

// The same of A^T, and what k_ipm_normal asks of it, against A (whose rows
// have been checked and are in order): flags bit 1, a row pointer that is not
// one; bit 2, an index out of range; bit 4, one that repeats in its row (of an
// entry that A has; others are differences); and three sums for each block,
// |a^T - a| over the entries of A^T (a = 0 where A has none), |a| of those that
// A has, and |a| over A.  mark: an int for each entry of A, zero.  A row
// pointer that is not one makes no access leave the arrays.
__global__ __launch_bounds__(kBlock) void k_ipm_check_at(const int32_t* rp, const int32_t* col, const double* val,
                                                         const int32_t* trp, const int32_t* tcol, const double* tval,
                                                         int32_t m, int32_t n, int32_t nnz, const double* d_row,
                                                         const double* d_col, int32_t* mark, int32_t* flags,
                                                         double* out, double* part) {
    const int lane = threadIdx.x & (kWave - 1);
    const int64_t t = blockIdx.x * (int64_t)kBlock + threadIdx.x, step = (int64_t)gridDim.x * kBlock;
    double v[3] = {0.0, 0.0, 0.0};
    int f = t == 0 && (trp[0] != 0 || trp[n] != nnz) ? 1 : 0;
    for (int64_t j = t / kWave; j < n; j += step / kWave) {
        const int s0 = trp[j], e0 = trp[j + 1];
        if (e0 < s0) f |= 1;
        const int s = min(max(s0, 0), nnz), e = min(max(e0, s), nnz);
        const double dc = d_col ? d_col[j] : 1.0;
        for (int k = s + lane; k < e; k += kWave) {
            const int i = tcol[k];
            if (i < 0 || i >= m) {
                f |= 2;
                continue;
            }
            const double a = tval[k];
            int lo = rp[i], hi = rp[i + 1] - 1;  // A's entry (i, j), if it has one
            while (lo < hi) {
                const int mid = (lo + hi) >> 1;
                if (col[mid] < j) lo = mid + 1;
                else hi = mid;
            }
            double b = 0.0;
            if (lo == hi && col[lo] == j) {
                b = val[lo];
                if (atomicExch(mark + lo, 1)) f |= 4;
                v[1] += fabs(b);
            }
            v[0] += fabs(a - b);
            out[k] = ((d_row ? d_row[i] : 1.0) * a) * dc;
        }
    }
    for (int64_t k = t; k < nnz; k += step) v[2] += fabs(val[k]);
    if (f) atomicOr(flags, f);
    block_partials<3>(v, false, part);
}

// sum (x + ap dx)(z + ad dz)
__global__ __launch_bounds__(kBlock) void k_ipm_mu_at(const double* x, const double* dx, const double* z,
                                                      const double* dz, int64_t n, const double* bounds,
                                                      double* part) {
    const double ap = fmin(1.0, bounds[0]), ad = fmin(1.0, bounds[1]);
    double v[1] = {0.0};
    for (int64_t j = blockIdx.x * (int64_t)kBlock + threadIdx.x; j < n; j += (int64_t)gridDim.x * kBlock)
        v[0] += (x[j] + ap * dx[j]) * (z[j] + ad * dz[j]);
    block_partials<1>(v, false, part);
}

// ||r_c||^2, c~^T x, x^T z over n; ||r_b||^2, b~^T y over m (two launches)
__global__ __launch_bounds__(kBlock) void k_ipm_sums3(const double* a, const double* b, const double* c,
                                                      const double* d, int64_t n, double* part) {
    double v[3] = {0.0, 0.0, 0.0};
    for (int64_t j = blockIdx.x * (int64_t)kBlock + threadIdx.x; j < n; j += (int64_t)gridDim.x * kBlock) {
        v[0] += a[j] * a[j];
        v[1] += b[j] * c[j];
        if (d) v[2] += c[j] * d[j];
    }
    block_partials<3>(v, false, part);
}

template <int W>
__global__ __launch_bounds__(kBlock) void k_ipm_final(const double* part, int G, int minimum_mask, double* out) {
    __shared__ double sh[kBlock];
    for (int q = 0; q < W; ++q) {
        const bool mn = (minimum_mask >> q) & 1;
        double s = mn ? INFINITY : 0.0;
        for (int g = threadIdx.x; g < G; g += kBlock) {
            const double v = part[(int64_t)g * W + q];
            s = mn ? fmin(s, v) : s + v;
        }
        sh[threadIdx.x] = s;
        __syncthreads();
        for (int st = kBlock / 2; st > 0; st >>= 1) {
            if (threadIdx.x < st)
                sh[threadIdx.x] = mn ? fmin(sh[threadIdx.x], sh[threadIdx.x + st]) : sh[threadIdx.x] + sh[threadIdx.x + st];
            __syncthreads();
        }
        if (threadIdx.x == 0) out[q] = sh[0];
        __syncthreads();
    }
}

// v += a s .* dv for up to three (vector, direction, step slot) triples
__global__ void k_ipm_step(double* x, const double* dx, int64_t n, double* y, const double* dy, int64_t m, double* z,
                           const double* dz, double ap, double ad) {
    for (int64_t j = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; j < n; j += (int64_t)gridDim.x * blockDim.x) {
        x[j] = x[j] + ap * dx[j];
        z[j] = z[j] + ad * dz[j];
    }
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < m; i += (int64_t)gridDim.x * blockDim.x)
        y[i] = y[i] + ad * dy[i];
}

__global__ void k_zero_flag(int32_t* f, double* scal) {
    if (threadIdx.x < 4) f[threadIdx.x] = 0;
    if (threadIdx.x < 16) scal[threadIdx.x] = 0.0;
}

// v + s for Mehrotra's shifts
__global__ void k_ipm_shift(double* v, int64_t n, double s) {
    for (int64_t j = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; j < n; j += (int64_t)gridDim.x * blockDim.x)
        v[j] = v[j] + s;
}

// sum and min of a vector, and its dot with another: part[g] = {sum a, min a, sum a b}
__global__ __launch_bounds__(kBlock) void k_ipm_summin(const double* a, const double* b, int64_t n, double* part) {
    double v[3] = {0.0, INFINITY, 0.0};
    for (int64_t j = blockIdx.x * (int64_t)kBlock + threadIdx.x; j < n; j += (int64_t)gridDim.x * kBlock) {
        v[0] += a[j];
        v[1] = fmin(v[1], a[j]);
        if (b) v[2] += a[j] * b[j];
    }
    // min needs its own combine: reuse block_partials twice
    double s[2] = {v[0], v[2]};
    double mn[1] = {v[1]};
    block_partials<2>(s, false, part);
    __syncthreads();
    block_partials<1>(mn, true, part + 2 * (int64_t)gridDim.x);
}

struct IpmWs {
    double *M, *av, *atv, *bt, *ct, *x, *y, *z, *dx, *dy, *dz, *dxa, *dya, *dza, *d, *t, *v, *rb, *rc, *rhs;
    double *xc, *yc, *zc, *part, *scal;
    double *linv, *y1, *y2;  // inverted diagonal factors; the triangular solves' vectors
    int32_t *flag, *ticket;
    void* cws;  // centering workspace
    size_t bytes;
};

// order of the dense matrix: m rounded up to whole blocks
int64_t ipm_ld(int64_t m) { return (m + kNb - 1) / kNb * kNb; }

IpmWs carve_ipm(void* base, int64_t m, int64_t n, int64_t nnz) {
    Carver cv(base, 0);
    IpmWs w;
    const int64_t ld = ipm_ld(m);
    w.M = cv.take<double>((size_t)(ld * ld));
    w.av = cv.take<double>(nnz);
    w.atv = cv.take<double>(nnz);
    w.bt = cv.take<double>(m);
    w.ct = cv.take<double>(n);
    w.x = cv.take<double>(n);
    w.y = cv.take<double>(m);
    w.z = cv.take<double>(n);
    w.dx = cv.take<double>(n);
    w.dy = cv.take<double>(m);
    w.dz = cv.take<double>(n);
    w.dxa = cv.take<double>(n);
    w.dya = cv.take<double>(m);
    w.dza = cv.take<double>(n);
    w.d = cv.take<double>(n);
    w.t = cv.take<double>(n);
    w.v = cv.take<double>(std::max(m, n));
    w.rb = cv.take<double>(m);
    w.rc = cv.take<double>(n);
    w.rhs = cv.take<double>(m);
    w.xc = cv.take<double>(n);
    w.yc = cv.take<double>(m);
    w.zc = cv.take<double>(n);
    w.part = cv.take<double>((size_t)kRedBlocks * 4);
    w.scal = cv.take<double>(16);
    w.linv = cv.take<double>((size_t)(ld * kNb));
    w.y1 = cv.take<double>((size_t)ld);
    w.y2 = cv.take<double>((size_t)ld);
    w.flag = cv.take<int32_t>(4);
    w.ticket = cv.take<int32_t>(4);
    w.cws = cv.take<char>(mipdhg_center_workspace_size((int32_t)n));
    w.bytes = cv.off;
    return w;
}

int red_grid(int64_t n) { return (int)std::max<int64_t>(1, std::min<int64_t>(kRedBlocks, (n + kBlock - 1) / kBlock)); }
int rows_grid(int64_t rows) { return (int)((rows + kBlock / kWave - 1) / (kBlock / kWave)); }

struct Ipm {
    const mipdhg_lp& lp;
    const mipdhg_ipm_options& o;
    hipStream_t s;
    IpmWs w;
    int64_t m, n;
    int pivots = 0;

    int spmv_a(const double* v, const double* s0, double sgn, const double* s1, double* out) {
        hipLaunchKernelGGL(k_ipm_spmv, dim3(rows_grid(m)), dim3(kBlock), 0, s, lp.a_rowptr, lp.a_col,
                           (const double*)w.av, v, (int32_t)m, s0, sgn, s1, out);
        MIP_LAUNCH_CHECK();
        return 0;
    }
    int spmv_at(const double* v, const double* s0, double sgn, const double* s1, double* out) {
        hipLaunchKernelGGL(k_ipm_spmv, dim3(rows_grid(n)), dim3(kBlock), 0, s, lp.at_rowptr, lp.at_col,
                           (const double*)w.atv, v, (int32_t)n, s0, sgn, s1, out);
        MIP_LAUNCH_CHECK();
        return 0;
    }
    // the kernels that may need more than 64 KB of LDS
    int allow_lds() {
        MIP_HIP(hipFuncSetAttribute((const void*)k_chol_step, hipFuncAttributeMaxDynamicSharedMemorySize,
                                    (int)kCholLds));
        MIP_HIP(hipFuncSetAttribute((const void*)k_ipm_normal, hipFuncAttributeMaxDynamicSharedMemorySize,
                                    (int)(kIpmMaxM * 8)));
        return 0;
    }
    // M = A~ diag(wt) A~^T (lower), then its Cholesky factor in place
    int factor(const double* wt) {
        const int ld = (int)ipm_ld(m), nbk = ld / kNb;
        hipLaunchKernelGGL(k_ipm_normal, dim3(ld), dim3(kWave), (size_t)ld * 8, s, lp.a_rowptr, lp.a_col,
                           (const double*)w.av, lp.at_rowptr, lp.at_col, (const double*)w.atv, wt, (int32_t)m, ld,
                           w.M);
        MIP_LAUNCH_CHECK();
        for (int k = 0; k < nbk; ++k) {
            const int R = nbk - 1 - k;  // block rows below, and right of, column k
            hipLaunchKernelGGL(k_chol_step, dim3(R + 1 + (k > 0 ? R * (R + 1) / 2 : 0)), dim3(kCholBlock), kCholLds, s,
                               w.M, ld, nbk, k, w.linv, w.flag);
        }
        MIP_LAUNCH_CHECK();
        return 0;
    }
    // x <- M^-1 x with the factor in M
    int solve(double* x) {
        const int ld = (int)ipm_ld(m), nbk = ld / kNb;
        hipLaunchKernelGGL(k_trsv_prepare, dim3((ld + kBlock - 1) / kBlock), dim3(kBlock), 0, s,
                           (unsigned long long*)w.y1, (unsigned long long*)w.y2, ld, w.ticket);
        hipLaunchKernelGGL(k_trsv_lower, dim3(nbk), dim3(kBlock), 0, s, (const double*)w.M, ld, (const double*)w.linv,
                           (int32_t)m, (const double*)x, w.y1, w.ticket, w.flag + 1);
        hipLaunchKernelGGL(k_trsv_upper_t, dim3(nbk), dim3(kBlock), 0, s, (const double*)w.M, ld,
                           (const double*)w.linv, nbk, (int32_t)m, (const double*)w.y1, w.y2, x, w.ticket + 1,
                           w.flag + 1);
        MIP_LAUNCH_CHECK();
        return 0;
    }
    // Scalars stay on the device until the host decides with them: the sums of
    // the partials go to slots of w.scal, and one copy brings several.  (A copy
    // with its wait is about 20 us of an idle device; a Newton step has three,
    // where fetching each sum by itself and sending the steps back took seven.)
    template <int W>
    int reduce(int G, int minmask, int slot, int64_t skip = 0) {
        hipLaunchKernelGGL((k_ipm_final<W>), dim3(1), dim3(kBlock), 0, s, (const double*)(w.part + skip), G, minmask,
                           w.scal + slot);
        MIP_LAUNCH_CHECK();
        return 0;
    }
    int fetch(double* host, int slot, int count) {
        MIP_HIP(hipMemcpyAsync(host, w.scal + slot, count * sizeof(double), hipMemcpyDeviceToHost, s));
        MIP_HIP(hipStreamSynchronize(s));
        return 0;
    }

    // Mehrotra's start: x = A~^T (A~ A~^T)^-1 b~, y = (A~ A~^T)^-1 A~ c~,
    // z = c~ - A~^T y, shifted by max(-1.5 min, 0), then by half of x^T z
    // over the sum of the other vector
    int cold_start() {
        int rc;
        if ((rc = factor(nullptr))) return rc;
        MIP_HIP(hipMemcpyAsync(w.rhs, w.bt, m * 8, hipMemcpyDeviceToDevice, s));
        if ((rc = solve(w.rhs))) return rc;
        if ((rc = spmv_at(w.rhs, nullptr, 1.0, nullptr, w.x))) return rc;
        if ((rc = spmv_a(w.ct, nullptr, 1.0, nullptr, w.y))) return rc;
        if ((rc = solve(w.y))) return rc;
        if ((rc = spmv_at(w.y, w.ct, -1.0, nullptr, w.z))) return rc;
        double h[6];  // {sum, sum of products, min} of x and of z
        if ((rc = summin(w.x, nullptr, 0)) || (rc = summin(w.z, nullptr, 3)) || (rc = fetch(h, 0, 6))) return rc;
        const double sx = std::max(-1.5 * h[2], 0.0), sz = std::max(-1.5 * h[5], 0.0);
        hipLaunchKernelGGL(k_ipm_shift, dim3(grid_for(n)), dim3(kBlock), 0, s, w.x, n, sx);
        hipLaunchKernelGGL(k_ipm_shift, dim3(grid_for(n)), dim3(kBlock), 0, s, w.z, n, sz);
        MIP_LAUNCH_CHECK();
        // x^T z, sum x, sum z of the shifted vectors
        if ((rc = summin(w.x, w.z, 0)) || (rc = summin(w.z, nullptr, 3)) || (rc = fetch(h, 0, 6))) return rc;
        const double xz = h[1];
        hipLaunchKernelGGL(k_ipm_shift, dim3(grid_for(n)), dim3(kBlock), 0, s, w.x, n, 0.5 * xz / h[3]);
        hipLaunchKernelGGL(k_ipm_shift, dim3(grid_for(n)), dim3(kBlock), 0, s, w.z, n, 0.5 * xz / h[0]);
        MIP_LAUNCH_CHECK();
        return 0;
    }
    // {sum a, sum a b, min a} into three slots
    int summin(const double* a, const double* b, int slot) {
        const int G = red_grid(n);
        hipLaunchKernelGGL(k_ipm_summin, dim3(G), dim3(kBlock), 0, s, a, b, n, w.part);
        MIP_LAUNCH_CHECK();
        int rc;
        if ((rc = reduce<2>(G, 0, slot))) return rc;
        return reduce<1>(G, 1, slot + 2, 2 * (int64_t)G);
    }
    // {sum a^2, sum b c, sum c d} into three slots
    int sums3(const double* a, const double* b, const double* c, const double* d, int64_t len, int slot) {
        const int G = red_grid(len);
        hipLaunchKernelGGL(k_ipm_sums3, dim3(G), dim3(kBlock), 0, s, a, b, c, d, len, w.part);
        MIP_LAUNCH_CHECK();
        return reduce<3>(G, 0, slot);
    }

    // the relative measures (rp, rd, gap) and c~^T x, b~^T y, x^T z; r_b, r_c left in the workspace
    int measures(double* rel, double* px, double* dy, double* xz) {
        int rc;
        if ((rc = spmv_a(w.x, w.bt, -1.0, nullptr, w.rb))) return rc;
        if ((rc = spmv_at(w.y, w.ct, -1.0, w.z, w.rc))) return rc;
        double h[6];
        if ((rc = sums3(w.rc, w.ct, w.x, w.z, n, 0)) || (rc = sums3(w.rb, w.bt, w.y, nullptr, m, 3)) ||
            (rc = fetch(h, 0, 6)))
            return rc;
        const double *hn = h, *hm = h + 3;
        rel[0] = sqrt(hm[0]) / (1.0 + bnorm);
        rel[1] = sqrt(hn[0]) / (1.0 + cnorm);
        *px = hn[1];
        *dy = hm[1];
        *xz = hn[2];
        rel[2] = fabs(*px - *dy) / (1.0 + fabs(*px) + fabs(*dy));
        return 0;
    }
    double bnorm = 0.0, cnorm = 0.0;

    // direction for r_xz of `mode` (see k_ipm_t) into (dx, dy, dz)
    int direction(int mode, double sigma_mu, double* dx, double* dy, double* dz) {
        int rc;
        hipLaunchKernelGGL(k_ipm_t, dim3(grid_for(n)), dim3(kBlock), 0, s, (const double*)w.x, (const double*)w.z,
                           (const double*)w.rc, mode, sigma_mu, (const double*)w.dxa, (const double*)w.dza, n, w.d,
                           w.t);
        MIP_LAUNCH_CHECK();
        if ((rc = spmv_a(w.t, w.rb, -1.0, nullptr, dy))) return rc;  // r_b - A~ t
        if ((rc = solve(dy))) return rc;
        if ((rc = spmv_at(dy, nullptr, 1.0, nullptr, w.v))) return rc;
        hipLaunchKernelGGL(k_ipm_dir, dim3(grid_for(n)), dim3(kBlock), 0, s, (const double*)w.d, (const double*)w.v,
                           (const double*)w.t, (const double*)w.rc, n, dx, dz);
        MIP_LAUNCH_CHECK();
        return 0;
    }
    // steps to the boundary of (x, dx) and (z, dz) into two slots
    int boundary(const double* dx, const double* dz, int slot) {
        const int G = red_grid(n);
        hipLaunchKernelGGL(k_ipm_ratio, dim3(G), dim3(kBlock), 0, s, (const double*)w.x, dx, (const double*)w.z, dz,
                           n, w.part);
        MIP_LAUNCH_CHECK();
        return reduce<2>(G, 3, slot);
    }

    // the iteration from the point in (x, y, z); fills info
    int run(mipdhg_ipm_info* info) {
        int rc;
        info->iters = 0;
        info->status = MIPDHG_ITER_LIMIT;
        for (int k = 0;; ++k) {
            double rel[3], px, dyv, xz;
            if ((rc = measures(rel, &px, &dyv, &xz))) return rc;
            info->pobj = px;
            info->dobj = dyv;
            info->mu = xz / (double)n;
            info->rel_rp = rel[0];
            info->rel_rd = rel[1];
            info->rel_gap = rel[2];
            if (!(std::isfinite(rel[0]) && std::isfinite(rel[1]) && std::isfinite(rel[2]))) {
                info->status = MIPDHG_NUMERICAL;
                break;
            }
            if (std::max(rel[0], std::max(rel[1], rel[2])) <= o.tol) {
                info->status = MIPDHG_OPTIMAL;
                break;
            }
            if (k == o.max_iter) break;
            const double mu = xz / (double)n;
            hipLaunchKernelGGL(k_ipm_vscale, dim3(grid_for(n)), dim3(kBlock), 0, s, (const double*)w.x,
                               (const double*)w.z, 1, n, w.d);  // D = X Z^-1
            MIP_LAUNCH_CHECK();
            if ((rc = factor(w.d))) return rc;
            // predictor
            if ((rc = direction(0, 0.0, w.dxa, w.dya, w.dza))) return rc;
            if ((rc = boundary(w.dxa, w.dza, 0))) return rc;
            const int G = red_grid(n);
            hipLaunchKernelGGL(k_ipm_mu_at, dim3(G), dim3(kBlock), 0, s, (const double*)w.x, (const double*)w.dxa,
                               (const double*)w.z, (const double*)w.dza, n, (const double*)w.scal, w.part);
            MIP_LAUNCH_CHECK();
            double mua[1];
            if ((rc = reduce<1>(G, 0, 2)) || (rc = fetch(mua, 2, 1))) return rc;
            const double sigma = std::pow((mua[0] / (double)n) / mu, 3.0);
            // corrector, with the same factor
            if ((rc = direction(1, sigma * mu, w.dx, w.dy, w.dz))) return rc;
            double st[2];
            if ((rc = boundary(w.dx, w.dz, 0)) || (rc = fetch(st, 0, 2))) return rc;
            const double steps[2] = {std::min(1.0, o.step_frac * st[0]), std::min(1.0, o.step_frac * st[1])};
            if (k == 0) {
                info->first_step_p = steps[0];
                info->first_step_d = steps[1];
            }
            hipLaunchKernelGGL(k_ipm_step, dim3(grid_for(std::max(m, n))), dim3(kBlock), 0, s, w.x,
                               (const double*)w.dx, n, w.y, (const double*)w.dy, m, w.z, (const double*)w.dz,
                               steps[0], steps[1]);
            MIP_LAUNCH_CHECK();
            info->iters = k + 1;
        }
        return 0;
    }
};

}  // namespace
}  // namespace mip

using namespace mip;

namespace {

int check_ipm(const mipdhg_lp* lp, const mipdhg_ipm_options* o) {
    int rc = check_lp(lp);
    if (rc) return rc;
    if (!o) return set_error("options are NULL"), MIPDHG_ERR_INVALID_ARG;
    if (lp->lo || lp->hi || lp->sense)
        return set_error("the interior-point consumer takes the standard form"), MIPDHG_ERR_UNSUPPORTED;
    if (lp->m > kIpmMaxM)
        return set_error("m = %d: the dense normal matrix is limited to m <= %d", lp->m, kIpmMaxM),
               MIPDHG_ERR_UNSUPPORTED;
    if (!(o->tol > 0.0) || o->max_iter < 0 || !(o->step_frac > 0.0 && o->step_frac < 1.0) || !(o->min_step >= 0.0) ||
        o->max_lifts < 0 || !(o->mu_min >= 0.0) || !(o->delta_max >= 0.0) || !(o->alpha_min > 0.0) ||
        !std::isfinite(o->tol) || !std::isfinite(o->alpha_min) || !std::isfinite(o->mu_min) ||
        !std::isfinite(o->delta_max))
        return set_error("ipm options: tol > 0, max_iter >= 0, 0 < step_frac < 1, min_step >= 0, max_lifts >= 0, "
                         "mu_min >= 0, delta_max >= 0, alpha_min > 0, all finite"),
               MIPDHG_ERR_INVALID_ARG;
    return 0;
}

// the scaled LP in the workspace, after checking that A's rows are sorted and
// that A^T is its transpose, each entry once (in any order within a row)
int ipm_setup(Ipm& P, const double* d_row, const double* d_col) {
    const mipdhg_lp& lp = P.lp;
    hipStream_t s = P.s;
    std::vector<int32_t> rp(lp.m + 1), col(lp.nnz);
    MIP_HIP(hipMemcpyAsync(rp.data(), lp.a_rowptr, rp.size() * 4, hipMemcpyDeviceToHost, s));
    if (lp.nnz) MIP_HIP(hipMemcpyAsync(col.data(), lp.a_col, col.size() * 4, hipMemcpyDeviceToHost, s));
    MIP_HIP(hipStreamSynchronize(s));
    int rc = check_rowptr(rp, lp.m, lp.nnz, "A");
    if (rc) return rc;
    for (int32_t r = 0; r < lp.m; ++r)
        for (int32_t k = rp[r]; k < rp[r + 1]; ++k) {
            if (col[k] < 0 || col[k] >= lp.n)
                return set_error("A: column index out of range in row %d", r), MIPDHG_ERR_BAD_CSR;
            if (k > rp[r] && col[k] <= col[k - 1])
                return set_error("A: the interior-point consumer needs each row's columns strictly increasing "
                                 "(row %d)", r),
                       MIPDHG_ERR_BAD_CSR;
        }
    const IpmWs& w = P.w;
    if ((rc = P.allow_lds())) return rc;
    hipLaunchKernelGGL(k_zero_flag, dim3(1), dim3(32), 0, s, w.flag, w.scal);
    // (A's scaled values take the marks' place)
    if (lp.nnz) MIP_HIP(hipMemsetAsync(w.av, 0, lp.nnz * sizeof(int32_t), s));
    constexpr int kCheckSums = 7, kCheckFlags = 10;  // slots of w.scal
    const int Gc = std::min(rows_grid(lp.n), kRedBlocks);
    hipLaunchKernelGGL(k_ipm_check_at, dim3(Gc), dim3(kBlock), 0, s, lp.a_rowptr, lp.a_col, lp.a_val, lp.at_rowptr,
                       lp.at_col, lp.at_val, lp.m, lp.n, (int32_t)lp.nnz, d_row, d_col, (int32_t*)w.av,
                       (int32_t*)(w.scal + kCheckFlags), w.atv, w.part);
    MIP_LAUNCH_CHECK();
    if ((rc = P.reduce<3>(Gc, 0, kCheckSums))) return rc;
    hipLaunchKernelGGL(k_ipm_scale_vals, dim3(grid_for((int64_t)lp.m * kWave)), dim3(kBlock), 0, s, lp.a_rowptr, lp.a_col, lp.a_val,
                       lp.m, d_row, d_col, w.av);
    hipLaunchKernelGGL(k_ipm_vscale, dim3(grid_for(lp.m)), dim3(kBlock), 0, s, lp.b, d_row, 0, (int64_t)lp.m, w.bt);
    hipLaunchKernelGGL(k_ipm_vscale, dim3(grid_for(lp.n)), dim3(kBlock), 0, s, lp.c, d_col, 0, (int64_t)lp.n, w.ct);
    MIP_LAUNCH_CHECK();
    double h[kCheckFlags + 1];
    if ((rc = P.sums3(w.bt, w.bt, w.bt, nullptr, lp.m, 0)) || (rc = P.sums3(w.ct, w.ct, w.ct, nullptr, lp.n, 3)) ||
        (rc = P.fetch(h, 0, kCheckFlags + 1)))
        return rc;
    int32_t bad;
    memcpy(&bad, h + kCheckFlags, sizeof(bad));
    if (bad & 1) return set_error("A^T: the row pointer does not rise from 0 to nnz"), MIPDHG_ERR_BAD_CSR;
    if (bad & 2) return set_error("A^T: column index out of range"), MIPDHG_ERR_BAD_CSR;
    if (bad & 4) return set_error("A^T: an index repeats in a row"), MIPDHG_ERR_BAD_CSR;
    const double differ = h[kCheckSums] + (h[kCheckSums + 2] - h[kCheckSums + 1]);
    if (differ > 1e-10 * h[kCheckSums + 2] + 1e-300)  // (false where a value is not finite: NUMERICAL, later)
        return set_error("A^T does not match A (entries differ by %.3g of %.3g in sum)", differ, h[kCheckSums + 2]),
               MIPDHG_ERR_TRANSPOSE;
    P.bnorm = sqrt(h[0]);
    P.cnorm = sqrt(h[3]);
    return 0;
}

// the point in the workspace, unscaled into the outputs; pivots into info (its
// measures are those that ended run())
int ipm_finish(Ipm& P, const double* d_row, const double* d_col, double* x, double* y, double* z,
               mipdhg_ipm_info* info) {
    hipStream_t s = P.s;
    const IpmWs& w = P.w;
    hipLaunchKernelGGL(k_ipm_vscale, dim3(grid_for(P.n)), dim3(kBlock), 0, s, (const double*)w.x, d_col, 0, P.n, x);
    hipLaunchKernelGGL(k_ipm_vscale, dim3(grid_for(P.m)), dim3(kBlock), 0, s, (const double*)w.y, d_row, 0, P.m, y);
    hipLaunchKernelGGL(k_ipm_vscale, dim3(grid_for(P.n)), dim3(kBlock), 0, s, (const double*)w.z, d_col, 1, P.n, z);
    MIP_LAUNCH_CHECK();
    int32_t flag[2] = {0, 0};  // pivots replaced, a triangular solve's wait that ran out
    MIP_HIP(hipMemcpyAsync(flag, w.flag, sizeof(flag), hipMemcpyDeviceToHost, s));
    MIP_HIP(hipStreamSynchronize(s));
    info->pivots_replaced = flag[0];
    if (flag[1]) return set_error("a triangular solve gave up waiting for an earlier block of rows"), MIPDHG_ERR_HIP;
    return 0;
}

}  // namespace

extern "C" void mipdhg_ipm_default_options(mipdhg_ipm_options* o) {
    if (!o) return;
    o->tol = 1e-8;
    o->max_iter = 100;
    o->step_frac = 0.9995;
    o->min_step = 1e-6;
    o->max_lifts = 12;
    o->mu_min = 1e-6;
    o->delta_max = 1e-4;
    o->alpha_min = 1e-6;
}

extern "C" int mipdhg_ipm_workspace_size(const mipdhg_lp* lp, size_t* bytes) {
    clear_error();
    if (!bytes) return set_error("bytes is NULL"), MIPDHG_ERR_INVALID_ARG;
    int rc = check_lp(lp);
    if (rc) return rc;
    if (lp->m > kIpmMaxM)
        return set_error("m = %d: the dense normal matrix is limited to m <= %d", lp->m, kIpmMaxM),
               MIPDHG_ERR_UNSUPPORTED;
    *bytes = carve_ipm(nullptr, lp->m, lp->n, lp->nnz).bytes;
    return 0;
}

extern "C" int mipdhg_ipm_solve(const mipdhg_lp* lp, const double* d_row, const double* d_col, const double* x_start,
                                const double* y_start, const double* z_start, const mipdhg_ipm_options* opt,
                                void* workspace, size_t workspace_bytes, void* stream, double* x, double* y, double* z,
                                mipdhg_ipm_info* info) {
    clear_error();
    int rc = check_ipm(lp, opt);
    if (rc) return rc;
    const bool cold = !x_start && !y_start && !z_start;
    if (!cold && !(x_start && y_start && z_start))
        return set_error("give all three of x_start, y_start, z_start or none"), MIPDHG_ERR_INVALID_ARG;
    if (!workspace || !x || !y || !z || !info) return set_error("workspace, outputs and info are required"),
                                                      MIPDHG_ERR_INVALID_ARG;
    if (((uintptr_t)workspace & 255) != 0) return set_error("workspace must be 256-byte aligned"), MIPDHG_ERR_INVALID_ARG;
    const auto t0 = std::chrono::steady_clock::now();
    Ipm P{*lp, *opt, (hipStream_t)stream, carve_ipm(workspace, lp->m, lp->n, lp->nnz), lp->m, lp->n};
    if (P.w.bytes > workspace_bytes)
        return set_error("workspace too small: %zu bytes given, %zu needed", workspace_bytes, P.w.bytes),
               MIPDHG_ERR_WORKSPACE;
    memset(info, 0, sizeof(*info));
    StreamDrain drain{P.s};
    if ((rc = ipm_setup(P, d_row, d_col))) return rc;
    if (cold) {
        if ((rc = P.cold_start())) return rc;
    } else {
        MIP_HIP(hipMemcpyAsync(P.w.x, x_start, P.n * 8, hipMemcpyDeviceToDevice, P.s));
        MIP_HIP(hipMemcpyAsync(P.w.y, y_start, P.m * 8, hipMemcpyDeviceToDevice, P.s));
        MIP_HIP(hipMemcpyAsync(P.w.z, z_start, P.n * 8, hipMemcpyDeviceToDevice, P.s));
    }
    if ((rc = P.run(info))) return rc;
    if ((rc = ipm_finish(P, d_row, d_col, x, y, z, info))) return rc;
    drain.armed = false;
    info->alpha_min = 0.0;
    info->ms_total = std::chrono::duration<double, std::milli>(std::chrono::steady_clock::now() - t0).count();
    return info->status;
}

extern "C" int mipdhg_ipm_warm(const mipdhg_lp* lp, const double* d_row, const double* d_col, const double* x_pdhg,
                               const double* y_pdhg, const double* z_pdhg, const mipdhg_ipm_options* opt,
                               void* workspace, size_t workspace_bytes, void* stream, double* x, double* y, double* z,
                               mipdhg_ipm_info* info) {
    clear_error();
    int rc = check_ipm(lp, opt);
    if (rc) return rc;
    if (!x_pdhg || !y_pdhg || !z_pdhg || !workspace || !x || !y || !z || !info)
        return set_error("the PDHG point, workspace, outputs and info are required"), MIPDHG_ERR_INVALID_ARG;
    if (((uintptr_t)workspace & 255) != 0) return set_error("workspace must be 256-byte aligned"), MIPDHG_ERR_INVALID_ARG;
    const auto t0 = std::chrono::steady_clock::now();
    Ipm P{*lp, *opt, (hipStream_t)stream, carve_ipm(workspace, lp->m, lp->n, lp->nnz), lp->m, lp->n};
    if (P.w.bytes > workspace_bytes)
        return set_error("workspace too small: %zu bytes given, %zu needed", workspace_bytes, P.w.bytes),
               MIPDHG_ERR_WORKSPACE;
    memset(info, 0, sizeof(*info));
    StreamDrain drain{P.s};
    if ((rc = ipm_setup(P, d_row, d_col))) return rc;
    // Algorithm 1 on the scaled point (x / D_c, y / D_r, z D_c)
    double mu_t = 0.0;
    if ((rc = mipdhg_center_start(lp->n, x_pdhg, z_pdhg, d_col, opt->mu_min, opt->delta_max, opt->alpha_min, P.w.cws,
                                  mipdhg_center_workspace_size(lp->n), stream, P.w.xc, P.w.zc, &mu_t)))
        return rc;
    hipLaunchKernelGGL(k_ipm_vscale, dim3(grid_for(P.m)), dim3(kBlock), 0, P.s, y_pdhg, d_row, 1, P.m, P.w.yc);
    MIP_LAUNCH_CHECK();
    double alpha = opt->alpha_min;
    int lifts = 0;
    while (true) {
        MIP_HIP(hipMemcpyAsync(P.w.x, P.w.xc, P.n * 8, hipMemcpyDeviceToDevice, P.s));
        MIP_HIP(hipMemcpyAsync(P.w.y, P.w.yc, P.m * 8, hipMemcpyDeviceToDevice, P.s));
        MIP_HIP(hipMemcpyAsync(P.w.z, P.w.zc, P.n * 8, hipMemcpyDeviceToDevice, P.s));
        if ((rc = P.run(info))) return rc;
        const bool small = info->iters >= 1 && std::min(info->first_step_p, info->first_step_d) < opt->min_step;
        if (!small || lifts >= opt->max_lifts) break;
        alpha *= 10.0;
        ++lifts;
        if ((rc = mipdhg_center_reclamp(lp->n, alpha, stream, P.w.xc, P.w.zc))) return rc;
    }
    if ((rc = ipm_finish(P, d_row, d_col, x, y, z, info))) return rc;
    drain.armed = false;
    info->lifts = lifts;
    info->alpha_min = alpha;
    info->mu_target = mu_t;
    info->ms_total = std::chrono::duration<double, std::milli>(std::chrono::steady_clock::now() - t0).count();
    return info->status;
}
