// Per-instance pieces shared by the batched solve and the unrolled map: the
// instance's scaled matrices laid out for one workgroup, fixed-order sums, and
// the instance set-up (norms, scaling, scaled values, power iteration, step
// and initial primal weight).
#pragma once

#include <hip/hip_runtime.h>

#include <type_traits>

#include "common.h"

namespace mip {

// Dot product of the sparse row [s, e) with a vector held in LDS, indexed by
// the instance-local column (16 bits: an instance's vectors fit in LDS, so
// its rows and columns number fewer than 65,536): the loads of four nonzeros
// are issued together, and the terms are added in the row's order.
template <typename Acc, typename V, typename X>
__device__ __forceinline__ Acc row_dot4(const V* vals, const uint16_t* cols, const X* xl, int s, int e) {
    Acc acc = 0;
    int k = s;
    for (; k + 4 <= e; k += 4) {
        int c[4];
        Acc v[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            c[q] = cols[k + q];
            v[q] = (Acc)ld_val_cached(vals, k + q);
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) acc += v[q] * (Acc)xl[c[q]];
    }
    for (; k < e; ++k) acc += (Acc)ld_val_cached(vals, k) * (Acc)xl[cols[k]];
    return acc;
}

// The same on the caller's float64 matrix and a float64 vector, the first of
// its entries being column c0's; MODE 0: sum of a x, 1: sum of |a| x, 2:
// maximum of |a| x.
template <int MODE>
__device__ __forceinline__ double row_f64(const double* vals, const int32_t* cols, const double* x, int s, int e,
                                          int c0 = 0) {
    double acc = 0.0;
    for (int k = s; k < e; k += 4) {
        double v[4], g[4];
        int c[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int kk = min(k + q, e - 1);
            c[q] = cols[kk];
            v[q] = vals[kk];
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) g[q] = x[c[q] - c0];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            if (k + q >= e) continue;
            if (MODE == 0) acc += v[q] * g[q];
            else if (MODE == 1) acc += fabs(v[q]) * g[q];
            else acc = fmax(acc, fabs(v[q]) * g[q]);
        }
    }
    return acc;
}

// Largest instance dimension the 16-bit local columns address.
constexpr int kInstMaxDim = 65535;

// Limits of the level layout: rows and columns that the set-up sorts in LDS,
// and the longest row (a level offset each).  (Byte offsets into a vector of
// doubles and its extra entry fit 16 bits.)
constexpr int kLevelMaxDim = 8190;
constexpr int kLevelMaxLen = 1024;

// One scaled matrix of an instance.  In the level layout the rows are taken
// in the order of decreasing length ("positions"; equal lengths keep their
// order) and the entries are stored level by level: level k holds the k-th
// entry of every row longer than k, which are the first positions, so entry
// (p, k) is at kp[k] + p.  The lanes of a wave, on consecutive positions, read
// consecutive values and columns whatever the row lengths, with no padding,
// and every row is still summed in its own order.  The vectors of an instance
// (and the columns stored here) are by position too.  Thread t holds the
// first K entries of the rows at positions t, t + BS, ... (R of them) in
// registers for good (RegSide); the rest of the first K0 levels lies in LDS
// (entry (p, k) at kl[k] + p), the other levels are streamed from the
// workspace.  An instance beyond the limits above keeps CSR order
// (levels == false, positions = rows).  Offsets are bytes in the workgroup's
// dynamic LDS.
template <typename V>
struct Side {
    bool levels;
    int K0;
    int o_kp, o_kl, o_len, o_val, o_col;
    const V* val;           // the instance's entries in the workspace
    const uint16_t* col;
    const int32_t* rowptr;  // of the instance's first row (CSR order)
    int z0;                 // first entry of the instance
};

typedef int32_t ii2 __attribute__((ext_vector_type(2)));

// acc + the terms of position p from level k on (k even); len: its row's
// length.  Four levels are three trips to LDS, one after the other; LONG: one,
// the next four levels' columns and values and the offsets of those after being
// read under a group's gathers (see LongRows).
template <bool LONG, typename Acc, typename V, typename X>
__device__ __forceinline__ Acc side_rest(const Side<V>& s, const unsigned char* lds, const X* xl, int p, int len, int k,
                                         Acc acc) {
    const uint32_t* kp = (const uint32_t*)(lds + s.o_kp);
    const int32_t* kl = (const int32_t*)(lds + s.o_kl);
    const V* lv = (const V*)(lds + s.o_val);
    const uint16_t* lc = (const uint16_t*)(lds + s.o_col);
    const int kr = min(len, s.K0);
    if constexpr (LONG) {
        if (k + 4 <= kr) {
            ii2 oa = *(const ii2*)(kl + k), ob = *(const ii2*)(kl + k + 2);
            int c[4] = {lc[oa[0] + p], lc[oa[1] + p], lc[ob[0] + p], lc[ob[1] + p]};
            V v[4] = {lv[oa[0] + p], lv[oa[1] + p], lv[ob[0] + p], lv[ob[1] + p]};
            bool more = k + 8 <= kr;
            if (more) {
                oa = *(const ii2*)(kl + k + 4);
                ob = *(const ii2*)(kl + k + 6);
            }
            for (;;) {
                X x[4];
#pragma unroll
                for (int q = 0; q < 4; ++q) x[q] = xl[c[q]];
                // (the last group reads its own entries again)
                V w[4] = {lv[oa[0] + p], lv[oa[1] + p], lv[ob[0] + p], lv[ob[1] + p]};
                c[0] = lc[oa[0] + p];
                c[1] = lc[oa[1] + p];
                c[2] = lc[ob[0] + p];
                c[3] = lc[ob[1] + p];
                k += 4;
                const bool next = more;
                more = k + 8 <= kr;
                if (more) {
                    oa = *(const ii2*)(kl + k + 4);
                    ob = *(const ii2*)(kl + k + 6);
                }
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    acc += (Acc)ld_val_cached(&v[q], 0) * (Acc)x[q];
                    v[q] = w[q];
                }
                if (!next) break;
            }
        }
    }
    for (; k + 4 <= kr; k += 4) {
        const ii2 oa = *(const ii2*)(kl + k), ob = *(const ii2*)(kl + k + 2);
        const int o[4] = {oa[0], oa[1], ob[0], ob[1]};
        int c[4];
        Acc v[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            c[q] = lc[o[q] + p];
            v[q] = (Acc)ld_val_cached(lv, o[q] + p);
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) acc += v[q] * (Acc)xl[c[q]];
    }
    for (; k < kr; ++k) {
        const int e = kl[k] + p;
        acc += (Acc)ld_val_cached(lv, e) * (Acc)xl[lc[e]];
    }
    for (; k + 4 <= len; k += 4) {
        int c[4];
        Acc v[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int e = (int)kp[k + q] + p;
            c[q] = s.col[e];
            v[q] = (Acc)ld_val_cached(s.val, e);
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) acc += v[q] * (Acc)xl[c[q]];
    }
    for (; k < len; ++k) {
        const int e = (int)kp[k] + p;
        acc += (Acc)ld_val_cached(s.val, e) * (Acc)xl[s.col[e]];
    }
    return acc;
}

// The whole row at position p, none of it in registers; the positions below
// P0 have their first KK levels only in the workspace
template <bool LONG, typename Acc, typename V, typename X>
__device__ __forceinline__ Acc side_dot(const Side<V>& s, const unsigned char* lds, const X* xl, int p, int P0, int KK) {
    if (!s.levels) return row_dot4<Acc>(s.val, s.col, xl, s.rowptr[p] - s.z0, s.rowptr[p + 1] - s.z0);
    const int len = ((const uint16_t*)(lds + s.o_len))[p];
    Acc acc = 0;
    int k = 0;
    if (p < P0) {
        const uint32_t* kp = (const uint32_t*)(lds + s.o_kp);
        const int ke = min(len, KK);
        for (; k + 4 <= ke; k += 4) {
            int c[4];
            Acc v[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int e = (int)kp[k + q] + p;
                c[q] = s.col[e];
                v[q] = (Acc)ld_val_cached(s.val, e);
            }
#pragma unroll
            for (int q = 0; q < 4; ++q) acc += v[q] * (Acc)xl[c[q]];
        }
        for (; k < ke; ++k) {
            const int e = (int)kp[k] + p;
            acc += (Acc)ld_val_cached(s.val, e) * (Acc)xl[s.col[e]];
        }
        if (len <= KK) return acc;
    }
    return side_rest<LONG, Acc>(s, lds, xl, p, len, k, acc);
}

// Rows and entries per row that a thread holds: R rows of K entries, of which
// the columns are byte offsets into the gathered vector, two to a register.
// Absent entries are a zero value and the vector's extra zero entry.  Three
// columns of six and one row of sixteen entries are 51 registers in FP32, of
// the 128 that four waves to a SIMD leave a thread (the compiler spills 35 to
// 64 others in the iteration kernels and 41 to 82 in the reverse sweep; in FP32
// nearly all of that lies outside the loop).  16-bit values lie two to a
// register as well: with one each, 81 and 124 were spilled, in the loop too,
// and maps of near-dense instances took longer than from L2 (307 of 37 x 55, 30
// entries a column, K = 150: 3.62 ms from L2, 4.11, so 3.58; 4,096 LPs of 20 to
// 2,000 rows, 256 iterations: 31.7, 22.2, 16.7).
template <typename V, int R, int K, bool LONG = false>
struct RegSide {
    static constexpr bool kPacked = sizeof(V) == 2;
    typedef typename std::conditional<kPacked, uint32_t, V>::type W;
    static constexpr int KW = kPacked ? K / 2 : K;
    W v[R][KW];
    uint32_t c[R][K / 2];
    int len[R];
    // entry k of slot r
    __device__ __forceinline__ auto value(int r, int k) const {
        if constexpr (kPacked) return __uint_as_float((k & 1) ? v[r][k / 2] & 0xffff0000u : v[r][k / 2] << 16);
        else return v[r][k];
    }
    // Called in the loop that uses them: the entries as they are stored stay
    // in the registers (their conversions and offsets, computed ahead of the
    // loop, would take twice as many and spill)
    __device__ __forceinline__ void pin() {
#pragma unroll
        for (int r = 0; r < R; ++r) {
#pragma unroll
            for (int k = 0; k < KW; ++k) asm volatile("" : "+v"(v[r][k]));
#pragma unroll
            for (int k = 0; k < K / 2; ++k) asm volatile("" : "+v"(c[r][k]));
        }
    }
};
template <typename V>
struct RegShape {  // columns (rows of A^T) and rows (of A)
    static constexpr int RC = 3, KC = sizeof(V) == 8 ? 4 : 6;
    static constexpr int RR = 1, KR = sizeof(V) == 8 ? 8 : 16;
};

template <int BS, typename T, typename V, int R, int K, bool LONG>
__device__ __forceinline__ void reg_load(RegSide<V, R, K, LONG>& g, const Side<V>& s, const unsigned char* lds, int dim, int other) {
    const uint32_t* kp = (const uint32_t*)(lds + s.o_kp);
    const uint16_t* len = (const uint16_t*)(lds + s.o_len);
    const bool any = s.levels && len[0] > 0;  // uniform
    const uint32_t none = ((uint32_t)other * (uint32_t)sizeof(T)) & 0xffffu;
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int p = (int)threadIdx.x + r * BS;
        const int l = any && p < dim ? len[min(p, dim - 1)] : 0;
        g.len[r] = l;
        uint32_t c[K];
        V w[K];
        // (branch-free: absent entries load the instance's first one)
#pragma unroll
        for (int k = 0; k < K; ++k) {
            const int e = k < l ? (int)kp[k] + p : 0;
            const V v = any ? s.val[e] : (V)0;
            const uint32_t cc = any ? (uint32_t)s.col[e] * (uint32_t)sizeof(T) : none;
            w[k] = k < l ? v : (V)0;
            c[k] = k < l ? cc : none;
        }
#pragma unroll
        for (int k = 0; k < K; k += 2) g.c[r][k / 2] = c[k] | (c[k + 1] << 16);
        if constexpr (RegSide<V, R, K, LONG>::kPacked) {
#pragma unroll
            for (int k = 0; k < K; k += 2) g.v[r][k / 2] = (uint32_t)w[k] | ((uint32_t)w[k + 1] << 16);
        } else {
#pragma unroll
            for (int k = 0; k < K; ++k) g.v[r][k] = w[k];
        }
    }
}

// The first KE entries of register slot r: the gathers are issued together,
// the terms added in order
template <int KE, typename Acc, typename V, typename X, int R, int K, bool LONG>
__device__ __forceinline__ Acc reg_terms(const RegSide<V, R, K, LONG>& g, const X* xl, int r) {
    X x[KE];
#pragma unroll
    for (int k = 0; k < KE; ++k)
        x[k] = *(const X*)((const unsigned char*)xl + ((k & 1) ? g.c[r][k / 2] >> 16 : g.c[r][k / 2] & 0xffffu));
    Acc acc = 0;
#pragma unroll
    for (int k = 0; k < KE; ++k) acc += (Acc)g.value(r, k) * (Acc)x[k];
    return acc;
}

// The row of register slot r.  The wave's longest row is its first lane's, so
// a wave of short rows issues no more gathers than it needs, in steps.
template <typename Acc, typename V, typename X, int R, int K, bool LONG>
__device__ __forceinline__ Acc reg_dot(const RegSide<V, R, K, LONG>& g, const Side<V>& s, const unsigned char* lds,
                                       const X* xl, int r, int p) {
    const int longest = __builtin_amdgcn_readfirstlane(g.len[r]);
    if (K > 4 && longest <= 4) return reg_terms<(K > 4 ? 4 : K), Acc>(g, xl, r);
    if (K > 8 && longest <= 8) return reg_terms<(K > 8 ? 8 : K), Acc>(g, xl, r);
    if (K > 12 && longest <= 12) return reg_terms<(K > 12 ? 12 : K), Acc>(g, xl, r);
    Acc acc = reg_terms<K, Acc>(g, xl, r);
    if (longest > K) acc = side_rest<LONG, Acc>(s, lds, xl, p, g.len[r], K, acc);
    return acc;
}

// The value of a uniform number, in scalar registers: what is the same for
// the whole workgroup but comes from LDS or memory would else take a vector
// register each, and the iterations' matrix entries need those
__device__ __forceinline__ int uniform(int v) { return __builtin_amdgcn_readfirstlane(v); }
__device__ __forceinline__ double uniform(double v) {
    union {
        double d;
        int i[2];
    } u;
    u.d = v;
    u.i[0] = __builtin_amdgcn_readfirstlane(u.i[0]);
    u.i[1] = __builtin_amdgcn_readfirstlane(u.i[1]);
    return u.d;
}

__device__ __forceinline__ int64_t uniform64(int64_t v) {
    const uint32_t lo = (uint32_t)uniform((int)v), hi = (uint32_t)uniform((int)(v >> 32));
    return (int64_t)((uint64_t)hi << 32 | lo);
}

// v, computed anew: what depends on it is not moved out of the surrounding
// loops (addresses formed ahead of the iterations take registers from them)
__device__ __forceinline__ int opaque(int v) {
    asm volatile("" : "+v"(v));
    return v;
}

// Fixed-order sums over [0, count), whatever the workgroup's size BS (64, or
// 256 and more): 256 partial sums, i added to the partial i mod 256 in
// increasing order, then a butterfly over each 64 of them, then the four in
// order.  f(i, s) adds i's terms and must only read.  Every thread gets the
// sums; sh holds 4 NS doubles.  Starts with the workgroup in step, and ends
// with all of f's reads done.
template <int BS, int NS, class F>
__device__ __forceinline__ void inst_sums(int count, double* sh, double (&out)[NS], F f) {
    __syncthreads();
    if constexpr (BS < 256) {
#pragma unroll 1
        for (int w = 0; w < 4; ++w) {
            double s[NS];
#pragma unroll
            for (int q = 0; q < NS; ++q) s[q] = 0.0;
#pragma unroll 2
            for (int i = opaque(64 * w + (int)threadIdx.x); i < count; i += 256) f(i, s);
#pragma unroll
            for (int q = 0; q < NS; ++q) {
                const double v = wave_sum(s[q]);
                out[q] = uniform(w == 0 ? v : out[q] + v);
            }
        }
        __syncthreads();
    } else {
        if (threadIdx.x < 256) {
            double s[NS];
#pragma unroll
            for (int q = 0; q < NS; ++q) s[q] = 0.0;
#pragma unroll 4
            for (int i = opaque(threadIdx.x); i < count; i += 256) f(i, s);
#pragma unroll
            for (int q = 0; q < NS; ++q) {
                const double v = wave_sum(s[q]);
                if ((threadIdx.x & (kWave - 1)) == 0) sh[q * 4 + threadIdx.x / kWave] = v;
            }
        }
        __syncthreads();
#pragma unroll
        for (int q = 0; q < NS; ++q) out[q] = uniform(((sh[q * 4] + sh[q * 4 + 1]) + sh[q * 4 + 2]) + sh[q * 4 + 3]);
    }
}

// Maximum over the workgroup's threads; sh holds BS / 64 doubles.
template <int BS>
__device__ __forceinline__ double inst_max(double v, double* sh) {
#pragma unroll
    for (int o = kWave / 2; o > 0; o >>= 1) v = fmax(v, __shfl_xor(v, o, kWave));
    if constexpr (BS > kWave) {
        __syncthreads();
        if ((threadIdx.x & (kWave - 1)) == 0) sh[threadIdx.x / kWave] = v;
        __syncthreads();
        v = sh[0];
        for (int w = 1; w < BS / kWave; ++w) v = fmax(v, sh[w]);
    }
    return uniform(v);
}

struct InstMat {  // the caller's float64 block-diagonal LP
    const int32_t *a_rowptr, *a_col;
    const double* a_val;
    const int32_t *at_rowptr, *at_col;
    const double* at_val;
    const double *b, *c;
};

struct InstSetup {
    double b_norm, c_norm, sigma_hat, eta, omega0;
};

// What an instance keeps in the workspace beside its vectors: the scaled
// values and local columns of A and A^T in side order, and the rows at each
// position (perm, of rows and columns).
template <typename V>
struct InstStore {
    V *a_vs, *at_vs;
    uint16_t *a_cl, *at_cl, *perm_r, *perm_c;
};

// The instance a workgroup holds: sizes, its vectors in LDS (yl of m, xl of n,
// by position, each followed by a zero) and its two matrices.
template <typename T, typename V>
struct Inst {
    int r0, c0, m, n, z0, nnz;
    bool levels;
    const uint16_t *perm_r, *perm_c;
    T *yl, *xl;
    Side<V> A, AT;
    int o_scr;  // LDS scratch of max(m, n) doubles, or -1
    // the row (column) at position p, in the whole batch
    __device__ __forceinline__ int row(int p) const { return r0 + (levels ? (int)perm_r[p] : p); }
    __device__ __forceinline__ int column(int p) const { return c0 + (levels ? (int)perm_c[p] : p); }
};

__host__ __device__ inline int inst_align(int b) { return (b + 15) & ~15; }
__host__ __device__ inline int inst_pow2(int v) {
    int p = 1;
    while (p < v) p <<= 1;
    return p;
}
// LDS bytes of the vectors, and of the whole instance with its matrices and
// scratch (the levels' offsets taken at their mean length twice over, which
// only shapes the launch)
__host__ __device__ inline int inst_vec_bytes(int m, int n, int ts) {
    return inst_align((m + 1) * ts) + inst_align((n + 1) * ts);
}
// (nreg: the entries that threads hold in registers)
inline int64_t inst_full_bytes(int64_t m, int64_t n, int64_t nnz, int ts, int vs, int64_t nreg) {
    const int64_t lens = 2 * (m + n) + 16 * (nnz / (m > 0 ? m : 1) + nnz / (n > 0 ? n : 1)) + 320;
    const int64_t sort = 4 * (int64_t)inst_pow2((int)(m > n ? m : n)) + 4 * (m + n) + 128;
    const int64_t left = 2 * nnz > nreg ? 2 * nnz - nreg : 0;
    const int64_t rest = lens + 8 * (m > n ? m : n) + left * (vs + 2) + 128;
    return inst_vec_bytes((int)m, (int)n, ts) + (rest > sort ? rest : sort);
}

// Whether one wave is to run an m x n instance that a sixteenth of a compute
// unit's LDS holds, and not 256 threads; count: the instances that a quarter of
// it holds.  No more than one row and column to a lane, or more instances than
// 256-thread workgroups hold at once (four to a compute unit), where a wave
// keeps four times as many in flight.  256 iterations in FP32, one wave against
// 256 threads: 1,024 instances of 62 columns 1.15 and 1.15 ms, of 150 columns
// 1.67 and 1.43, of 200 columns 2.26 and 1.39; 2,048 of them 1.46 and 1.96,
// 1.96 and 2.35, 2.69 and 2.48; 4,096 1.91 and 3.50, 2.64 and 4.10, 3.52 and 4.45.
// (11 of 65 x 45, FP64: 1.55 and 1.24, the 65th row being a second pass.)
inline bool one_wave(int64_t count, int cus, int m, int n) {
    return (m > n ? m : n) <= kWave || count > 4 * (int64_t)cus;
}

// Whether a launch's instances take the LONG form of side_rest: where their rows
// go on past the registers for 8 entries on average.  FP32, 200 LPs
// of 200 rows and 400 columns, 256 iterations, without and with it: 8 entries a
// row 1.11 and 1.17 ms, 16 1.63 and 1.59, 24 2.05 and 1.91, 32 2.59 and 2.29; 64
// maps of the same, K = 150: 1.75 and 1.84, 2.43 and 2.42, 3.01 and 2.88, 3.69 and
// 3.40 (21 of 95 x 380, 64 entries a row: 5.01 and 4.19, from L2 4.62).  Not for
// values of eight bytes, whose registers it takes (64 maps in FP64, 16 entries a
// row 2.14 and 2.35, 24 2.70 and 2.74, 32 3.25 and 3.21), and not for long columns
// alone (31 LPs of 212 x 212, 16 entries a column and a row, 1.92 and 2.03).
template <typename V>
struct LongRows {
    static constexpr bool ok = sizeof(V) < 8;
    static bool pays(int64_t m, int64_t nnz) { return ok && nnz >= m * (RegShape<V>::KR + 8); }
};

// perm <- the positions' rows: rows by decreasing length, equal lengths in
// order (a bitonic sort of (length, row) keys in LDS, skipped when all
// lengths are equal)
template <int BS>
__device__ void inst_sort(const int32_t* rowptr, int dim, uint32_t* keys, uint16_t* perm, double* sh) {
    const int tid = threadIdx.x;
    double mx = 0.0, mn = 0.0;
    for (int i = tid; i < dim; i += BS) {
        const double l = (double)(rowptr[i + 1] - rowptr[i]);
        mx = fmax(mx, l);
        mn = fmax(mn, 65536.0 - l);
    }
    mx = inst_max<BS>(mx, sh);
    mn = 65536.0 - inst_max<BS>(mn, sh);
    if (mx == mn) {  // uniform
        for (int i = tid; i < dim; i += BS) perm[i] = (uint16_t)i;
        return;
    }
    const int P = inst_pow2(dim);
    for (int i = tid; i < P; i += BS)
        keys[i] = i < dim ? ((0xffffu - (uint32_t)(rowptr[i + 1] - rowptr[i])) << 16) | (uint32_t)i : 0xffffffffu;
    __syncthreads();
    for (int k = 2; k <= P; k <<= 1)
        for (int j = k >> 1; j > 0; j >>= 1) {
            for (int i = tid; i < P; i += BS) {
                const int l = i ^ j;
                if (l > i) {
                    const uint32_t a = keys[i], b = keys[l];
                    if ((a > b) == ((i & k) == 0)) {
                        keys[i] = b;
                        keys[l] = a;
                    }
                }
            }
            __syncthreads();
        }
    for (int i = tid; i < dim; i += BS) perm[i] = (uint16_t)(keys[i] & 0xffffu);
    __syncthreads();
}

// Lengths by position and level offsets of one side in LDS (kp of the
// workspace, kl of the entries that LDS holds: below level KK those from
// position P0 on), o: the next free byte (advanced); returns the number of
// levels.
template <int BS, typename V>
__device__ int inst_levels(const int32_t* rowptr, const uint16_t* perm, int dim, int P0, int KK, unsigned char* lds,
                           int& o, Side<V>& s) {
    const int tid = threadIdx.x;
    s.o_len = o;
    uint16_t* len = (uint16_t*)(lds + s.o_len);
    o = inst_align(o + 2 * dim);
    for (int p = tid; p < dim; p += BS) len[p] = (uint16_t)(rowptr[perm[p] + 1] - rowptr[perm[p]]);
    __syncthreads();
    const int K = uniform((int)len[0]);
    s.o_kp = o;
    uint32_t* kp = (uint32_t*)(lds + s.o_kp);
    o = inst_align(o + 4 * (K + 4));
    s.o_kl = o;
    int32_t* kl = (int32_t*)(lds + s.o_kl);
    o = inst_align(o + 4 * (K + 4));
    // rows longer than k, then the running sums
    for (int p = tid; p < dim; p += BS) {
        const int lo = p + 1 < dim ? len[p + 1] : 0;
        for (int k = lo; k < len[p]; ++k) kp[k + 1] = (uint32_t)(p + 1);
    }
    if (tid == 0) kp[0] = 0;
    __syncthreads();
    if (tid < kWave) {
        int carry = 0, carry_l = 0;
        for (int b = 0; b <= K; b += kWave) {
            const int k = b + tid;
            int v = k <= K ? (int)kp[k] : 0;
            int l = k > 0 && k - 1 < KK ? max(v - P0, 0) : v;
#pragma unroll
            for (int d = 1; d < kWave; d <<= 1) {
                const int u = __shfl_up(v, d, kWave), ul = __shfl_up(l, d, kWave);
                if (tid >= d) {
                    v += u;
                    l += ul;
                }
            }
            v += carry;
            l += carry_l;
            if (k <= K) {
                kp[k] = (uint32_t)v;
                kl[k] = l - (k < KK && k < K ? P0 : 0);
            }
            carry = __shfl(v, kWave - 1, kWave);
            carry_l = __shfl(l, kWave - 1, kWave);
        }
    }
    __syncthreads();
    return K;
}

// The workgroup's LDS for instance I (sizes and vectors set): the vectors'
// zero entries, lengths, level offsets, and, as far as `budget` bytes go, the
// scratch and what the threads' registers leave of the first levels of A^T
// and A, copied from the workspace if fill; in CSR order only the scratch.
template <typename T, typename V, int BS>
__device__ void inst_load(Inst<T, V>& I, const InstMat& M, const InstStore<V>& S, unsigned char* lds, int budget,
                          bool fill) {
    typedef RegShape<V> RS;
    int o = inst_vec_bytes(I.m, I.n, sizeof(T));
    if (threadIdx.x == 0) {
        I.yl[I.m] = (T)0;
        I.xl[I.n] = (T)0;
    }
    I.A.levels = I.AT.levels = I.levels;
    I.A.rowptr = M.a_rowptr + I.r0;
    I.AT.rowptr = M.at_rowptr + I.c0;
    I.A.z0 = I.AT.z0 = I.z0;
    I.A.val = S.a_vs + I.z0;
    I.AT.val = S.at_vs + I.z0;
    I.A.col = S.a_cl + I.z0;
    I.AT.col = S.at_cl + I.z0;
    I.A.K0 = I.AT.K0 = 0;
    I.A.o_kp = I.A.o_kl = I.A.o_len = I.A.o_val = I.A.o_col = 0;
    I.AT.o_kp = I.AT.o_kl = I.AT.o_len = I.AT.o_val = I.AT.o_col = 0;
    int KA = 0, KT = 0;
    if (I.levels) {
        KA = inst_levels<BS>(I.A.rowptr, I.perm_r, I.m, RS::RR * BS, RS::KR, lds, o, I.A);
        KT = inst_levels<BS>(I.AT.rowptr, I.perm_c, I.n, RS::RC * BS, RS::KC, lds, o, I.AT);
    }
    const int scr = 8 * max(I.m, I.n);
    I.o_scr = -1;
    int64_t left = 0;  // entries beside those in registers
    if (I.levels)
        left = (int64_t)((const int32_t*)(lds + I.A.o_kl))[KA] + ((const int32_t*)(lds + I.AT.o_kl))[KT];
    left = uniform((int)left);
    const bool all = o + scr + left * ((int)sizeof(V) + 2) + 96 <= budget;
    if (all || (o + scr <= budget && 6 * scr <= budget)) {  // otherwise the matrix needs the room more
        I.o_scr = o;
        o = inst_align(o + scr);
    }
    if (!I.levels) return;
    auto take = [&](Side<V>& s, int K, int P0, int KK) {
        // kl[k] + p is level k's entry: its first position in LDS is P0 below level KK
        const int32_t* kl = (const int32_t*)(lds + s.o_kl);
        const int room = max(0, budget - o - 32) / ((int)sizeof(V) + 2);
        auto first = [&](int k) { return kl[k] + (k < KK && k < K ? P0 : 0); };
        int k0 = K;
        if (first(K) > room) {  // whole groups of four levels
            k0 = K & ~3;
            while (k0 > 0 && first(k0) > room) k0 -= 4;
        }
        const int z = uniform(first(k0));
        s.K0 = uniform(k0);
        s.o_val = o;
        o = inst_align(o + z * (int)sizeof(V));
        s.o_col = o;
        o = inst_align(o + z * 2);
    };
    take(I.AT, KT, RS::RC * BS, RS::KC);
    take(I.A, KA, RS::RR * BS, RS::KR);
    if (!fill) return;
    auto copy = [&](const Side<V>& s, int P0, int KK, int dim) {
        const uint32_t* kp = (const uint32_t*)(lds + s.o_kp);
        const int32_t* kl = (const int32_t*)(lds + s.o_kl);
        V* v = (V*)(lds + s.o_val);
        uint16_t* c = (uint16_t*)(lds + s.o_col);
        for (int k = 0; k < s.K0; ++k) {
            const int cnt = (int)(kp[k + 1] - kp[k]);
            for (int p = (k < KK ? P0 : 0) + (int)threadIdx.x; p < cnt; p += BS) {
                v[kl[k] + p] = s.val[kp[k] + p];
                c[kl[k] + p] = s.col[kp[k] + p];
            }
        }
    };
    copy(I.AT, RS::RC * BS, RS::KC, I.n);
    copy(I.A, RS::RR * BS, RS::KR, I.m);
    __syncthreads();
}

// f(p, r, sum) for every row at position p of one side, its sum over the
// gathered vector xl: the rows in registers (slot r), then the others (r = -1).
// A wave leaves out the slots whose positions all lie past the end.
template <int BS, int R, typename Acc, typename V, typename X, int K, bool LONG, class F>
__device__ __forceinline__ void inst_rows(bool levels, int dim, const RegSide<V, R, K, LONG>& g, const Side<V>& s,
                                          const unsigned char* lds, const X* xl, F f) {
    const int tid = threadIdx.x;
    const int w0 = __builtin_amdgcn_readfirstlane(tid & ~(kWave - 1));
    int p = opaque(tid);
    if (levels) {
#pragma unroll
        for (int r = 0; r < R; ++r) {
            if (w0 + r * BS >= dim) return;
            const int pr = tid + r * BS;
            const Acc a = reg_dot<Acc>(g, s, lds, xl, r, pr);
            if (pr < dim) f(pr, r, a);
        }
        p += R * BS;
    }
    for (; p < dim; p += BS) f(p, -1, side_dot<LONG, Acc>(s, lds, xl, p, 0, 0));
}

template <typename V>
__device__ __forceinline__ void put_scaled(V* out, int64_t k, double v) {
    if constexpr (sizeof(V) == 2) out[k] = f32_to_bf16_rne((float)v);
    else out[k] = (V)v;
}

// Sets up the instance with rows [r0, r1), columns [c0, c1) by a workgroup of
// BS threads with `budget` bytes of LDS.  Writes D_r, D_c (float64), the scaled
// values of the instance's entries of A and A^T (type V) with their local
// columns in side order, b~ and c~ by position (type T), fills I, and returns
// the norms, sigma_hat, eta and omega_0.  pu[n], pav[m] are float64 scratch
// vectors of the whole batch.  The results do not depend on BS.
template <typename T, typename V, int BS>
__device__ InstSetup inst_setup(Inst<T, V>& I, const InstMat& M, const InstStore<V>& S, double* d_row, double* d_col,
                                double* pu, double* pav, T* bt, T* ct, int ruiz, int pc, int power_iters,
                                double step_safety, unsigned char* lds, int budget, double* sh) {
    const int tid = threadIdx.x;
    const int r0 = I.r0, c0 = I.c0, m = I.m, n = I.n;
    const int32_t *arp = M.a_rowptr + r0, *trp = M.at_rowptr + c0;

    // norms of b and c
    double nb[1], nc[1];
    inst_sums<BS, 1>(m, sh, nb, [&](int i, double(&s)[1]) { s[0] += M.b[r0 + i] * M.b[r0 + i]; });
    inst_sums<BS, 1>(n, sh, nc, [&](int j, double(&s)[1]) { s[0] += M.c[c0 + j] * M.c[c0 + j]; });
    const double b_norm = sqrt(nb[0]), c_norm = sqrt(nc[0]);

    // the layout: levels if every row and column is short enough and the
    // sort's keys fit
    double mx = 0.0;
    for (int i = tid; i < m; i += BS) mx = fmax(mx, (double)(arp[i + 1] - arp[i]));
    for (int j = tid; j < n; j += BS) mx = fmax(mx, (double)(trp[j + 1] - trp[j]));
    mx = inst_max<BS>(mx, sh);
    const int big = max(m, n);
    const int o_tmp = inst_vec_bytes(m, n, sizeof(T));
    // (the level offsets of both sides are at most 16 (mx + 4) bytes)
    const int longest = uniform((int)mx);
    I.levels = mx <= (double)kLevelMaxLen && big <= kLevelMaxDim &&
               o_tmp + max(4 * inst_pow2(big) + 64, 2 * (m + n) + 16 * (longest + 4) + 160) + 2 * (m + n) <= budget;
    if (I.levels) {
        uint32_t* keys = (uint32_t*)(lds + o_tmp);
        inst_sort<BS>(arp, m, keys, S.perm_r + r0, sh);
        __syncthreads();
        inst_sort<BS>(trp, n, keys, S.perm_c + c0, sh);
        __syncthreads();
    }
    I.perm_r = S.perm_r + r0;
    I.perm_c = S.perm_c + c0;

    // scaling: Ruiz infinity-norm passes, then one Pock-Chambolle pass
    // (D_r and D_c of a pass and of the next in LDS where they fit: what bounds
    // a pass is the latency of a row's range, entries and gathers, one after
    // the other; in the workspace the gathers are L2 accesses)
    const int passes = ruiz + (pc ? 1 : 0);
    if (16 * (m + n) <= budget) {
        double* cur = (double*)lds;
        double* nxt = cur + m + n;
        __syncthreads();
        for (int i = tid; i < m + n; i += BS) cur[i] = 1.0;
        __syncthreads();
        for (int ps = 0; ps < passes; ++ps) {
            const bool mxm = ps < ruiz;
            auto scale = [&](int i, double acc) {
                const double s = cur[i] * acc;
                nxt[i] = s > 0.0 ? cur[i] * (1.0 / sqrt(s)) : cur[i];
            };
            for (int i = tid; i < m; i += BS)
                scale(i, mxm ? row_f64<2>(M.a_val, M.a_col, cur + m, arp[i], arp[i + 1], c0)
                             : row_f64<1>(M.a_val, M.a_col, cur + m, arp[i], arp[i + 1], c0));
            for (int j = tid; j < n; j += BS)
                scale(m + j, mxm ? row_f64<2>(M.at_val, M.at_col, cur, trp[j], trp[j + 1], r0)
                                 : row_f64<1>(M.at_val, M.at_col, cur, trp[j], trp[j + 1], r0));
            __syncthreads();
            double* t = cur;
            cur = nxt;
            nxt = t;
        }
        for (int i = tid; i < m; i += BS) d_row[r0 + i] = cur[i];
        for (int j = tid; j < n; j += BS) d_col[c0 + j] = cur[m + j];
        __syncthreads();
    } else {
        for (int i = tid; i < m; i += BS) d_row[r0 + i] = 1.0;
        for (int j = tid; j < n; j += BS) d_col[c0 + j] = 1.0;
        __syncthreads();
        double *stat_r = pav, *stat_c = pu;
        for (int ps = 0; ps < passes; ++ps) {
            const bool mxm = ps < ruiz;
            for (int i = tid; i < m; i += BS) {
                const double acc = mxm ? row_f64<2>(M.a_val, M.a_col, d_col, arp[i], arp[i + 1])
                                       : row_f64<1>(M.a_val, M.a_col, d_col, arp[i], arp[i + 1]);
                stat_r[r0 + i] = d_row[r0 + i] * acc;
            }
            for (int j = tid; j < n; j += BS) {
                const double acc = mxm ? row_f64<2>(M.at_val, M.at_col, d_row, trp[j], trp[j + 1])
                                       : row_f64<1>(M.at_val, M.at_col, d_row, trp[j], trp[j + 1]);
                stat_c[c0 + j] = d_col[c0 + j] * acc;
            }
            __syncthreads();
            for (int i = tid; i < m; i += BS) {
                const double s = stat_r[r0 + i];
                if (s > 0.0) d_row[r0 + i] *= 1.0 / sqrt(s);
            }
            for (int j = tid; j < n; j += BS) {
                const double s = stat_c[c0 + j];
                if (s > 0.0) d_col[c0 + j] *= 1.0 / sqrt(s);
            }
            __syncthreads();
        }
    }

    // scaled values in the iteration precision, in side order
    if (I.levels) {
        inst_load<T, V, BS>(I, M, S, lds, budget, false);
        // positions of the rows and columns, in LDS that the sides' copies take over afterwards
        uint16_t* pos_r = (uint16_t*)(lds + budget - 2 * (m + n));
        uint16_t* pos_c = pos_r + m;
        for (int p = tid; p < m; p += BS) pos_r[I.perm_r[p]] = (uint16_t)p;
        for (int p = tid; p < n; p += BS) pos_c[I.perm_c[p]] = (uint16_t)p;
        __syncthreads();
        const uint32_t* kpa = (const uint32_t*)(lds + I.A.o_kp);
        const uint32_t* kpt = (const uint32_t*)(lds + I.AT.o_kp);
        for (int p = tid; p < m; p += BS) {
            const int i = I.perm_r[p], s = arp[i], len = arp[i + 1] - s;
            const double dr = d_row[r0 + i];
            for (int k = 0; k < len; ++k) {
                const int j = M.a_col[s + k];
                const int64_t e = (int64_t)I.z0 + kpa[k] + p;
                put_scaled(S.a_vs, e, dr * M.a_val[s + k] * d_col[j]);
                S.a_cl[e] = pos_c[j - c0];
            }
        }
        for (int p = tid; p < n; p += BS) {
            const int j = I.perm_c[p], s = trp[j], len = trp[j + 1] - s;
            const double dc = d_col[c0 + j];
            for (int k = 0; k < len; ++k) {
                const int i = M.at_col[s + k];
                const int64_t e = (int64_t)I.z0 + kpt[k] + p;
                put_scaled(S.at_vs, e, dc * M.at_val[s + k] * d_row[i]);
                S.at_cl[e] = pos_r[i - r0];
            }
        }
    } else {
        for (int i = tid; i < m; i += BS) {
            const double dr = d_row[r0 + i];
            for (int k = arp[i]; k < arp[i + 1]; ++k) {
                const int j = M.a_col[k];
                put_scaled(S.a_vs, k, dr * M.a_val[k] * d_col[j]);
                S.a_cl[k] = (uint16_t)(j - c0);
            }
        }
        for (int j = tid; j < n; j += BS) {
            const double dc = d_col[c0 + j];
            for (int k = trp[j]; k < trp[j + 1]; ++k) {
                const int i = M.at_col[k];
                put_scaled(S.at_vs, k, dc * M.at_val[k] * d_row[i]);
                S.at_cl[k] = (uint16_t)(i - r0);
            }
        }
    }
    __syncthreads();
    inst_load<T, V, BS>(I, M, S, lds, budget, true);
    // b~ and c~ by position, their norms in float64
    for (int p = tid; p < m; p += BS) {
        const int g = I.row(p);
        bt[r0 + p] = (T)(d_row[g] * M.b[g]);
    }
    for (int p = tid; p < n; p += BS) {
        const int g = I.column(p);
        ct[c0 + p] = (T)(d_col[g] * M.c[g]);
    }
    inst_sums<BS, 1>(m, sh, nb, [&](int i, double(&s)[1]) {
        const double v = d_row[r0 + i] * M.b[r0 + i];
        s[0] += v * v;
    });
    inst_sums<BS, 1>(n, sh, nc, [&](int j, double(&s)[1]) {
        const double v = d_col[c0 + j] * M.c[c0 + j];
        s[0] += v * v;
    });
    const double nbt = sqrt(nb[0]), nct = sqrt(nc[0]);

    // power iteration on the scaled iteration copy (the values and 16-bit
    // columns the iterations apply), as in the single-LP solve: vectors in
    // the iterate type, held in LDS (v in xl, A~ v in yl), products and sums
    // in float64.  u = A~^T (A~ v) overwrites v, which it no longer needs.
    // The float64 entries pass through the scratch to be summed in order.
    T *xl = I.xl, *yl = I.yl;
    double* const scr = (double*)(lds + max(I.o_scr, 0));
    typedef RegShape<V> RS;
    RegSide<V, RS::RC, RS::KC> gt;
    RegSide<V, RS::RR, RS::KR> ga;
    reg_load<BS, T>(gt, I.AT, lds, n, m);
    reg_load<BS, T>(ga, I.A, lds, m, n);
    int ir[RS::RR], jc[RS::RC];  // the rows and columns of the register slots
#pragma unroll
    for (int r = 0; r < RS::RR; ++r) ir[r] = I.row(min(tid + r * BS, m - 1)) - r0;
#pragma unroll
    for (int r = 0; r < RS::RC; ++r) jc[r] = I.column(min(tid + r * BS, n - 1)) - c0;
    for (int p = tid; p < n; p += BS) xl[p] = (T)(1.0 / sqrt((double)n));
    __syncthreads();
    double h = 0.0, h_m10 = 0.0;
    for (int kk = 0; kk <= power_iters; ++kk) {
        double s[1];
        ga.pin();
        gt.pin();
        inst_rows<BS, RS::RR, double>(I.levels, m, ga, I.A, lds, xl, [&](int p, int r, double t) {
            yl[p] = (T)t;
            const int i = r >= 0 ? ir[r] : I.row(p) - r0;
            if (I.o_scr >= 0) scr[i] = t;
            else pav[r0 + i] = t;
        });
        if (I.o_scr >= 0) inst_sums<BS, 1>(m, sh, s, [&](int i, double(&q)[1]) { q[0] += scr[i] * scr[i]; });
        else inst_sums<BS, 1>(m, sh, s, [&](int i, double(&q)[1]) { q[0] += pav[r0 + i] * pav[r0 + i]; });
        h = sqrt(s[0]);
        if (kk == power_iters - 10) h_m10 = h;
        if (kk == power_iters) break;
        inst_rows<BS, RS::RC, double>(I.levels, n, gt, I.AT, lds, yl, [&](int p, int r, double t) {
            xl[p] = (T)t;
            const int j = r >= 0 ? jc[r] : I.column(p) - c0;
            if (I.o_scr >= 0) scr[j] = t;
            else pu[c0 + j] = t;
        });
        if (I.o_scr >= 0) inst_sums<BS, 1>(n, sh, s, [&](int j, double(&q)[1]) { q[0] += scr[j] * scr[j]; });
        else inst_sums<BS, 1>(n, sh, s, [&](int j, double(&q)[1]) { q[0] += pu[c0 + j] * pu[c0 + j]; });
        const double nu = sqrt(s[0]);
        if (nu != 0.0)
            for (int p = tid; p < n; p += BS) xl[p] = (T)((double)xl[p] / nu);
        __syncthreads();
    }
    const double sigma_hat = h;
    double eta;
    if (sigma_hat <= 0.0) eta = step_safety;
    else if (pc && power_iters >= 10 && fabs(h - h_m10) > 1e-3 * h) eta = step_safety;
    else eta = step_safety / sigma_hat;
    const double omega0 = (nbt > 1e-10 && nct > 1e-10) ? nct / nbt : 1.0;
    InstSetup out;
    out.b_norm = b_norm;
    out.c_norm = c_norm;
    out.sigma_hat = sigma_hat;
    out.eta = eta;
    out.omega0 = omega0;
    return out;
}

}  // namespace mip
