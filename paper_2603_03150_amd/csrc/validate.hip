// Input validation shared by the single and batched solves: column ranges,
// finiteness, and a dot-product test that A^T is the transpose of A.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <vector>

#include "common.h"
#include "plain.h"

namespace mip {

// flags: bit0 column index out of range, bit1 non-finite value, bit2 non-finite b/c
__global__ void k_check_entries(const int32_t* col, const double* val, int64_t nnz, int32_t ncols,
                                int32_t* flags) {
    int f = 0;
    for (int64_t k = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; k < nnz;
         k += (int64_t)gridDim.x * blockDim.x) {
        int32_t j = col[k];
        if (j < 0 || j >= ncols) f |= 1;
        if (!isfinite(val[k])) f |= 2;
    }
    if (f) atomicOr(flags, f);
}

__global__ void k_check_vec(const double* v, int64_t n, int32_t* flags) {
    int f = 0;
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x)
        if (!isfinite(v[i])) f |= 4;
    if (f) atomicOr(flags, f);
}

// general form: bit3 a bound is NaN, lo = +inf, hi = -inf or lo > hi;
// bit4 a row sense outside {0, 1, 2}
__global__ void k_check_bounds(const double* lo, const double* hi, int64_t n, int32_t* flags) {
    int f = 0;
    for (int64_t j = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; j < n; j += (int64_t)gridDim.x * blockDim.x) {
        const double l = lo ? lo[j] : 0.0, u = hi ? hi[j] : INFINITY;
        if (!(l <= u) || l == INFINITY || u == -INFINITY) f |= 8;  // NaN fails l <= u
    }
    if (f) atomicOr(flags, f);
}

__global__ void k_check_sense(const int8_t* sense, int64_t m, int32_t* flags) {
    int f = 0;
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < m; i += (int64_t)gridDim.x * blockDim.x)
        if (sense[i] < 0 || sense[i] > 2) f |= 16;
    if (f) atomicOr(flags, f);
}

__device__ __forceinline__ double hash_unit(uint32_t i, uint32_t seed) {
    uint32_t h = i * 0x9E3779B1u ^ seed;
    h ^= h >> 16;
    h *= 0x85EBCA6Bu;
    h ^= h >> 13;
    h *= 0xC2B2AE35u;
    h ^= h >> 16;
    return (double)h * (2.0 / 4294967296.0) - 1.0;  // [-1, 1)
}

// With u = hash(row), v = hash(col): partial sums of u_r (M v)_r (ABS = false)
// or of |u_r| sum_c |M_rc v_c| (ABS = true) over the rows of M.
template <bool ABS>
__global__ __launch_bounds__(kBlock) void k_transpose_dot(TilePlan p, const int32_t* col, const double* val,
                                                          uint32_t seed_row, uint32_t seed_col, double* partials) {
    extern __shared__ __align__(16) unsigned char smem_t[];
    const auto L = tile_lds<double>(smem_t, p);
    double s[1] = {0.0};
    double mx[1] = {0.0};
    auto prod = [&](int b, int j) {
        const int64_t k = (int64_t)b + j;
        const double t = val[k] * hash_unit((uint32_t)col[k], seed_col);
        return ABS ? fabs(t) : t;
    };
    auto epi = [&](int r, double t) {
        const double u = hash_unit((uint32_t)r, seed_row);
        s[0] += (ABS ? fabs(u) : u) * t;
    };
    auto le = lepi(epi);
    tiled_rows<false>(p, own_tile(), L, prod, le);
    block_reduce_store<1, 0>(s, mx, partials + blockIdx.x);
}

__global__ __launch_bounds__(kBlock) void k_sum_partials(const double* partials, int G, double* out) {
    __shared__ double sh[kBlock];
    double s = 0.0;
    for (int g = threadIdx.x; g < G; g += kBlock) s += partials[g];
    sh[threadIdx.x] = s;
    __syncthreads();
    for (int st = kBlock / 2; st > 0; st >>= 1) {
        if (threadIdx.x < st) sh[threadIdx.x] += sh[threadIdx.x + st];
        __syncthreads();
    }
    if (threadIdx.x == 0) *out = sh[0];
}

// Order-independent 64-bit hash of a column index array: the wrapping sum
// over k of a mix of (k, col[k]) (integer adds commute, so the result does
// not depend on the launch).
__device__ __forceinline__ uint64_t mix64(uint64_t v) {
    v ^= v >> 33;
    v *= 0xff51afd7ed558ccdull;
    v ^= v >> 33;
    v *= 0xc4ceb9fe1a85ec53ull;
    v ^= v >> 33;
    return v;
}

__global__ void k_hash_cols(const int32_t* col, int64_t nnz, unsigned long long* out) {
    uint64_t h = 0;
    for (int64_t k = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; k < nnz; k += (int64_t)gridDim.x * blockDim.x)
        h += mix64(((uint64_t)k << 32) ^ (uint32_t)col[k]);
    for (int o = kWave / 2; o > 0; o >>= 1) h += __shfl_xor(h, o, kWave);
    if ((threadIdx.x & (kWave - 1)) == 0) atomicAdd(out, (unsigned long long)h);
}

int column_hash(const int32_t* col, int64_t nnz, uint64_t* scratch, hipStream_t stream, uint64_t* out) {
    MIP_HIP(hipMemsetAsync(scratch, 0, 8, stream));
    if (nnz > 0)
        hipLaunchKernelGGL(k_hash_cols, dim3(grid_for(nnz)), dim3(kBlock), 0, stream, col, nnz,
                           (unsigned long long*)scratch);
    MIP_LAUNCH_CHECK();
    MIP_HIP(hipMemcpyAsync(out, scratch, 8, hipMemcpyDeviceToHost, stream));
    MIP_HIP(hipStreamSynchronize(stream));
    return 0;
}

int allow_validate_lds(int bytes) {
    if (bytes <= 65536) return 0;
    if (hipFuncSetAttribute((const void*)k_transpose_dot<false>, hipFuncAttributeMaxDynamicSharedMemorySize, bytes) !=
            hipSuccess ||
        hipFuncSetAttribute((const void*)k_transpose_dot<true>, hipFuncAttributeMaxDynamicSharedMemorySize, bytes) !=
            hipSuccess)
        return set_error("tile shape needs %d bytes of LDS per workgroup, more than the device allows", bytes),
               MIPDHG_ERR_UNSUPPORTED;
    return 0;
}

int validate_device(const mipdhg_lp& lp, const TilePlan& ta, const TilePlan& tat, int32_t* flags,
                    double* partials, double* red, hipStream_t stream) {
    const int64_t nnz = lp.nnz;
    MIP_HIP(hipMemsetAsync(flags, 0, 4, stream));
    if (nnz > 0) {
        hipLaunchKernelGGL(k_check_entries, dim3(grid_for(nnz)), dim3(kBlock), 0, stream, lp.a_col, lp.a_val, nnz,
                           lp.n, flags);
        hipLaunchKernelGGL(k_check_entries, dim3(grid_for(nnz)), dim3(kBlock), 0, stream, lp.at_col, lp.at_val,
                           nnz, lp.m, flags);
    }
    hipLaunchKernelGGL(k_check_vec, dim3(grid_for(lp.m)), dim3(kBlock), 0, stream, lp.b, (int64_t)lp.m, flags);
    hipLaunchKernelGGL(k_check_vec, dim3(grid_for(lp.n)), dim3(kBlock), 0, stream, lp.c, (int64_t)lp.n, flags);
    if (has_bounds(lp))
        hipLaunchKernelGGL(k_check_bounds, dim3(grid_for(lp.n)), dim3(kBlock), 0, stream, lp.lo, lp.hi,
                           (int64_t)lp.n, flags);
    if (has_sense(lp))
        hipLaunchKernelGGL(k_check_sense, dim3(grid_for(lp.m)), dim3(kBlock), 0, stream, lp.sense, (int64_t)lp.m,
                           flags);
    MIP_LAUNCH_CHECK();
    int32_t f = 0;
    MIP_HIP(hipMemcpyAsync(&f, flags, 4, hipMemcpyDeviceToHost, stream));
    MIP_HIP(hipStreamSynchronize(stream));
    if (f & 1) return set_error("column index out of range"), MIPDHG_ERR_BAD_CSR;
    if (f & 6) return set_error("NaN or Inf in A, A^T, b or c"), MIPDHG_ERR_NONFINITE;
    if (f & 8) return set_error("a bound is NaN, lo = +inf, hi = -inf or lo > hi"), MIPDHG_ERR_INVALID_ARG;
    if (f & 16) return set_error("a row sense is not 0, 1 or 2"), MIPDHG_ERR_INVALID_ARG;
    if (nnz == 0) return 0;
    // u^T (A v) against v^T (A^T u), and the scale sum |u||A||v|
    const uint32_t su = 0x1234u, sv = 0xABCDu;
    hipLaunchKernelGGL((k_transpose_dot<false>), dim3(ta.ntiles), dim3(kBlock), tile_lds_bytes(ta, 8), stream, ta, lp.a_col,
                       lp.a_val, su, sv, partials);
    hipLaunchKernelGGL(k_sum_partials, dim3(1), dim3(kBlock), 0, stream, (const double*)partials, ta.ntiles, red);
    hipLaunchKernelGGL((k_transpose_dot<true>), dim3(ta.ntiles), dim3(kBlock), tile_lds_bytes(ta, 8), stream, ta, lp.a_col,
                       lp.a_val, su, sv, partials);
    hipLaunchKernelGGL(k_sum_partials, dim3(1), dim3(kBlock), 0, stream, (const double*)partials, ta.ntiles,
                       red + 1);
    hipLaunchKernelGGL((k_transpose_dot<false>), dim3(tat.ntiles), dim3(kBlock), tile_lds_bytes(tat, 8), stream, tat, lp.at_col,
                       lp.at_val, sv, su, partials);
    hipLaunchKernelGGL(k_sum_partials, dim3(1), dim3(kBlock), 0, stream, (const double*)partials, tat.ntiles,
                       red + 2);
    hipLaunchKernelGGL((k_transpose_dot<true>), dim3(tat.ntiles), dim3(kBlock), tile_lds_bytes(tat, 8), stream, tat, lp.at_col,
                       lp.at_val, sv, su, partials);
    hipLaunchKernelGGL(k_sum_partials, dim3(1), dim3(kBlock), 0, stream, (const double*)partials, tat.ntiles,
                       red + 3);
    MIP_LAUNCH_CHECK();
    double r[4];
    MIP_HIP(hipMemcpyAsync(r, red, 4 * 8, hipMemcpyDeviceToHost, stream));
    MIP_HIP(hipStreamSynchronize(stream));
    const double scale = std::max(r[1], r[3]);
    if (!(fabs(r[0] - r[2]) <= 1e-10 * scale + 1e-300))
        return set_error("A^T does not match A (dot test %.17g vs %.17g)", r[0], r[2]), MIPDHG_ERR_TRANSPOSE;
    return 0;
}

// ---------------------------------------------------------------------------
// batches: row pointers and entries of a block-diagonal pair, on the device
// ---------------------------------------------------------------------------
// bit64: the row pointer does not start at 0, end at nnz or rises nowhere
// down; bit128: it differs from nnz_off at an instance's first row
__global__ void k_check_rowptr(const int32_t* rowptr, int32_t nrows, int64_t nnz, const int32_t* off,
                               const int64_t* nnz_off, int B, int32_t* flags) {
    int f = 0;
    const int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x, step = (int64_t)gridDim.x * blockDim.x;
    for (int64_t r = t; r < nrows; r += step)
        if (rowptr[r + 1] < rowptr[r]) f |= 64;
    if (t == 0 && (rowptr[0] != 0 || (int64_t)rowptr[nrows] != nnz)) f |= 64;
    for (int64_t i = t; i <= B; i += step)
        if ((int64_t)rowptr[off[i]] != nnz_off[i]) f |= 128;
    if (f) atomicOr(flags, f);
}

// the largest i in [lo, hi] with a[i] <= v, or lo (any a: stays in range)
template <typename I>
__device__ __forceinline__ int last_not_above(const I* a, int lo, int hi, int64_t v) {
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if ((int64_t)a[mid] <= v) lo = mid;
        else hi = mid - 1;
    }
    return lo;
}

// The entries of one matrix: bit1 column out of range, bit2 non-finite value,
// bit32 column outside the diagonal block of its row's instance; and the two
// sums of k_transpose_dot, u_r a v_c and its absolute value, as partials[g]
// and partials[gridDim + g].  A workgroup takes kCheckChunk entries at a time,
// finds their rows' and instances' ranges and each entry's row among those:
// one pass over the entries, whatever the row lengths, where the row tiles
// took five and a plan made on the host from a copy of the row pointers.  A
// row pointer that is not one (checked beside this) makes no access leave it.
constexpr int kCheckChunk = 2048;
__global__ __launch_bounds__(kBlock) void k_check_blocks(const int32_t* rowptr, const int32_t* col, const double* val,
                                                         int64_t nnz, int32_t nrows, int32_t ncols,
                                                         const int32_t* row_off, const int32_t* col_off, int B,
                                                         uint32_t seed_row, uint32_t seed_col, int32_t* flags,
                                                         double* partials) {
    __shared__ int32_t rows[kCheckChunk + 1];
    __shared__ int range[4];
    const int tid = threadIdx.x;
    double s = 0.0, sa = 0.0;
    int f = 0;
    const int64_t chunks = (nnz + kCheckChunk - 1) / kCheckChunk;
    for (int64_t c = blockIdx.x; c < chunks; c += gridDim.x) {
        const int64_t k0 = c * kCheckChunk, k1 = min(k0 + kCheckChunk, nnz);
        __syncthreads();  // the last chunk's rows are read
        if (tid < 2) {
            const int r = last_not_above(rowptr, 0, nrows - 1, tid == 0 ? k0 : k1 - 1);
            range[tid] = r;
            range[2 + tid] = last_not_above(row_off, 0, B - 1, r);
        }
        __syncthreads();
        const int r0 = range[0], r1 = max(range[1], r0), i0 = range[2], i1 = max(range[3], i0);
        const bool in_lds = r1 - r0 <= kCheckChunk;
        if (in_lds)
            for (int r = r0 + tid; r <= r1; r += kBlock) rows[r - r0] = rowptr[r];
        __syncthreads();
        for (int64_t k = k0 + tid; k < k1; k += kBlock) {
            const int r = in_lds ? r0 + last_not_above(rows, 0, r1 - r0, k) : last_not_above(rowptr, r0, r1, k);
            const int inst = last_not_above(row_off, i0, i1, r);
            const int32_t j = col[k];
            const double a = val[k];
            if (j < 0 || j >= ncols) f |= 1;
            if (!isfinite(a)) f |= 2;
            if (j < col_off[inst] || j >= col_off[inst + 1]) f |= 32;
            const double u = hash_unit((uint32_t)r, seed_row), t = a * hash_unit((uint32_t)j, seed_col);
            s += u * t;
            sa += fabs(u) * fabs(t);
        }
    }
    if (f) atomicOr(flags, f);
    double q[2] = {s, sa}, mx[1] = {0.0};
    __shared__ double out[2];
    block_reduce_store<2, 0>(q, mx, out);
    __syncthreads();
    if (tid < 2) partials[(int64_t)tid * gridDim.x + blockIdx.x] = out[tid];
}

int check_blocks(const mipdhg_batch& bt, bool entries, const int32_t* row_off_dev, const int32_t* col_off_dev,
                 int64_t* nnz_off_dev, int32_t* flags, double* partials, hipStream_t stream) {
    const mipdhg_lp& lp = bt.whole;
    const int B = bt.count;
    MIP_HIP(hipMemcpyAsync(nnz_off_dev, bt.nnz_off, ((size_t)B + 1) * 8, hipMemcpyHostToDevice, stream));
    MIP_HIP(hipMemsetAsync(flags, 0, kCheckFlagBytes, stream));
    hipLaunchKernelGGL(k_check_rowptr, dim3(grid_for(lp.m)), dim3(kBlock), 0, stream, lp.a_rowptr, lp.m, lp.nnz,
                       row_off_dev, nnz_off_dev, B, flags);
    hipLaunchKernelGGL(k_check_rowptr, dim3(grid_for(lp.n)), dim3(kBlock), 0, stream, lp.at_rowptr, lp.n, lp.nnz,
                       col_off_dev, nnz_off_dev, B, flags);
    double* const red = (double*)(flags + 32);  // u^T (A v) and v^T (A^T u), each with its absolute terms' sum
    if (entries) {
        hipLaunchKernelGGL(k_check_vec, dim3(grid_for(lp.m)), dim3(kBlock), 0, stream, lp.b, (int64_t)lp.m, flags);
        hipLaunchKernelGGL(k_check_vec, dim3(grid_for(lp.n)), dim3(kBlock), 0, stream, lp.c, (int64_t)lp.n, flags);
        if (lp.nnz > 0) {
            const int G = (int)std::min<int64_t>((lp.nnz + kCheckChunk - 1) / kCheckChunk, kCheckGrid);
            const uint32_t su = 0x1234u, sv = 0xABCDu;
            hipLaunchKernelGGL(k_check_blocks, dim3(G), dim3(kBlock), 0, stream, lp.a_rowptr, lp.a_col, lp.a_val,
                               lp.nnz, lp.m, lp.n, row_off_dev, col_off_dev, B, su, sv, flags, partials);
            hipLaunchKernelGGL(k_check_blocks, dim3(G), dim3(kBlock), 0, stream, lp.at_rowptr, lp.at_col, lp.at_val,
                               lp.nnz, lp.n, lp.m, col_off_dev, row_off_dev, B, sv, su, flags, partials + 2 * G);
            for (int q = 0; q < 4; ++q)
                hipLaunchKernelGGL(k_sum_partials, dim3(1), dim3(kBlock), 0, stream, (const double*)(partials + q * G),
                                   G, red + q);
        }
    }
    MIP_LAUNCH_CHECK();
    struct {
        int32_t f[32];
        double red[4];
    } h;
    MIP_HIP(hipMemcpyAsync(&h, flags, sizeof(h), hipMemcpyDeviceToHost, stream));
    MIP_HIP(hipStreamSynchronize(stream));
    const int32_t f = h.f[0];
    if (f & (64 | 128)) {  // which row or instance, from the row pointers themselves
        std::vector<int32_t> rpa(lp.m + 1), rpat(lp.n + 1);
        MIP_HIP(hipMemcpyAsync(rpa.data(), lp.a_rowptr, (lp.m + 1) * 4, hipMemcpyDeviceToHost, stream));
        MIP_HIP(hipMemcpyAsync(rpat.data(), lp.at_rowptr, (lp.n + 1) * 4, hipMemcpyDeviceToHost, stream));
        MIP_HIP(hipStreamSynchronize(stream));
        int rc;
        if ((rc = check_rowptr(rpa, lp.m, lp.nnz, "A"))) return rc;
        if ((rc = check_rowptr(rpat, lp.n, lp.nnz, "A^T"))) return rc;
        for (int i = 0; i <= B; ++i)
            if (rpa[bt.row_off[i]] != bt.nnz_off[i] || rpat[bt.col_off[i]] != bt.nnz_off[i])
                return set_error("nnz_off does not match the row pointers at instance %d", i), MIPDHG_ERR_BAD_CSR;
        return set_error("the row pointers changed while they were checked"), MIPDHG_ERR_BAD_CSR;
    }
    if (!entries) return 0;
    if (f & 1) return set_error("column index out of range"), MIPDHG_ERR_BAD_CSR;
    if (f & 6) return set_error("NaN or Inf in A, A^T, b or c"), MIPDHG_ERR_NONFINITE;
    if (lp.nnz > 0) {
        const double scale = std::max(h.red[1], h.red[3]);
        if (!(fabs(h.red[0] - h.red[2]) <= 1e-10 * scale + 1e-300))
            return set_error("A^T does not match A (dot test %.17g vs %.17g)", h.red[0], h.red[2]),
                   MIPDHG_ERR_TRANSPOSE;
    }
    if (f & 32) return set_error("an entry lies outside its instance's diagonal block"), MIPDHG_ERR_BAD_CSR;
    return 0;
}

}  // namespace mip
