// CSR transpose (stable, deterministic) and FP64 checks of the transport.
#include "gsrad_internal.h"
#include "trace_api.h"

namespace gsrad {

namespace {

constexpr int kWavesPerBlock = 4;

__global__ void __launch_bounds__(256) k_expand_rows(const int64_t *__restrict__ row_ptr, int64_t n,
                                                     uint32_t *__restrict__ rows, uint32_t *__restrict__ keys_col,
                                                     const int32_t *__restrict__ col, uint32_t *__restrict__ ids) {
    const int64_t row = (int64_t)blockIdx.x * kWavesPerBlock + threadIdx.x / 64;
    if (row >= n) return;
    const int64_t b = row_ptr[row], e = row_ptr[row + 1];
    for (int64_t k = b + __lane_id(); k < e; k += 64) {
        rows[k] = (uint32_t)row;
        keys_col[k] = (uint32_t)col[k];
        ids[k] = (uint32_t)k;
    }
}

// Row pointers of the transpose from the column-sorted keys: position p of
// the sorted list starts every column c with keys[p-1] < c <= keys[p]
// (keys[-1] = -1, keys[nnz] = n), so each of the n + 1 pointers is written
// exactly once.
__global__ void __launch_bounds__(256) k_col_bounds(const uint32_t *__restrict__ keys, int64_t nnz, int64_t n,
                                                    int64_t *__restrict__ t_row_ptr) {
    const int64_t p = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (p > nnz) return;
    const int64_t a = p == 0 ? -1 : (int64_t)keys[p - 1];
    const int64_t b = p == nnz ? n : (int64_t)keys[p];
    for (int64_t c = a + 1; c <= b; ++c) t_row_ptr[c] = p;
}

__global__ void __launch_bounds__(256) k_transpose_gather(const uint32_t *__restrict__ sorted_ids,
                                                          const uint32_t *__restrict__ rows,
                                                          const float *__restrict__ val, int64_t nnz,
                                                          int32_t *__restrict__ t_col, float *__restrict__ t_val) {
    const int64_t k = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (k >= nnz) return;
    const uint32_t e = sorted_ids[k];
    t_col[k] = (int32_t)rows[e];
    t_val[k] = val[e];
}

// FP64 residual of the fixed point and the other checks.
__global__ void __launch_bounds__(256) k_check(const int64_t *__restrict__ row_ptr, const int32_t *__restrict__ col,
                                               const float *__restrict__ val, int64_t n, int C,
                                               const float *__restrict__ rho, const float *__restrict__ E,
                                               const float *__restrict__ B, double *acc) {
    const int64_t row = (int64_t)blockIdx.x * kWavesPerBlock + threadIdx.x / 64;
    if (row >= n) return;
    const int lane = __lane_id();
    const int64_t b = row_ptr[row], e = row_ptr[row + 1];
    double r2 = 0.0, b2 = 0.0, bad = 0.0, rs = 0.0;
    for (int c = lane; c < C; c += 64) {
        double s = 0.0;
        for (int64_t k = b; k < e; ++k) s += (double)val[k] * (double)B[(int64_t)col[k] * C + c];
        const double Bi = B[row * C + c], Ei = E[row * C + c], ri = rho[row * 3 + c % 3];
        if (!isfinite(Bi) || !isfinite(Ei) || !isfinite(ri)) bad += 1.0;
        const double r = Ei + ri * s - Bi;
        r2 += r * r;
        b2 += Bi * Bi;
    }
    for (int64_t k = b + lane; k < e; k += 64) rs += (double)val[k];
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) {
        r2 += __shfl_xor(r2, o, 64);
        b2 += __shfl_xor(b2, o, 64);
        bad += __shfl_xor(bad, o, 64);
        rs += __shfl_xor(rs, o, 64);
    }
    if (lane == 0) {
        unsafeAtomicAdd(&acc[0], r2);
        unsafeAtomicAdd(&acc[1], b2);
        unsafeAtomicAdd(&acc[3], bad);
        // max of non-negative doubles through their bit patterns
        atomicMax(reinterpret_cast<unsigned long long *>(&acc[2]), (unsigned long long)__double_as_longlong(rs));
    }
}

// Reciprocity of the estimated operator (A_i F_ij = A_j F_ji for the exact
// form factors, App. E areas): per stored entry the FP64 difference with
// its mirror entry F_ji (binary search in row j; 0 if not stored).
// acc[0] += |A_i F_ij - A_j F_ji|, acc[1] += A_i F_ij,
// acc[2] = max |A_i F_ij - A_j F_ji| / max(A_i F_ij, A_j F_ji) (bit order).
__global__ void __launch_bounds__(256) k_reciprocity(const int64_t *__restrict__ row_ptr,
                                                     const int32_t *__restrict__ col, const float *__restrict__ val,
                                                     int64_t n, const double *__restrict__ area, double *acc) {
    const int64_t row = (int64_t)blockIdx.x * kWavesPerBlock + threadIdx.x / 64;
    if (row >= n) return;
    const int lane = __lane_id();
    double sd = 0.0, sf = 0.0, mx = 0.0;
    const double ai = area[row];
    for (int64_t k = row_ptr[row] + lane; k < row_ptr[row + 1]; k += 64) {
        const int64_t j = col[k];
        int64_t lo = row_ptr[j], hi = row_ptr[j + 1];
        while (lo < hi) {
            const int64_t mid = (lo + hi) >> 1;
            if (col[mid] < row) lo = mid + 1;
            else hi = mid;
        }
        const double fji = (lo < row_ptr[j + 1] && col[lo] == row) ? (double)val[lo] : 0.0;
        const double a = ai * (double)val[k], b = area[j] * fji;
        const double d = fabs(a - b);
        sd += d;
        sf += a;
        const double m = fmax(a, b);
        if (m > 0.0) mx = fmax(mx, d / m);
    }
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) {
        sd += __shfl_xor(sd, o, 64);
        sf += __shfl_xor(sf, o, 64);
        mx = fmax(mx, __shfl_xor(mx, o, 64));
    }
    if (lane == 0) {
        unsafeAtomicAdd(&acc[0], sd);
        unsafeAtomicAdd(&acc[1], sf);
        atomicMax(reinterpret_cast<unsigned long long *>(&acc[2]), (unsigned long long)__double_as_longlong(mx));
    }
}

inline unsigned row_blocks(int64_t n) { return (unsigned)((n + kWavesPerBlock - 1) / kWavesPerBlock); }

}  // namespace

size_t transpose_temp_bytes(int64_t n, int64_t nnz) {
    size_t b = 0;
    b += 4 * ((size_t)nnz * 4 + 256);       // rows, keys, ids, sorted keys
    b += (size_t)nnz * 4 + 256;             // sorted ids
    b += radix_temp_bytes(nnz) + 256;
    return b;
}

static inline char *carve(char *&p, size_t bytes) {
    char *r = p;
    p += (bytes + 255) / 256 * 256;
    return r;
}

gsrad_status csr_transpose(const Csr &A, int64_t *t_row_ptr, int32_t *t_col, float *t_val, void *temp,
                           size_t temp_bytes, hipStream_t st) {
    const int64_t n = A.n, nnz = A.nnz;
    char *p = static_cast<char *>(temp);
    uint32_t *rows = reinterpret_cast<uint32_t *>(carve(p, (size_t)nnz * 4));
    uint32_t *keys = reinterpret_cast<uint32_t *>(carve(p, (size_t)nnz * 4));
    uint32_t *ids = reinterpret_cast<uint32_t *>(carve(p, (size_t)nnz * 4));
    uint32_t *skeys = reinterpret_cast<uint32_t *>(carve(p, (size_t)nnz * 4));
    uint32_t *sids = reinterpret_cast<uint32_t *>(carve(p, (size_t)nnz * 4));
    const size_t rbytes = radix_temp_bytes(nnz);
    void *rtemp = carve(p, rbytes);
    if ((size_t)(p - static_cast<char *>(temp)) > temp_bytes) {
        set_error("transpose: temp too small");
        return GSRAD_EINVAL;
    }
    gsrad_status s;
    if (nnz > 0) {
        hipLaunchKernelGGL(k_expand_rows, dim3(row_blocks(n)), dim3(256), 0, st, A.row_ptr, n, rows, keys, A.col, ids);
        int bits = 1;
        while (bits < 32 && ((int64_t)1 << bits) < n) ++bits;
        s = radix_sort_pairs(keys, ids, skeys, sids, nnz, bits, rtemp, rbytes, st);
        if (s != GSRAD_OK) return s;
        hipLaunchKernelGGL(k_transpose_gather, dim3((unsigned)((nnz + 255) / 256)), dim3(256), 0, st, sids, rows,
                           A.val, nnz, t_col, t_val);
    }
    hipLaunchKernelGGL(k_col_bounds, dim3((unsigned)((nnz + 1 + 255) / 256)), dim3(256), 0, st, skeys, nnz, n,
                       t_row_ptr);
    return check_hip(hipGetLastError(), "transpose");
}

gsrad_status launch_reciprocity(const Csr &F, const double *area, double *acc, hipStream_t st) {
    if (F.n == 0) return GSRAD_OK;
    hipLaunchKernelGGL(k_reciprocity, dim3(row_blocks(F.n)), dim3(256), 0, st, F.row_ptr, F.col, F.val, F.n, area, acc);
    return check_hip(hipGetLastError(), "reciprocity launch");
}

gsrad_status launch_check(const Csr &F, int C, const float *rho, const float *E, const float *B, double *acc,
                          hipStream_t st) {
    hipLaunchKernelGGL(k_check, dim3(row_blocks(F.n)), dim3(256), 0, st, F.row_ptr, F.col, F.val, F.n, C, rho, E, B,
                       acc);
    return check_hip(hipGetLastError(), "check launch");
}

}  // namespace gsrad
