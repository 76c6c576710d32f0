// Batched transport over scenes of uneven size: the scenes' form factors
// form one block-diagonal F (global row and column indices), scene s owns
// rows [row_off[s], row_off[s+1]) and C_s = Lt_s * K * 3 columns, so B, E
// and the gradients are ragged: scene s's rows are a [N_s][C_s] block at
// val_off[s] of one array.
//
// With BF16 rows each bounce (and each adjoint step) is ONE persistent launch
// over all scenes: groups of LPR lanes take rows from a work queue (eight ranges,
// one per XCD, drained by the others once their own is done), so scenes of
// 2k and 65k surfels and 8 or 100 lights share the chip without tail
// effects.  The queue holds each ray-cast scene's rows in the receivers'
// Morton order, scene after scene (rows that one XCD takes together gather
// from nearby columns), else all rows by cost (entries x columns, largest
// first).
// LPR (lanes per row: 64, 32 or 16) is the tile shape the autotuner picks;
// every variant accumulates each output in the same order (the row's
// entries in CSR order), so the choice never changes a result bit.
#include "gsrad_internal.h"
#include "batch_api.h"

namespace gsrad {

namespace {

// Work-queue position -> row, for a group of LPR lanes: one lane takes the
// next index and the group shares it.  The queue is cut into eight equal
// ranges with a counter each; a group takes from the range of the XCD it
// runs on first (consecutive rows of the order, nearby receivers of one
// scene, share that XCD's L2) and from the others once it is drained.
// Every position below `rows` is handed out exactly once; `rows` means done.
template <int LPR>
__device__ __forceinline__ int64_t next_row(uint32_t *counter, int64_t rows, int lane_in_group, int group_base) {
    int q = (int)rows;
    if (lane_in_group == 0) {
        const int xcc = __builtin_amdgcn_s_getreg((3 << 11) | (0 << 6) | 20) & 7;   // HW_REG_XCC_ID
        for (int t = 0; t < 8; ++t) {
            const int x = (xcc + t) & 7;
            const int64_t lo = rows * x / 8, len = rows * (x + 1) / 8 - lo;
            const uint32_t idx = atomicAdd(counter + x, 1u);
            if ((int64_t)idx < len) {
                q = (int)(lo + idx);
                break;
            }
        }
    }
    return (int64_t)__shfl(q, group_base, 64);
}

// out = E + rho * (F in) on the rows of all scenes (bounce), or
// out = F^T (rho in) and gE += out (adjoint, FT given as F, rho applied to
// the gathered rows).  The gathered rows `in` are BF16, the sums FP32; one
// column chunk of LPR per pass over a row's entries (64 uneven rooms with
// 8-100 lights: bounces 3.0 s with one chunk, 3.3 s with two, 4.8 s with
// four).  FP32 rows: rows.hip.
template <int LPR, bool ADJ>
__global__ void __launch_bounds__(256) k_ragged_spmm(BatchDev bd, const int64_t *__restrict__ row_ptr,
                                                     const int32_t *__restrict__ col, const float *__restrict__ val,
                                                     const __bf16 *__restrict__ in, const float *__restrict__ E,
                                                     const float *__restrict__ rho, float *__restrict__ out,
                                                     float *__restrict__ gE, uint32_t *counter) {
    const int lane = __lane_id();
    const int lig = lane % LPR;                 // lane in group
    const int gbase = lane - lig;               // first lane of the group
    for (;;) {
        const int64_t q = next_row<LPR>(counter, bd.rows, lig, gbase);
        if (q >= bd.rows) break;
        const int64_t row = bd.order[q];
        const int s = bd.row_scene[row];
        const int C = bd.scene_C[s];
        const int64_t r0 = bd.row_off[s], base = bd.val_off[s];
        const int64_t lr = row - r0;
        const int64_t b = row_ptr[row], e = row_ptr[row + 1];
        for (int c0 = 0; c0 < C; c0 += LPR) {
            const int c = c0 + lig;
            const bool on = c < C;
            const int cc = on ? c : 0;   // lanes past C gather column 0 and discard it
            const int colour = cc % 3;
            float acc = 0.0f;
            for (int64_t k0 = b; k0 < e; k0 += LPR) {
                const int64_t kk = k0 + lig;
                const int jv = kk < e ? col[kk] : (int)r0;
                const float vv = kk < e ? val[kk] : 0.0f;
                const int m = (int)min<int64_t>(LPR, e - k0);
                int t = 0;
                // eight entries' gathers in flight, added in CSR order
                for (; t + 8 <= m; t += 8) {
                    float w[8], x[8];
#pragma unroll
                    for (int u = 0; u < 8; ++u) {
                        const int64_t j = __shfl(jv, gbase + t + u, 64);
                        w[u] = __shfl(vv, gbase + t + u, 64);
                        if (ADJ) w[u] *= rho[j * 3 + colour];
                        x[u] = (float)in[base + (j - r0) * C + cc];
                    }
#pragma unroll
                    for (int u = 0; u < 8; ++u) acc = __builtin_fmaf(w[u], x[u], acc);
                }
                for (; t < m; ++t) {
                    const int64_t j = __shfl(jv, gbase + t, 64);
                    float w = __shfl(vv, gbase + t, 64);
                    if (ADJ) w *= rho[j * 3 + colour];
                    acc = __builtin_fmaf(w, (float)in[base + (j - r0) * C + cc], acc);
                }
            }
            if (on) {
                const int64_t o = base + lr * C + c;
                if (ADJ) {
                    out[o] = acc;
                    gE[o] += acc;
                } else {
                    out[o] = __builtin_fmaf(rho[row * 3 + colour], acc, E[o]);
                }
            }
        }
    }
}

__global__ void k_reset_counter(uint32_t *counter) {
    if (threadIdx.x < 8) counter[threadIdx.x] = 0u;
}

// row -> scene and the per-row cost (entries x columns) used for ordering
__global__ void __launch_bounds__(256) k_row_cost(BatchDev bd, const int64_t *__restrict__ row_ptr,
                                                  uint32_t *__restrict__ keys, uint32_t *__restrict__ ids) {
    const int64_t r = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (r >= bd.rows) return;
    int lo = 0, hi = bd.scenes - 1;
    while (lo < hi) {   // last scene with row_off <= r
        const int mid = (lo + hi + 1) >> 1;
        if (bd.row_off[mid] <= r) lo = mid;
        else hi = mid - 1;
    }
    bd.row_scene[r] = lo;
    const uint64_t cost = (uint64_t)(row_ptr[r + 1] - row_ptr[r] + 1) * (uint64_t)bd.scene_C[lo];
    // descending cost: sort ascending on the complement, saturated to 32 bits
    keys[r] = ~(uint32_t)min<uint64_t>(cost, 0xffffffffull);
    ids[r] = (uint32_t)r;
}

__global__ void __launch_bounds__(256) k_copy_u32_to_i64(const uint32_t *__restrict__ a, int64_t n,
                                                         int64_t *__restrict__ b) {
    const int64_t r = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (r < n) b[r] = a[r];
}

inline unsigned persistent_blocks() { return 256 * 8; }   // 8 workgroups of 4 waves per CU

}  // namespace

gsrad_status batch_order_rows(const BatchDev &bd, const int64_t *row_ptr, void *temp, size_t temp_bytes,
                              hipStream_t st) {
    const int64_t n = bd.rows;
    if (n == 0) return GSRAD_OK;
    char *p = static_cast<char *>(temp);
    auto carve = [&](size_t bytes) {
        char *r = p;
        p += (bytes + 255) / 256 * 256;
        return r;
    };
    uint32_t *keys = reinterpret_cast<uint32_t *>(carve((size_t)n * 4));
    uint32_t *ids = reinterpret_cast<uint32_t *>(carve((size_t)n * 4));
    uint32_t *skeys = reinterpret_cast<uint32_t *>(carve((size_t)n * 4));
    uint32_t *sids = reinterpret_cast<uint32_t *>(carve((size_t)n * 4));
    const size_t rbytes = radix_temp_bytes(n);
    void *rtemp = carve(rbytes);
    if ((size_t)(p - static_cast<char *>(temp)) > temp_bytes) {
        set_error("batch ordering: temp too small");
        return GSRAD_EINVAL;
    }
    const unsigned g = (unsigned)((n + 255) / 256);
    hipLaunchKernelGGL(k_row_cost, dim3(g), dim3(256), 0, st, bd, row_ptr, keys, ids);
    gsrad_status s = radix_sort_pairs(keys, ids, skeys, sids, n, 32, rtemp, rbytes, st);
    if (s != GSRAD_OK) return s;
    hipLaunchKernelGGL(k_copy_u32_to_i64, dim3(g), dim3(256), 0, st, sids, n, const_cast<int64_t *>(bd.order));
    return check_hip(hipGetLastError(), "batch ordering");
}

size_t batch_order_temp_bytes(int64_t n) { return 4 * ((size_t)n * 4 + 256) + radix_temp_bytes(n) + 256; }

gsrad_status launch_ragged_spmm(const BatchDev &bd, const Csr &F, int lpr, bool adjoint, const void *in,
                                const float *E, const float *rho, float *out, float *gE, uint32_t *counter,
                                hipStream_t st) {
    hipLaunchKernelGGL(k_reset_counter, dim3(1), dim3(64), 0, st, counter);
    const dim3 grid(persistent_blocks()), block(256);
    auto run = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, grid, block, 0, st, bd, F.row_ptr, F.col, F.val, static_cast<const __bf16 *>(in), E,
                           rho, out, gE, counter);
    };
    if (lpr == 64) {
        if (adjoint) run(k_ragged_spmm<64, true>);
        else run(k_ragged_spmm<64, false>);
    } else if (lpr == 32) {
        if (adjoint) run(k_ragged_spmm<32, true>);
        else run(k_ragged_spmm<32, false>);
    } else if (lpr == 16) {
        if (adjoint) run(k_ragged_spmm<16, true>);
        else run(k_ragged_spmm<16, false>);
    } else {
        set_error("ragged product: lanes per row must be 16, 32 or 64");
        return GSRAD_EINVAL;
    }
    return check_hip(hipGetLastError(), "ragged product launch");
}

}  // namespace gsrad

namespace gsrad {

namespace {

__global__ void __launch_bounds__(256) k_offset_copy_i32(const int32_t *__restrict__ in, int64_t n, int32_t add,
                                                         int32_t *__restrict__ out) {
    for (int64_t k = (int64_t)blockIdx.x * 256 + threadIdx.x; k < n; k += (int64_t)gridDim.x * 256)
        out[k] = in[k] + add;
}

__global__ void __launch_bounds__(256) k_offset_copy_i64(const int64_t *__restrict__ in, int64_t n, int64_t add,
                                                         int64_t *__restrict__ out) {
    for (int64_t k = (int64_t)blockIdx.x * 256 + threadIdx.x; k < n; k += (int64_t)gridDim.x * 256)
        out[k] = in[k] + add;
}

__global__ void __launch_bounds__(256) k_offset_widen(const int32_t *__restrict__ in, int64_t n, int64_t add,
                                                      int64_t *__restrict__ out) {
    for (int64_t k = (int64_t)blockIdx.x * 256 + threadIdx.x; k < n; k += (int64_t)gridDim.x * 256)
        out[k] = (int64_t)in[k] + add;
}

__global__ void __launch_bounds__(256) k_copy_f32(const float *__restrict__ in, int64_t n, float *__restrict__ out) {
    for (int64_t k = (int64_t)blockIdx.x * 256 + threadIdx.x; k < n; k += (int64_t)gridDim.x * 256) out[k] = in[k];
}

inline unsigned grid_for(int64_t n) { return (unsigned)std::max<int64_t>(1, std::min<int64_t>((n + 255) / 256, 8192)); }

}  // namespace

gsrad_status launch_offset_copy_i32(const int32_t *in, int64_t n, int32_t add, int32_t *out, hipStream_t st) {
    if (n <= 0) return GSRAD_OK;
    hipLaunchKernelGGL(k_offset_copy_i32, dim3(grid_for(n)), dim3(256), 0, st, in, n, add, out);
    return check_hip(hipGetLastError(), "offset copy launch");
}

gsrad_status launch_offset_widen(const int32_t *in, int64_t n, int64_t add, int64_t *out, hipStream_t st) {
    if (n <= 0) return GSRAD_OK;
    hipLaunchKernelGGL(k_offset_widen, dim3(grid_for(n)), dim3(256), 0, st, in, n, add, out);
    return check_hip(hipGetLastError(), "offset widen launch");
}

gsrad_status launch_offset_copy_i64(const int64_t *in, int64_t n, int64_t add, int64_t *out, hipStream_t st) {
    if (n <= 0) return GSRAD_OK;
    hipLaunchKernelGGL(k_offset_copy_i64, dim3(grid_for(n)), dim3(256), 0, st, in, n, add, out);
    return check_hip(hipGetLastError(), "offset copy launch");
}

__global__ void __launch_bounds__(256) k_round_bf16(const float *__restrict__ in, int64_t n, __bf16 *__restrict__ out) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i < n) out[i] = (__bf16)in[i];   // round to nearest even
}

gsrad_status launch_round_bf16(const float *in, int64_t n, void *out, hipStream_t st) {
    if (n <= 0) return GSRAD_OK;
    hipLaunchKernelGGL(k_round_bf16, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, in, n,
                       static_cast<__bf16 *>(out));
    return check_hip(hipGetLastError(), "bf16 rounding launch");
}

gsrad_status launch_copy_f32(const float *in, int64_t n, float *out, hipStream_t st) {
    if (n <= 0) return GSRAD_OK;
    hipLaunchKernelGGL(k_copy_f32, dim3(grid_for(n)), dim3(256), 0, st, in, n, out);
    return check_hip(hipGetLastError(), "copy launch");
}

}  // namespace gsrad
