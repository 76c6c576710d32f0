// Directional transfer of spherical-harmonic radiance through the diffuse +
// Phong BRDF (Eq. final-radiosity with f_i = f^c_i x Ybar, Sec. 3.2,
// Eq. brdf, App. A), its adjoint and the BRDF coefficients.
//
// The coefficient vectors of surfel i live in its tangent frame
// (t_u, t_v, n).  Per stored entry (i, j) of F the directional factors use
// the unit direction d from p_i to p_j:
//   (T X)_i[l][a][c] = sum_j F_ij Y_a(d in i's frame) sum_b Y_b(-d in j's frame) X_j[l][b][c]
//   B^(k+1) = E + R (.) (T B^(k)),  R_i = pi o_i f^c_i  (per coefficient, colour)
// The adjoint T^T has the same form on F^T with the roles of the row and the
// column swapped, so one kernel serves both (the backward propagates with
// the decay term reversed).
//
// One wave owns one output row: its lanes take the row's entries (one each,
// 64 at a time), evaluate both SH bases of the pair and accumulate all K x 3
// outputs of the light; a butterfly over the wave then sums the lanes in a
// fixed order (deterministic results).  The senders' records and rows come
// through LDS: a lane that reads its own row 16 bytes at a time makes 64
// lanes touch 64 cache lines with each of 17 loads, and a CU's first-level
// cache takes one line a clock.  Loaded as they lie in memory, consecutive
// lanes consecutive 16 bytes, the same rows take a quarter of the accesses.
// A batch's rows are loaded while the one before is computed.  25 M entries,
// K = 16: a bounce 0.93 ms, now 0.49 ms; the gradient of F over eight bounces
// 9.1 ms, now 4.1 ms.  What bounds them now: 200 requests to L2 per 64
// entries, a fifth of which miss it (a bounce's rows are 9.6 MB, an XCD's L2
// 4 MB), beside 390 vector instructions.
#include <algorithm>

#include "gsrad_internal.h"
#include "sh_api.h"
#include "sh_basis.h"
#include "trace_api.h"

namespace gsrad {

namespace {

constexpr int kWavesPerBlock = 2;   // LDS of K = 16: five workgroups a CU
constexpr float kPi = 3.14159265358979324f;

__device__ __forceinline__ int64_t xcd_block(int64_t b, int64_t g) {
    const int64_t x = b & 7, q = b >> 3, per = g >> 3, rem = g & 7;
    return x * per + (x < rem ? x : rem) + q;
}

// Unit direction from the centre of `ri` to the centre of `rj` in ri's
// frame (di) and its opposite in rj's frame (ej).  Coincident centres take
// the receiver's normal as the direction.
__device__ __forceinline__ void pair_dirs(const Frame &ri, const Frame &rj, float (&di)[3], float (&ej)[3]) {
    float dx = rj.p[0] - ri.p[0], dy = rj.p[1] - ri.p[1], dz = rj.p[2] - ri.p[2];
    const float len2 = dx * dx + dy * dy + dz * dz;
    if (len2 > 0.0f) {
        const float inv = 1.0f / sqrtf(len2);
        dx *= inv;
        dy *= inv;
        dz *= inv;
    } else {
        dx = ri.n[0];
        dy = ri.n[1];
        dz = ri.n[2];
    }
    di[0] = dx * ri.u[0] + dy * ri.u[1] + dz * ri.u[2];
    di[1] = dx * ri.v[0] + dy * ri.v[1] + dz * ri.v[2];
    di[2] = dx * ri.n[0] + dy * ri.n[1] + dz * ri.n[2];
    ej[0] = -(dx * rj.u[0] + dy * rj.u[1] + dz * rj.u[2]);
    ej[1] = -(dx * rj.v[0] + dy * rj.v[1] + dz * rj.v[2]);
    ej[2] = -(dx * rj.n[0] + dy * rj.n[1] + dz * rj.n[2]);
}

// Sums v[0 .. N) over the wave's lanes, in the order of a butterfly from
// distance 32 down.  While N is even a lane keeps one half of the values and
// gives the other away; at the end a lane holds kept() values, from index
// first on, with the same lanes' values in each group of copies() lanes.
template <int N, int OFF = 32>
struct WaveSum {
    static constexpr bool kHalve = N % 2 == 0 && OFF >= 1;
    using Next = WaveSum<kHalve ? N / 2 : N, OFF / 2>;
    static __device__ __forceinline__ void run(float *v, int lane, int &first) {
        if constexpr (OFF >= 1) {
            if constexpr (kHalve) {
                const bool up = (lane & OFF) != 0;
#pragma unroll
                for (int q = 0; q < N / 2; ++q) {
                    const float give = up ? v[q] : v[q + N / 2];
                    const float keep = up ? v[q + N / 2] : v[q];
                    v[q] = keep + __shfl_xor(give, OFF, 64);
                }
                first += up ? N / 2 : 0;
            } else {
#pragma unroll
                for (int q = 0; q < N; ++q) v[q] += __shfl_xor(v[q], OFF, 64);
            }
            Next::run(v, lane, first);
        }
    }
    static constexpr int kept() {
        if constexpr (OFF >= 1) return Next::kept();
        else return N;
    }
    // lanes that end with the same values: those whose last halving bit is above
    static constexpr int copies() {
        if constexpr (OFF >= 1) return kHalve ? Next::copies() : 2 * Next::copies();
        else return 1;
    }
};

// Rows of 64 senders in LDS, `Bytes` each, loaded in pieces of 16 bytes (base
// and rows aligned to them) or of 12, which take 16 in LDS: piece s of the 64
// rows' pieces by lane s % 64.  Where a row is a multiple of four pieces, its
// pieces are exchanged by row, so that 16 lanes reading the same piece of
// their rows reach 16 different groups of four banks.
template <int Bytes, bool Aligned = true>
struct Staged {
    static constexpr int kPiece = Aligned && Bytes % 16 == 0 ? 16 : 12;
    static constexpr int kPieces = Bytes / kPiece;
    static constexpr int kSize = 64 * kPieces * 16;
    static constexpr int kFours = kPieces % 4 == 0 ? 4 : kPieces % 2 == 0 ? 2 : 1;
    static constexpr int kPeriod = kPieces / kFours;   // loads after which lanes take the same pieces, 16 rows on
    static __device__ __forceinline__ int exchange(int row) {
        return kPieces % 16 == 0 ? row & 15 : kPieces % 4 == 0 ? (row >> 2) & 3 : 0;
    }
    // row j of the lane at base + j * stride; lds is the same for the wave
    static __device__ __forceinline__ void load(char *lds, const void *base, int64_t stride, uint32_t j, int lane) {
        // all rows' indices first: a load's turn does not wait for its own
        uint32_t of[kPieces];
#pragma unroll
        for (int t = 0; t < kPieces; ++t)
            of[t] = (uint32_t)__shfl((int)j, (t % kPeriod * 64 + lane) / kPieces + t / kPeriod * (kPeriod * 64 / kPieces));
#pragma unroll
        for (int t = 0; t < kPieces; ++t) {
            const int s = t % kPeriod * 64 + lane, p = (s % kPieces) ^ exchange(s / kPieces);
            const char *src = static_cast<const char *>(base) + (int64_t)of[t] * stride + p * kPiece;
            const auto *from = (const __attribute__((address_space(1))) void *)src;
            auto *to = (__attribute__((address_space(3))) void *)(lds + t * 64 * 16);
            if constexpr (kPiece == 16) __builtin_amdgcn_global_load_lds(from, to, 16, 0, 0);
            else __builtin_amdgcn_global_load_lds(from, to, 12, 0, 0);
        }
    }
    static __device__ __forceinline__ void read(const char *lds, int lane, float *x) {
        constexpr int kF = kPiece / 4;
        const char *row = lds + lane * kPieces * 16;
        const int ex = exchange(lane);
#pragma unroll
        for (int p = 0; p < kPieces; ++p) {
            const float *v = reinterpret_cast<const float *>(row + ((p ^ ex) << 4));
#pragma unroll
            for (int c = 0; c < kF; ++c) x[kF * p + c] = v[c];
        }
    }
};

constexpr int kWaitVm0 = 0x0F70;   // s_waitcnt vmcnt(0), other counters unconstrained

constexpr int kWaitLgkm0 = 0xC07F;   // s_waitcnt lgkmcnt(0), other counters unconstrained

using Frames = Staged<(int)sizeof(Frame)>;

__device__ __forceinline__ Frame staged_frame(const char *lds, int lane) {
    float x[12];
    Frames::read(lds, lane, x);
    return Frame{{x[0], x[1], x[2]}, {x[3], x[4], x[5]}, {x[6], x[7], x[8]}, {x[9], x[10], x[11]}};
}

// mode 0 (bounce):  acc = (T X)_row;  out_a = acc (if set);  out_b = E + R (.) acc
// mode 1 (adjoint): acc = (T^T X)_row on F^T;  out_a = acc;  out_b += acc
template <int K, bool Aligned>
__global__ void __launch_bounds__(64 * kWavesPerBlock, 2) k_transfer_sh(const Frame *__restrict__ frames, const int64_t *__restrict__ row_ptr,
                                                                     const int32_t *__restrict__ col,
                                                                     const float *__restrict__ val, int64_t n, int Lt,
                                                                     const float *__restrict__ X,
                                                                     const float *__restrict__ E,
                                                                     const float *__restrict__ R,
                                                                     float *__restrict__ out_a,
                                                                     float *__restrict__ out_b, int mode,
                                                                     int64_t nblocks,
                                                                     const int32_t *__restrict__ order) {
    constexpr int W = 3 * K, N = W + W % 2;
    using Rows = Staged<4 * W, Aligned>;
    __shared__ __align__(16) char stage[kWavesPerBlock][Rows::kSize + (K > 1 ? Frames::kSize : 0)];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / 64);
    const int64_t idx = xcd_block(blockIdx.x, nblocks) * kWavesPerBlock + wave;
    if (idx >= n) return;
    const int64_t row = order ? (int64_t)order[idx] : idx;
    const int lane = __lane_id();
    char *rows = stage[wave], *recs = rows + Rows::kSize;
    const Frame ri = frames[row];
    const int64_t b = row_ptr[row], e = row_ptr[row + 1];
    for (int l = 0; l < Lt; ++l) {
        float acc[N];
#pragma unroll
        for (int q = 0; q < N; ++q) acc[q] = 0.0f;
        // a batch's rows are loaded while the one before is computed, its
        // entries one batch earlier still
        const char *base = reinterpret_cast<const char *>(X + (int64_t)l * W);
        const int64_t stride = (int64_t)Lt * W * 4;
        uint32_t j = 0;
        float w = 0.0f, w1 = 0.0f;
        if (b < e) {
            const int64_t k1 = min(b + lane, e - 1), k2 = min(b + 64 + lane, e - 1);
            const uint32_t j1 = (uint32_t)col[k1];
            w1 = val[k1];
            j = (uint32_t)col[k2];
            w = val[k2];
            if constexpr (K > 1) Frames::load(recs, frames, sizeof(Frame), j1, lane);
            Rows::load(rows, base, stride, j1, lane);
        }
        for (int64_t k0 = b; k0 < e; k0 += 64) {
            const bool live = k0 + lane < e;
            const float wc = w1;
            w1 = w;
            __builtin_amdgcn_s_waitcnt(kWaitVm0);
            Frame rj = ri;
            if constexpr (K > 1) rj = staged_frame(recs, lane);
            float x[W];
            Rows::read(rows, lane, x);
            __builtin_amdgcn_s_waitcnt(kWaitLgkm0);
            if (k0 + 64 < e) {
                if constexpr (K > 1) Frames::load(recs, frames, sizeof(Frame), j, lane);
                Rows::load(rows, base, stride, j, lane);
                const int64_t next = min(k0 + 128 + lane, e - 1);
                j = (uint32_t)col[next];
                w = val[next];
            }
            float di[3] = {}, ej[3] = {};
            if constexpr (K > 1) pair_dirs(ri, rj, di, ej);
            float Ye[K];
            sh_eval<K>(ej[0], ej[1], ej[2], Ye);
            float s0 = 0.0f, s1 = 0.0f, s2 = 0.0f;
#pragma unroll
            for (int q = 0; q < K; ++q) {
                s0 = __builtin_fmaf(Ye[q], x[3 * q + 0], s0);
                s1 = __builtin_fmaf(Ye[q], x[3 * q + 1], s1);
                s2 = __builtin_fmaf(Ye[q], x[3 * q + 2], s2);
            }
            if (live) {
                float Yd[K];
                sh_eval<K>(di[0], di[1], di[2], Yd);
                s0 *= wc;
                s1 *= wc;
                s2 *= wc;
#pragma unroll
                for (int a = 0; a < K; ++a) {
                    acc[3 * a + 0] = __builtin_fmaf(Yd[a], s0, acc[3 * a + 0]);
                    acc[3 * a + 1] = __builtin_fmaf(Yd[a], s1, acc[3 * a + 1]);
                    acc[3 * a + 2] = __builtin_fmaf(Yd[a], s2, acc[3 * a + 2]);
                }
            }
        }
        using Sum = WaveSum<N>;
        int first = 0;
        Sum::run(acc, lane, first);
        for (int q = lane % Sum::copies(); q < Sum::kept(); q += Sum::copies()) {
            float v = 0.0f;
#pragma unroll
            for (int z = 0; z < Sum::kept(); ++z) v = q == z ? acc[z] : v;
            if (first + q >= W) continue;
            const int64_t o = (row * Lt + l) * W + first + q;
            if (mode == 0) {
                if (out_a) out_a[o] = v;
                out_b[o] = __builtin_fmaf(R[row * W + first + q], v, E[o]);
            } else {
                out_a[o] = v;
                out_b[o] += v;
            }
        }
    }
}

// u = R (.) lambda, per light
__global__ void __launch_bounds__(256) k_scale_rows(const float *__restrict__ lam, const float *__restrict__ R,
                                                    int64_t n, int Lt, int W, float *__restrict__ u) {
    const int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (t >= n * Lt * W) return;
    const int64_t q = t % W, i = t / ((int64_t)Lt * W);
    u[t] = R[i * W + q] * lam[t];
}

// grad_F[e] = sum_k sum_l sum_c (Yd . (R (.) lambda^(k+1))_i[l][:, c]) (Ye . B^(k)_j[l][:, c])
// of bounces k0 .. k1 (added to the earlier ones' where k0 > 0)
template <int K>
__global__ void __launch_bounds__(64 * kWavesPerBlock, K == 9 ? 2 : 3) k_sddmm_sh(const Frame *__restrict__ frames, const int64_t *__restrict__ row_ptr,
                                                                  const int32_t *__restrict__ col, int64_t n, int Lt,
                                                                  int k0, int k1, const float *__restrict__ Btape,
                                                                  const float *__restrict__ Ltape,
                                                                  const float *__restrict__ R,
                                                                  float *__restrict__ grad_F, int64_t nblocks,
                                                                  const int32_t *__restrict__ order) {
    constexpr int W = 3 * K;
    using Rows = Staged<4 * W>;
    __shared__ __align__(16) char stage[kWavesPerBlock][Rows::kSize + (K > 1 ? Frames::kSize : 0)];
    __shared__ float own[kWavesPerBlock][W];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / 64);
    const int64_t idx = xcd_block(blockIdx.x, nblocks) * kWavesPerBlock + wave;
    if (idx >= n) return;
    const int64_t row = order ? (int64_t)order[idx] : idx;
    const int lane = __lane_id();
    char *rows = stage[wave], *recs = rows + Rows::kSize;
    float *u = own[wave];
    const Frame ri = frames[row];
    const int64_t b = row_ptr[row], e = row_ptr[row + 1];
    const size_t plane = (size_t)n * Lt * W;
    if (b >= e) return;
    const float r = lane < W ? R[row * W + lane] : 0.0f;
    // steps: a batch's bounces and lights; the rows of the next step are
    // loaded while one is computed, the entries one batch earlier still
    const int64_t stride = (int64_t)Lt * W * 4;
    auto rows_of = [&](int k, int l) { return reinterpret_cast<const char *>(Btape + k * plane + (int64_t)l * W); };
    auto own_of = [&](int k, int l) { return lane < W ? r * Ltape[k * plane + (row * Lt + l) * W + lane] : 0.0f; };
    uint32_t j = (uint32_t)col[min(b + lane, e - 1)];
    uint32_t jn = (uint32_t)col[min(b + 64 + lane, e - 1)];
    if constexpr (K > 1) Frames::load(recs, frames, sizeof(Frame), j, lane);   // (degree 0 is a constant)
    Rows::load(rows, rows_of(k0, 0), stride, j, lane);
    float un = own_of(k0, 0), g = 0.0f;
    float Yd[K], Ye[K];
    int64_t e0 = b;
    int k = k0, l = 0;
    for (;;) {
        const bool head = k == k0 && l == 0;
        __builtin_amdgcn_s_waitcnt(kWaitVm0);
        if (lane < W) u[lane] = un;
        Frame rj = ri;
        if (K > 1 && head) rj = staged_frame(recs, lane);
        float x[W];
        Rows::read(rows, lane, x);
        __builtin_amdgcn_s_waitcnt(kWaitLgkm0);
        int64_t en = e0;
        int kn = k, ln = l + 1;
        if (ln == Lt) {
            ln = 0;
            if (++kn == k1) {
                kn = k0;
                en += 64;
            }
        }
        if (en < e) {
            if (en != e0) {
                j = jn;
                jn = (uint32_t)col[min(en + 64 + lane, e - 1)];
                if constexpr (K > 1) Frames::load(recs, frames, sizeof(Frame), j, lane);
            }
            Rows::load(rows, rows_of(kn, ln), stride, j, lane);
            un = own_of(kn, ln);
        }
        const int64_t kk = e0 + lane;
        if (head) {
            float di[3] = {}, ej[3] = {};
            if constexpr (K > 1) pair_dirs(ri, rj, di, ej);
            sh_eval<K>(di[0], di[1], di[2], Yd);
            sh_eval<K>(ej[0], ej[1], ej[2], Ye);
            g = k0 > 0 && kk < e ? grad_F[kk] : 0.0f;
        }
        float p0 = 0.0f, p1 = 0.0f, p2 = 0.0f, s0 = 0.0f, s1 = 0.0f, s2 = 0.0f;
#pragma unroll
        for (int q = 0; q < K; ++q) {
            p0 = __builtin_fmaf(Yd[q], u[3 * q + 0], p0);
            p1 = __builtin_fmaf(Yd[q], u[3 * q + 1], p1);
            p2 = __builtin_fmaf(Yd[q], u[3 * q + 2], p2);
            s0 = __builtin_fmaf(Ye[q], x[3 * q + 0], s0);
            s1 = __builtin_fmaf(Ye[q], x[3 * q + 1], s1);
            s2 = __builtin_fmaf(Ye[q], x[3 * q + 2], s2);
        }
        g = __builtin_fmaf(p0, s0, g);
        g = __builtin_fmaf(p1, s1, g);
        g = __builtin_fmaf(p2, s2, g);
        if (en != e0 && kk < e) grad_F[kk] = g;
        __builtin_amdgcn_wave_barrier();
        if (en >= e) break;
        e0 = en;
        k = kn;
        l = ln;
    }
}

// The same with every lane reading its own sender's row: no step waits for the
// one before, which counts where the rows come from L2 and a step is short.
template <int K>
__global__ void __launch_bounds__(256) k_sddmm_sh_own(const Frame *__restrict__ frames, const int64_t *__restrict__ row_ptr,
                                                      const int32_t *__restrict__ col, int64_t n, int Lt, int nb,
                                                      const float *__restrict__ Btape, const float *__restrict__ Ltape,
                                                      const float *__restrict__ R, float *__restrict__ grad_F,
                                                      int64_t nblocks, const int32_t *__restrict__ order) {
    constexpr int W = 3 * K;
    const int64_t idx = xcd_block(blockIdx.x, nblocks) * 4 + threadIdx.x / 64;
    if (idx >= n) return;
    const int64_t row = order ? (int64_t)order[idx] : idx;
    const Frame ri = frames[row];
    const int64_t b = row_ptr[row], e = row_ptr[row + 1];
    const float *Ri = R + row * W;
    const size_t plane = (size_t)n * Lt * W;
    for (int64_t kk = b + __lane_id(); kk < e; kk += 64) {
        const int32_t j = col[kk];
        float di[3] = {}, ej[3] = {};
        if constexpr (K > 1) pair_dirs(ri, frames[j], di, ej);
        float Yd[K], Ye[K];
        sh_eval<K>(di[0], di[1], di[2], Yd);
        sh_eval<K>(ej[0], ej[1], ej[2], Ye);
        float g = 0.0f;
        for (int k = 0; k < nb; ++k) {
            for (int l = 0; l < Lt; ++l) {
                const float *lam = Ltape + k * plane + (row * Lt + l) * W;
                const float *bj = Btape + k * plane + ((int64_t)j * Lt + l) * W;
                float p0 = 0.0f, p1 = 0.0f, p2 = 0.0f, s0 = 0.0f, s1 = 0.0f, s2 = 0.0f;
#pragma unroll
                for (int q = 0; q < K; ++q) {
                    p0 = __builtin_fmaf(Yd[q], Ri[3 * q + 0] * lam[3 * q + 0], p0);
                    p1 = __builtin_fmaf(Yd[q], Ri[3 * q + 1] * lam[3 * q + 1], p1);
                    p2 = __builtin_fmaf(Yd[q], Ri[3 * q + 2] * lam[3 * q + 2], p2);
                    s0 = __builtin_fmaf(Ye[q], bj[3 * q + 0], s0);
                    s1 = __builtin_fmaf(Ye[q], bj[3 * q + 1], s1);
                    s2 = __builtin_fmaf(Ye[q], bj[3 * q + 2], s2);
                }
                g = __builtin_fmaf(p0, s0, g);
                g = __builtin_fmaf(p1, s1, g);
                g = __builtin_fmaf(p2, s2, g);
            }
        }
        grad_F[kk] = g;
    }
}

// grad_R[i][q] = sum_k sum_l lambda^(k+1)_i[l][q] Q^(k)_i[l][q]
__global__ void __launch_bounds__(256) k_grad_R(const float *__restrict__ Ltape, const float *__restrict__ Qtape,
                                                int64_t n, int Lt, int W, int nb, float *__restrict__ grad_R) {
    const int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (t >= n * W) return;
    const int64_t i = t / W, q = t % W;
    const size_t plane = (size_t)n * Lt * W;
    float g = 0.0f;
    for (int k = 0; k < nb; ++k)
        for (int l = 0; l < Lt; ++l) {
            const size_t o = k * plane + (i * Lt + l) * W + q;
            g = __builtin_fmaf(Ltape[o], Qtape[o], g);
        }
    grad_R[t] = g;
}

// App. A: g_l(s) for the Phong lobe and its derivative, l = 1..3
__device__ __forceinline__ float lobe(int l, float s) {
    if (l == 1) return (s + 1.0f) / (s + 2.0f);
    if (l == 2) return s / (s + 3.0f);
    return ((s + 1.0f) * (s - 1.0f)) / ((s + 2.0f) * (s + 4.0f));
}

__device__ __forceinline__ float lobe_ds(int l, float s) {
    if (l == 1) return 1.0f / ((s + 2.0f) * (s + 2.0f));
    if (l == 2) return 3.0f / ((s + 3.0f) * (s + 3.0f));
    const float D = (s + 2.0f) * (s + 4.0f);
    return (2.0f * s * D - (s * s - 1.0f) * (2.0f * s + 6.0f)) / (D * D);
}

__device__ __forceinline__ float brdf_coef(int a, int c, float k, const float *ad, const float *as, float s) {
    if (a == 0) return 4.0f * k * ad[c] + (1.0f - k) * as[c];
    const float sgn = (sh_m(a) & 1) ? -1.0f : 1.0f;
    return sgn * (1.0f - k) * lobe(sh_l(a), s) * as[c];
}

__global__ void __launch_bounds__(256) k_brdf_reflectance(BvhDev bv, const float *__restrict__ kd,
                                                          const float *__restrict__ ad, const float *__restrict__ as,
                                                          const float *__restrict__ shin, int K, float *__restrict__ R) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= bv.n) return;
    const float o = bv.op[i];
    for (int a = 0; a < K; ++a)
        for (int c = 0; c < 3; ++c)
            R[(i * K + a) * 3 + c] = kPi * o * brdf_coef(a, c, kd[i], ad + 3 * i, as + 3 * i, shin[i]);
}

__global__ void __launch_bounds__(256) k_brdf_backward(BvhDev bv, const float *__restrict__ kd,
                                                       const float *__restrict__ ad, const float *__restrict__ as,
                                                       const float *__restrict__ shin, int K,
                                                       const float *__restrict__ G, float *g_o, float *g_k,
                                                       float *g_ad, float *g_as, float *g_s) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= bv.n) return;
    const float o = bv.op[i], oraw = bv.raw_op[i];
    const bool inside = oraw > 0.0f && oraw < kOpacityMax;
    const float k = kd[i], s = shin[i];
    const float *adi = ad + 3 * i, *asi = as + 3 * i, *Gi = G + i * K * 3;
    float go = 0.0f, gk = 0.0f, gs = 0.0f, gad[3], gas[3];
    for (int c = 0; c < 3; ++c) {
        const float gp = kPi * o * Gi[c];
        gad[c] = gp * 4.0f * k;
        gas[c] = gp * (1.0f - k);
        gk += gp * (4.0f * adi[c] - asi[c]);
    }
    for (int a = 0; a < K; ++a) {
        const float sgn = (sh_m(a) & 1) ? -1.0f : 1.0f;
        const int l = sh_l(a);
        for (int c = 0; c < 3; ++c) {
            go += Gi[3 * a + c] * brdf_coef(a, c, k, adi, asi, s);
            if (a == 0) continue;
            const float gp = kPi * o * Gi[3 * a + c];
            gk -= gp * sgn * lobe(l, s) * asi[c];
            gas[c] += gp * sgn * (1.0f - k) * lobe(l, s);
            gs += gp * sgn * (1.0f - k) * lobe_ds(l, s) * asi[c];
        }
    }
    if (g_o) g_o[i] = inside ? kPi * go : 0.0f;
    if (g_k) g_k[i] = gk;
    if (g_s) g_s[i] = gs;
    for (int c = 0; c < 3; ++c) {
        if (g_ad) g_ad[3 * i + c] = gad[c];
        if (g_as) g_as[3 * i + c] = gas[c];
    }
}

unsigned row_blocks_sh(int64_t n) { return (unsigned)((n + kWavesPerBlock - 1) / kWavesPerBlock); }

template <int K>
void launch_transfer_k(const Frame *frames, const Csr &F, int Lt, const float *X, const float *E, const float *R,
                       float *out_a, float *out_b, int mode, hipStream_t st) {
    const unsigned g = row_blocks_sh(F.n);
    const auto kernel = reinterpret_cast<uintptr_t>(X) % 16 == 0 ? k_transfer_sh<K, true> : k_transfer_sh<K, false>;
    hipLaunchKernelGGL(kernel, dim3(g), dim3(64 * kWavesPerBlock), 0, st, frames, F.row_ptr, F.col, F.val, F.n, Lt, X, E, R,
                       out_a, out_b, mode, (int64_t)g, F.order);
}

// Bounces of one launch of k_sddmm_sh: as many as have senders' rows of
// kSddmmBytesSh together, which an XCD's L2 still serves for the most part; a
// launch more costs the pair's bases again and grad_F once more.  Eight
// bounces of 50k surfels, K = 16 (9.6 MB each): 4.1 ms by one bounce, 4.2 ms
// by two, 4.8 ms by eight.
constexpr int64_t kSddmmBytesSh = (int64_t)7 << 20;

int sddmm_bounces_sh(int64_t n, int Lt, int K) {
    return (int)std::max<int64_t>(1, kSddmmBytesSh / (n * Lt * K * 12));
}

// (a sender is then gathered too few times for L2 to matter)
bool short_rows(const Csr &F) { return F.nnz <= 40 * F.n; }

// Rows read by their own lanes instead of through LDS: K = 4 and 9 for short rows
// and few of them (512 rows, eight lights, K = 9, four bounces: 153 us, staged
// 203; 6,000 rows of 256 entries, one light: 102 and 71), K = 1, whose 12 bytes a
// row gain nothing from LDS, until the senders' rows leave L2 (6,000 rows of a
// room, one light: 74 us, staged 108; 50k rows, eight lights: 4.1 and 3.6 ms).
bool sddmm_own(const Csr &F, int K) {
    if (K == 16) return false;
    if (K == 1) return short_rows(F) || F.n <= 30000;
    return F.n <= 1024 || (short_rows(F) && (K == 9 || F.n <= 2048));
}

template <int K>
void launch_sddmm_k(const Frame *frames, const Csr &F, int Lt, int nb, const float *Bt, const float *Lt_, const float *R,
                    float *grad_F, hipStream_t st) {
    if (sddmm_own(F, K)) {
        const unsigned own = (unsigned)((F.n + 3) / 4);
        hipLaunchKernelGGL(k_sddmm_sh_own<K>, dim3(own), dim3(256), 0, st, frames, F.row_ptr, F.col, F.n, Lt, nb, Bt, Lt_,
                           R, grad_F, (int64_t)own, F.order);
        return;
    }
    const unsigned g = row_blocks_sh(F.n);
    const int per = short_rows(F) ? nb : sddmm_bounces_sh(F.n, Lt, K);
    for (int k = 0; k < nb; k += per)
        hipLaunchKernelGGL(k_sddmm_sh<K>, dim3(g), dim3(64 * kWavesPerBlock), 0, st, frames, F.row_ptr, F.col, F.n, Lt, k,
                           std::min(nb, k + per), Bt, Lt_, R, grad_F, (int64_t)g, F.order);
}

}  // namespace

gsrad_status launch_transfer_sh(const Frame *fr, const Csr &F, int Lt, int K, const float *X, const float *E,
                                const float *R, float *out_a, float *out_b, int mode, hipStream_t st) {
    if (F.n == 0) return GSRAD_OK;
    switch (K) {
        case 1: launch_transfer_k<1>(fr, F, Lt, X, E, R, out_a, out_b, mode, st); break;
        case 4: launch_transfer_k<4>(fr, F, Lt, X, E, R, out_a, out_b, mode, st); break;
        case 9: launch_transfer_k<9>(fr, F, Lt, X, E, R, out_a, out_b, mode, st); break;
        case 16: launch_transfer_k<16>(fr, F, Lt, X, E, R, out_a, out_b, mode, st); break;
        default: set_error("SH transfer: K must be 1, 4, 9 or 16"); return GSRAD_EINVAL;
    }
    return check_hip(hipGetLastError(), "SH transfer launch");
}

gsrad_status launch_scale_rows(const float *lam, const float *R, int64_t n, int Lt, int K, float *u, hipStream_t st) {
    const int64_t total = n * Lt * K * 3;
    if (total == 0) return GSRAD_OK;
    hipLaunchKernelGGL(k_scale_rows, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, st, lam, R, n, Lt, K * 3, u);
    return check_hip(hipGetLastError(), "SH scale launch");
}

gsrad_status launch_sddmm_sh(const Frame *fr, const Csr &F, int Lt, int K, int nb, const float *Btape,
                             const float *Ltape, const float *R, float *grad_F, hipStream_t st) {
    if (F.n == 0 || F.nnz == 0) return GSRAD_OK;
    switch (K) {
        case 1: launch_sddmm_k<1>(fr, F, Lt, nb, Btape, Ltape, R, grad_F, st); break;
        case 4: launch_sddmm_k<4>(fr, F, Lt, nb, Btape, Ltape, R, grad_F, st); break;
        case 9: launch_sddmm_k<9>(fr, F, Lt, nb, Btape, Ltape, R, grad_F, st); break;
        case 16: launch_sddmm_k<16>(fr, F, Lt, nb, Btape, Ltape, R, grad_F, st); break;
        default: set_error("SH sddmm: K must be 1, 4, 9 or 16"); return GSRAD_EINVAL;
    }
    return check_hip(hipGetLastError(), "SH sddmm launch");
}

gsrad_status launch_grad_R(const float *Ltape, const float *Qtape, int64_t n, int Lt, int K, int nb, float *grad_R,
                           hipStream_t st) {
    const int64_t total = n * K * 3;
    hipLaunchKernelGGL(k_grad_R, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, st, Ltape, Qtape, n, Lt, K * 3,
                       nb, grad_R);
    return check_hip(hipGetLastError(), "SH grad_R launch");
}

gsrad_status launch_brdf_reflectance(const BvhDev &bv, const float *kd, const float *ad, const float *as,
                                     const float *shin, int K, float *R, hipStream_t st) {
    hipLaunchKernelGGL(k_brdf_reflectance, dim3((unsigned)((bv.n + 255) / 256)), dim3(256), 0, st, bv, kd, ad, as, shin,
                       K, R);
    return check_hip(hipGetLastError(), "BRDF reflectance launch");
}

gsrad_status launch_brdf_backward(const BvhDev &bv, const float *kd, const float *ad, const float *as,
                                  const float *shin, int K, const float *G, float *g_o, float *g_k, float *g_ad,
                                  float *g_as, float *g_s, hipStream_t st) {
    hipLaunchKernelGGL(k_brdf_backward, dim3((unsigned)((bv.n + 255) / 256)), dim3(256), 0, st, bv, kd, ad, as, shin, K,
                       G, g_o, g_k, g_ad, g_as, g_s);
    return check_hip(hipGetLastError(), "BRDF backward launch");
}

}  // namespace gsrad
