// Monte-Carlo TD(0) radiosity solver (Sec. 7, App. D): K-Means groups of
// the surfels, next-event sampling of a group and a member, the one-point
// estimate with the centre-to-centre decay and the running averages.
#include "gsrad_internal.h"
#include "sh_api.h"
#include "trace_api.h"
#include "traverse.h"

namespace gsrad {

namespace {

// ---------------------------------------------------------------------------
// Monte-Carlo TD(0) solver (Sec. 7, Alg. Monte-Carlo Solver, App. D)
// ---------------------------------------------------------------------------
// K-Means groups of the surfels (positions; the group keeps its mean
// centre, mean normal and the summed luminance of its members' current
// radiance as the proxy), then per step one next event per selected
// receiver a: a group g drawn with probability proportional to
//   w_g = L_g (|n_a . w_g| + beta)(|nbar_g . w_g| + beta) / max(r_g^2, r_min^2)
// and a member j != a of g proportional to the importance of Eq.
// importance-sampling, w_j = lum(B_j) |n_a . v||n_j . v| / |v|^4 (v = p_j - p_a);
// the one-point estimate (Eq. one-point-estimator) with the centre-to-centre
// decay of Sec. 8,
//   delta_a = E_a + rho_a F_aj B_j / Pr[j],  F_aj = lambda_j A_j T_aj |a||b| / (pi |v|^4),
// then the TD(0) averages (Eq. update): S += delta, S2 += delta^2, D += 1.
// Draws: Philox4x64-10 with counter (slot, step, 0, 2) (next event) and
// (slot, step, 1, 1) (receiver selection), key (seed, 0).
constexpr float kMcBeta = 0.05f;

__device__ __forceinline__ float lum3(const float *b) {
    return fmaxf(0.0f, 0.2126f * b[0] + 0.7152f * b[1] + 0.0722f * b[2]);
}

__device__ __forceinline__ float u01(uint64_t w) { return (float)(uint32_t)(w >> 40) * 0x1p-24f; }

__global__ void __launch_bounds__(256) k_km_init(BvhDev bv, int G, float *__restrict__ cent) {
    const int g = blockIdx.x * 256 + threadIdx.x;
    if (g >= G) return;
    const int64_t sidx = (int64_t)(((double)g + 0.5) * (double)bv.n / (double)G);
    const SurfRec r = bv.rec[min<int64_t>(sidx, bv.n - 1)];
    cent[3 * g + 0] = r.a.x;
    cent[3 * g + 1] = r.a.y;
    cent[3 * g + 2] = r.a.z;
}

__global__ void __launch_bounds__(256) k_km_assign(BvhDev bv, int G, const float *__restrict__ cent,
                                                   uint32_t *__restrict__ key, uint32_t *__restrict__ ids,
                                                   uint32_t *__restrict__ count) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= bv.n) return;
    const SurfRec r = bv.rec[bv.inv[i]];
    float best = INFINITY;
    int bg = 0;
    for (int g = 0; g < G; ++g) {
        const float dx = r.a.x - cent[3 * g], dy = r.a.y - cent[3 * g + 1], dz = r.a.z - cent[3 * g + 2];
        const float d2 = dx * dx + dy * dy + dz * dz;
        if (d2 < best) {
            best = d2;
            bg = g;
        }
    }
    key[i] = (uint32_t)bg;
    ids[i] = (uint32_t)i;
    atomicAdd(count + bg, 1u);
}

// wave per group: mean centre and mean normal of its members (fixed order);
// an empty group keeps its centre
__global__ void __launch_bounds__(256) k_km_update(BvhDev bv, int G, const int64_t *__restrict__ goff,
                                                   const uint32_t *__restrict__ members, float *__restrict__ cent,
                                                   float *__restrict__ gnrm) {
    const int g = blockIdx.x * 4 + threadIdx.x / 64;
    if (g >= G) return;
    const int lane = __lane_id();
    const int64_t b = goff[g], e = goff[g + 1];
    float s[6] = {0, 0, 0, 0, 0, 0};
    for (int64_t k = b + lane; k < e; k += 64) {
        const SurfRec r = bv.rec[bv.inv[members[k]]];
        s[0] += r.a.x;
        s[1] += r.a.y;
        s[2] += r.a.z;
        s[3] += r.b.x;
        s[4] += r.b.y;
        s[5] += r.b.z;
    }
#pragma unroll
    for (int q = 0; q < 6; ++q)
        for (int off = 32; off > 0; off >>= 1) s[q] += __shfl_xor(s[q], off, 64);
    if (lane == 0 && e > b) {
        const float inv = 1.0f / (float)(e - b);
        cent[3 * g + 0] = s[0] * inv;
        cent[3 * g + 1] = s[1] * inv;
        cent[3 * g + 2] = s[2] * inv;
        gnrm[3 * g + 0] = s[3] * inv;
        gnrm[3 * g + 1] = s[4] * inv;
        gnrm[3 * g + 2] = s[5] * inv;
    }
}

// wave per group: summed luminance of the members' current radiance (the
// DC coefficient of every light)
__global__ void __launch_bounds__(256) k_mc_lum(int G, const int64_t *__restrict__ goff,
                                                const uint32_t *__restrict__ members, const float *__restrict__ B,
                                                int Lt, int K, float *__restrict__ L) {
    const int g = blockIdx.x * 4 + threadIdx.x / 64;
    if (g >= G) return;
    const int lane = __lane_id();
    const int C = Lt * K * 3;
    float s = 0.0f;
    for (int64_t k = goff[g] + lane; k < goff[g + 1]; k += 64) {
        const float *bj = B + (int64_t)members[k] * C;
        for (int l = 0; l < Lt; ++l) s += lum3(bj + l * K * 3);
    }
    for (int off = 32; off > 0; off >>= 1) s += __shfl_xor(s, off, 64);
    if (lane == 0) L[g] = s;
}

__device__ __forceinline__ float member_weight(const SurfRec &ra, const SurfRec &rj, float lumj) {
    const float vx = rj.a.x - ra.a.x, vy = rj.a.y - ra.a.y, vz = rj.a.z - ra.a.z;
    const float r2 = vx * vx + vy * vy + vz * vz;
    if (!(r2 > 0.0f)) return 0.0f;
    const float ca = fabsf(ra.b.x * vx + ra.b.y * vy + ra.b.z * vz);
    const float cj = fabsf(rj.b.x * vx + rj.b.y * vy + rj.b.z * vz);
    return lumj * (ca * cj) / (r2 * r2);
}

__device__ __forceinline__ float group_weight(const SurfRec &ra, const float *cent, const float *gnrm, float Lg,
                                              float rmin2) {
    const float vx = cent[0] - ra.a.x, vy = cent[1] - ra.a.y, vz = cent[2] - ra.a.z;
    const float r2 = fmaxf(vx * vx + vy * vy + vz * vz, rmin2);
    const float il = 1.0f / sqrtf(r2);
    const float ca = fabsf(ra.b.x * vx + ra.b.y * vy + ra.b.z * vz) * il;
    const float cg = fabsf(gnrm[0] * vx + gnrm[1] * vy + gnrm[2] * vz) * il;
    return Lg * (ca + kMcBeta) * (cg + kMcBeta) / r2;
}

// What the member draws read of a surfel, in the groups' member order:
// centre and the luminance of its current radiance, normal and index.  Made
// once a round, so that a draw streams its group's members instead of
// following three indices to each.
struct McMember {
    float4 p, n;
};

__global__ void __launch_bounds__(256) k_mc_members(BvhDev bv, const uint32_t *__restrict__ members,
                                                    const float *__restrict__ B, int Lt, int K,
                                                    McMember *__restrict__ mem) {
    const int64_t k = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (k >= bv.n) return;
    const uint32_t j = members[k];
    const SurfRec r = bv.rec[bv.inv[j]];
    const float *bj = B + (int64_t)j * Lt * K * 3;
    float lj = 0.0f;
    for (int l = 0; l < Lt; ++l) lj += lum3(bj + l * K * 3);
    mem[k].p = make_float4(r.a.x, r.a.y, r.a.z, lj);
    mem[k].n = make_float4(r.b.x, r.b.y, r.b.z, __uint_as_float(j));
}

// Inverse CDF of weight(0 .. n) by a row of 16 lanes: `at`, the first w > 0
// whose running sum exceeds u times the total (else the last w > 0; -1: the
// total is not positive).  Each lane forms the weight of every 16th entry, and
// all lanes add them in order, broadcast lane by lane, so the sums are those
// of one lane that walks the list.  The running sum is kept at 16 points of
// the list, one per lane, and the pick starts from the last point before it
// instead of forming all weights again.
struct RowPick {
    int64_t at = -1;
    float w = 0.0f, total = 0.0f;
};

template <typename Weight>
__device__ __forceinline__ RowPick row_pick(int64_t n, float u, Weight &&weight) {
    constexpr auto kRow = std::make_integer_sequence<int, 16>{};
    const int l = threadIdx.x & 15, row = (int)__lane_id() & 48;
    auto lane_weight = [&](int64_t k) { return k < n ? weight(k) : 0.0f; };
    const int64_t part = ((n + 255) / 256) * 16;   // entries between two points
    RowPick p;
    float run = 0.0f, mine = 0.0f;   // sum of the positive weights; at the end of part l
    for (int64_t k0 = 0, end = part; k0 < n; k0 += 16) {
        each_lane(kRow, lane_weight(k0 + l), [&](int, float x) {
            p.total += x;
            run += x <= 0.0f ? 0.0f : x;
        });
        if (k0 + 16 == end || k0 + 16 >= n) {
            if ((end / part - 1) == l) mine = run;
            end += part;
        }
    }
    if (!(p.total > 0.0f)) return p;
    const float target = u * p.total;
    const uint32_t over = (uint32_t)(__ballot(mine > target) >> row) & 0xffffu;
    const int first = over ? __ffs((int)over) - 1 : 0;
    const float before = __shfl(mine, row + max(first - 1, 0));
    float acc = first > 0 ? before : 0.0f;
    bool found = false;
    for (int64_t k0 = first * part; k0 < n && !found; k0 += 16) {
        each_lane(kRow, lane_weight(k0 + l), [&](int i, float x) {
            if (found || x <= 0.0f) return;
            acc += x;
            p.at = k0 + i;
            p.w = x;
            found = acc > target;
        });
    }
    return p;
}

// One draw per slot: receiver recv[slot] (slot itself when recv is NULL) draws
// a group and a member of it; jsel (-1: none) and its probability.  16 lanes
// per receiver.  One lane per receiver left most of the chip without work and
// waited for each member's record in turn: draw and walk 1.65 ms for 50k
// receivers, now 0.11 and 0.24 ms.
__global__ void __launch_bounds__(kRowThreads) k_mc_select(BvhDev bv, int G, const int64_t *__restrict__ goff,
                                                           const McMember *__restrict__ mem,
                                                           const float *__restrict__ cent,
                                                           const float *__restrict__ gnrm,
                                                           const float *__restrict__ Lg, float rmin2,
                                                           const int32_t *__restrict__ recv, int64_t block0,
                                                           int64_t slots, uint64_t seed, int step, int32_t *__restrict__ jsel_out,
                                                           float *__restrict__ pj_out) {
    const int64_t s = (block0 + blockIdx.x) * (kRowThreads / 16) + threadIdx.x / 16;
    if (s >= slots) return;
    const int64_t a = recv ? (int64_t)recv[s] : s;
    const SurfRec ra = bv.rec[bv.inv[a]];
    uint64_t w[4];
    philox4x64_10((uint64_t)s, (uint64_t)step, 0ull, 2ull, seed, 0ull, w);
    const RowPick g = row_pick(G, u01(w[0]), [&](int64_t i) {
        return group_weight(ra, cent + 3 * i, gnrm + 3 * i, Lg[i], rmin2);
    });
    int64_t jsel = -1;
    float pj = 0.0f;
    if (g.at >= 0) {
        const McMember *list = mem + goff[g.at];
        const RowPick m = row_pick(goff[g.at + 1] - goff[g.at], u01(w[1]), [&](int64_t k) {
            const McMember r = list[k];
            if ((int64_t)__float_as_uint(r.n.w) == a) return 0.0f;
            SurfRec rj;
            rj.a = r.p;
            rj.b = r.n;
            return member_weight(ra, rj, r.p.w);
        });
        if (m.at >= 0) {
            jsel = (int64_t)__float_as_uint(list[m.at].n.w);
            pj = (g.w / g.total) * (m.w / m.total);
        }
    }
    if ((threadIdx.x & 15) == 0) {
        jsel_out[s] = (int32_t)jsel;
        pj_out[s] = pj;
    }
}

// The estimates of the drawn pairs: current radiance B, writes delta
// [slots][C], 16 lanes per slot.
__global__ void __launch_bounds__(kRowThreads) k_mc_ne(BvhDev bv, const int32_t *__restrict__ recv, int64_t block0,
                                                       int64_t slots,
                                                       const int32_t *__restrict__ jsel_in,
                                                       const float *__restrict__ pj_in,
                                                       const float *__restrict__ lambda,
                                                       const float *__restrict__ rho, const float *__restrict__ E,
                                                       const float *__restrict__ B, int C, float *__restrict__ delta,
                                                       int *err) {
    __shared__ uint64_t stack[kRowThreads / 16][kRowStack];
    const int64_t s = (block0 + blockIdx.x) * (kRowThreads / 16) + threadIdx.x / 16;
    if (s >= slots) return;
    const int64_t a = recv ? (int64_t)recv[s] : s;
    const SurfRec ra = bv.rec[bv.inv[a]];
    const float *Ea = E + a * C;
    float *out = delta + s * C;
    const int64_t jsel = jsel_in[s];
    const float pj = pj_in[s];
    float scale = 0.0f;
    if (jsel >= 0 && pj > 0.0f) {
        const SurfRec rj = bv.rec[bv.inv[jsel]];
        const Segment g = make_segment(ra, rj, bv.bounds[6]);
        const float T = row_segment(bv, g, (uint32_t)a, (uint32_t)jsel, stack[threadIdx.x / 16], err);
        const float aa = fabsf(ra.b.x * g.dx + ra.b.y * g.dy + ra.b.z * g.dz);
        const float bb = fabsf(rj.b.x * g.dx + rj.b.y * g.dy + rj.b.z * g.dz);
        const float r2 = g.dx * g.dx + g.dy * g.dy + g.dz * g.dz;
        const float F = lambda[jsel] * (float)bv.area[jsel] * T * (aa * bb) / (r2 * r2) * kInvPi;
        scale = F / pj;
    }
    const float *Bj = jsel >= 0 ? B + jsel * C : nullptr;
    for (int c = threadIdx.x & 15; c < C; c += 16) {
        const float add = Bj ? rho[3 * a + c % 3] * scale * Bj[c] : 0.0f;
        out[c] = Ea[c] + add;
    }
}

// B = S / D per receiver (0 where never visited)
__global__ void __launch_bounds__(256) k_mc_mean(const float *__restrict__ S, const uint32_t *__restrict__ D,
                                                 int64_t n, int C, float *__restrict__ B) {
    const int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (t >= n * C) return;
    const uint32_t d = D[t / C];
    B[t] = d ? S[t] / (float)d : 0.0f;
}

// Receivers add their slots' estimates in slot order (slots sorted by
// receiver; NULL recv: slot a is receiver a).  The first slot of a receiver
// adds them all, so that no receiver looks for its slots: by binary search
// 50 us for 50k slots, now 35 us.
__global__ void __launch_bounds__(256) k_mc_accum(const int32_t *__restrict__ recv, int64_t slots,
                                                  const float *__restrict__ delta, int C, float *__restrict__ S,
                                                  float *__restrict__ S2, uint32_t *__restrict__ D) {
    const int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const int64_t first = t / C;
    const int c = (int)(t % C);
    if (first >= slots) return;
    const int64_t a = recv ? (int64_t)recv[first] : first;
    if (recv && first > 0 && recv[first - 1] == a) return;
    float s = S[a * C + c], s2 = S2[a * C + c];
    int64_t k = first;
    do {
        const float d = delta[k * C + c];
        s += d;
        s2 = __builtin_fmaf(d, d, s2);
        ++k;
    } while (recv && k < slots && recv[k] == a);
    S[a * C + c] = s;
    S2[a * C + c] = s2;
    if (c == 0) D[a] += (uint32_t)(k - first);
}

// per-receiver variance of the estimates, summed over the columns, and its
// maximum (float bits)
__global__ void __launch_bounds__(256) k_mc_var(const float *__restrict__ S, const float *__restrict__ S2,
                                                const uint32_t *__restrict__ D, int64_t n, int C,
                                                float *__restrict__ var, uint32_t *maxbits) {
    const int64_t a = (int64_t)blockIdx.x * 256 + threadIdx.x;
    float v = 0.0f;
    if (a < n && D[a] > 0) {
        const float id = 1.0f / (float)D[a];
        for (int c = 0; c < C; ++c) {
            const float m = S[a * C + c] * id;
            v += fmaxf(0.0f, S2[a * C + c] * id - m * m);
        }
        var[a] = v;
    } else if (a < n) {
        var[a] = 0.0f;
    }
    for (int off = 32; off > 0; off >>= 1) v = fmaxf(v, __shfl_xor(v, off, 64));
    if (__lane_id() == 0 && v > 0.0f) atomicMax(maxbits, __float_as_uint(v));
}

// integer selection weights (variance relative to the maximum, 2^24 levels)
__global__ void __launch_bounds__(256) k_mc_quant(const float *__restrict__ var, const uint32_t *maxbits, int64_t n,
                                                  uint32_t *__restrict__ q) {
    const int64_t a = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (a >= n) return;
    const float m = __uint_as_float(*maxbits);
    q[a] = m > 0.0f ? (uint32_t)__float2uint_rn(var[a] / m * 16777216.0f) : 1u;
}

// slot s draws its receiver by the stratified inverse of the integer CDF:
// target = floor((s + xi_s) / N * total), receiver = first a with cdf[a+1] > target
__global__ void __launch_bounds__(256) k_mc_draw(const int64_t *__restrict__ cdf, int64_t n, uint64_t seed, int step,
                                                 int32_t *__restrict__ recv) {
    const int64_t s = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (s >= n) return;
    const uint64_t total = (uint64_t)cdf[n];
    uint64_t w[4];
    philox4x64_10((uint64_t)s, (uint64_t)step, 1ull, 1ull, seed, 0ull, w);
    // floor((s + w / 2^64) total / n) in integers
    int64_t target = (int64_t)(((uint64_t)s * total + __umul64hi(w[0], total)) / (uint64_t)n);
    if (target >= (int64_t)total) target = (int64_t)total - 1;
    int64_t l = 0, h = n;
    while (l < h) {
        const int64_t m = (l + h) >> 1;
        if (cdf[m + 1] <= target) l = m + 1;
        else h = m;
    }
    recv[s] = (int32_t)min<int64_t>(l, n - 1);
}

}  // namespace

// --- Monte-Carlo solver host side ---------------------------------------
size_t mc_member_bytes(int64_t n) { return (size_t)n * sizeof(McMember); }

gsrad_status mc_kmeans(const BvhDev &bv, int G, int iters, McBuffers &mb, hipStream_t st) {
    const int64_t n = bv.n;
    const unsigned gn = (unsigned)((n + 255) / 256);
    int bits = 1;
    while ((1 << bits) < G) ++bits;
    hipLaunchKernelGGL(k_km_init, dim3((unsigned)((G + 255) / 256)), dim3(256), 0, st, bv, G, mb.cent);
    for (int it = 0; it < iters; ++it) {
        gsrad_status e = check_hip(hipMemsetAsync(mb.count, 0, (size_t)G * 4, st), "k-means counts");
        if (e != GSRAD_OK) return e;
        hipLaunchKernelGGL(k_km_assign, dim3(gn), dim3(256), 0, st, bv, G, mb.cent, mb.key, mb.ids, mb.count);
        if ((e = radix_sort_pairs(mb.key, mb.ids, mb.skey, mb.members, n, bits, mb.rtemp, mb.rtemp_bytes, st)) !=
            GSRAD_OK)
            return e;
        if ((e = exclusive_scan_u32_i64(mb.count, mb.goff, G, mb.stemp, mb.stemp_bytes, st)) != GSRAD_OK) return e;
        hipLaunchKernelGGL(k_km_update, dim3((unsigned)((G + 3) / 4)), dim3(256), 0, st, bv, G, mb.goff, mb.members,
                           mb.cent, mb.gnrm);
    }
    return check_hip(hipGetLastError(), "k-means launch");
}

gsrad_status mc_step(const BvhDev &bv, const McBuffers &mb, int G, float rmin2, const float *lambda, const float *rho,
                     const float *E, const float *B, int Lt, int K, uint64_t seed, int step, const int32_t *recv,
                     float *delta, int *err, hipStream_t st) {
    const int64_t n = bv.n;
    hipLaunchKernelGGL(k_mc_lum, dim3((unsigned)((G + 3) / 4)), dim3(256), 0, st, G, mb.goff, mb.members, B, Lt, K,
                       mb.L);
    McMember *mem = static_cast<McMember *>(mb.mem);
    hipLaunchKernelGGL(k_mc_members, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, bv, mb.members, B, Lt, K, mem);
    const int64_t groups = (n + kRowThreads / 16 - 1) / (kRowThreads / 16);
    each_launch(groups, kRowThreads, [&](int64_t first, unsigned blocks) {
        hipLaunchKernelGGL(k_mc_select, dim3(blocks), dim3(kRowThreads), 0, st, bv, G, mb.goff, mem, mb.cent, mb.gnrm,
                           mb.L, rmin2, recv, first, n, seed, step, mb.jsel, mb.pj);
    });
    each_launch(groups, kRowThreads, [&](int64_t first, unsigned blocks) {
        hipLaunchKernelGGL(k_mc_ne, dim3(blocks), dim3(kRowThreads), 0, st, bv, recv, first, n, mb.jsel, mb.pj, lambda,
                           rho, E, B, Lt * K * 3, delta, err);
    });
    return check_hip(hipGetLastError(), "next event launch");
}

gsrad_status mc_solve(const BvhDev &bv, const McBuffers &mb, int G, float rmin2, const float *lambda,
                      const float *rho, const float *E, int Lt, int K, int T, uint64_t seed, float *B_out,
                      int *err, hipStream_t st) {
    const int64_t n = bv.n;
    const int C = Lt * K * 3;
    const size_t bytes = (size_t)n * C * 4;
    gsrad_status e;
    if ((e = check_hip(hipMemsetAsync(mb.S, 0, bytes, st), "mc zero")) != GSRAD_OK) return e;
    if ((e = check_hip(hipMemsetAsync(mb.S2, 0, bytes, st), "mc zero")) != GSRAD_OK) return e;
    if ((e = check_hip(hipMemsetAsync(mb.D, 0, (size_t)n * 4, st), "mc zero")) != GSRAD_OK) return e;
    const unsigned gv = (unsigned)((n * C + 255) / 256), gn = (unsigned)((n + 255) / 256);
    for (int t = 0; t < T; ++t) {
        hipLaunchKernelGGL(k_mc_mean, dim3(gv), dim3(256), 0, st, mb.S, mb.D, n, C, mb.B);
        const int32_t *recv = nullptr;
        if (t >= 8) {
            if ((e = check_hip(hipMemsetAsync(mb.maxbits, 0, 4, st), "mc max")) != GSRAD_OK) return e;
            hipLaunchKernelGGL(k_mc_var, dim3(gn), dim3(256), 0, st, mb.S, mb.S2, mb.D, n, C, mb.var, mb.maxbits);
            hipLaunchKernelGGL(k_mc_quant, dim3(gn), dim3(256), 0, st, mb.var, mb.maxbits, n, mb.q);
            if ((e = exclusive_scan_u32_i64(mb.q, mb.cdf, n, mb.stemp, mb.stemp_bytes, st)) != GSRAD_OK) return e;
            hipLaunchKernelGGL(k_mc_draw, dim3(gn), dim3(256), 0, st, mb.cdf, n, seed, t, mb.recv);
            recv = mb.recv;
        }
        if ((e = mc_step(bv, mb, G, rmin2, lambda, rho, E, mb.B, Lt, K, seed, t, recv, mb.delta, err, st)) != GSRAD_OK)
            return e;
        hipLaunchKernelGGL(k_mc_accum, dim3(gv), dim3(256), 0, st, recv, n, mb.delta, C, mb.S, mb.S2, mb.D);
    }
    hipLaunchKernelGGL(k_mc_mean, dim3(gv), dim3(256), 0, st, mb.S, mb.D, n, C, B_out);
    return check_hip(hipGetLastError(), "mc solve launch");
}

}  // namespace gsrad
