// Gradient kernels through the centre-to-centre form factors (Sec. 8), the
// ray-cast form factors' geometry (recorded hits) and the direct light.
//
// k_ff_center       one workgroup per row of a pattern: the centre-to-centre
//                   F with the learnable decay scale lambda.
// k_center_rows     its gradient with respect to lambda and every surfel
//                   field on each segment (endpoints and occluders);
//                   k_center_bwd what does not fit its lists.
// k_geometry_rec    dL/dF through the recorded hits to centres, frames,
//                   scales and opacities.
// k_light_*         the direct light's gradient: lights, albedo, receivers
//                   and shadow-segment occluders.
// The sums over surfels, scales and lights are 64-bit fixed point with a scale
// per field, one copy per XCD; the albedo's, a surfel's own, is FP32 in the
// order of the lights.  Both are bit-identical between runs.
#include <algorithm>
#include <cstring>
#include <functional>

#include "gsrad_internal.h"
#include "sh_api.h"
#include "trace_api.h"
#include "traverse.h"
#include "hit_lists.h"

namespace gsrad {

namespace {

// ---------------------------------------------------------------------------
// centre-to-centre form factors (Sec. 8) and their gradients
// ---------------------------------------------------------------------------
// F_ij = lambda_j A_j T_ij |n_i . v| |n_j . v| / (pi |v|^4) per stored entry
// of the pattern (v = p_j - p_i); one workgroup per row, 16 lanes per entry.
// Bound by the walks (row_crossings): 10 M segments of a 20k-surfel bowl in
// 14.6 ms, with a segment a lane 24.2 ms.
__global__ void __launch_bounds__(kRowThreads) k_ff_center(BvhDev bv, const int64_t *__restrict__ row_ptr,
                                                           const int32_t *__restrict__ col, int64_t n,
                                                           const float *__restrict__ lambda,
                                                           float *__restrict__ val, int64_t block0, int64_t nblocks,
                                                           const int32_t *__restrict__ order, int *err) {
    __shared__ int32_t stack[kRowThreads / 16][kCrossNodes + kCrossLeaves];
    const int64_t idx = xcd_block(block0 + blockIdx.x, nblocks);
    const int64_t row = order ? (int64_t)order[idx] : idx;
    const SurfRec ri = bv.rec[bv.inv[row]];
    const int64_t b = row_ptr[row], e = row_ptr[row + 1];
    const float t_eps = bv.bounds[6];
    for (int64_t kk = b + threadIdx.x / 16; kk < e; kk += kRowThreads / 16) {
        const int32_t j = col[kk];
        const SurfRec rj = bv.rec[bv.inv[j]];
        const Segment g = make_segment(ri, rj, t_eps);
        const float T = row_crossings(bv, g, (uint32_t)row, (uint32_t)j, stack[threadIdx.x / 16], err, [](int) {});
        const float a = ri.b.x * g.dx + ri.b.y * g.dy + ri.b.z * g.dz;
        const float bb = rj.b.x * g.dx + rj.b.y * g.dy + rj.b.z * g.dz;
        const float r2 = g.dx * g.dx + g.dy * g.dy + g.dz * g.dz;
        const float phi = (fabsf(a) * fabsf(bb)) / (r2 * r2);
        if ((threadIdx.x & 15) == 0) val[kk] = lambda[j] * (float)bv.area[j] * T * phi * kInvPi;
    }
}

// Accumulated fields of the gradient kernels, per surfel in 64-bit fixed
// point.  0-11 hold world-space sums (centre, t_u, t_v, n) of the terms that
// have no plane of their own: a receiver's or a segment's ends.  12 is the
// opacity, 13 a pair's sum of G T Phi (the chain through lambda_j A_j).
// 14-22 are the sums of what a crossing adds to the surfel it crosses: with h
// the crossing relative to its centre, du = dL/du / s_u, dw = dL/dw / s_v and
// beta = (du t_u + dw t_v) . d / (d . n),
//   p += beta n - du t_u - dw t_v,  t_u += du h,  t_v += dw h,  n -= beta h,
//   s_u -= du u,  s_v -= dw w.
// t_u, t_v, n are the surfel's own and h lies in its plane (h . n = 0), so h's
// two coordinates outside the largest axis of n give the third: ten sums per
// crossing (these nine and the opacity) instead of the fifteen gradients they
// determine, which k_fields_finish forms from them.
enum {
    kFp = 0, kFtu = 3, kFtv = 6, kFn = 9, kFo = 12, kFpair = 13,
    kFdu = 14, kFdw = 15, kFbeta = 16, kFduh = 17, kFdwh = 19, kFbetah = 21, kFields = 23
};

// Axis of n that k_fields_finish recovers (its largest; the first on ties)
__device__ __forceinline__ int plane_axis(float nx, float ny, float nz) {
    const float ax = fabsf(nx), ay = fabsf(ny), az = fabsf(nz);
    return ax >= ay && ax >= az ? 0 : (ay >= az ? 1 : 2);
}

// a crossing at h of a surfel with record r: what it adds to fields
// kFdu ... kFdu + 8
__device__ __forceinline__ void cross_terms(const SurfRec &r, float du, float dw, float beta, float hx,
                                            float hy, float hz, float *x) {
    const int ax = plane_axis(r.b.x, r.b.y, r.b.z);
    const float ha = ax == 0 ? hy : hx, hb = ax == 2 ? hy : hz;
    x[0] = du;
    x[1] = dw;
    x[2] = beta;
    x[3] = du * ha;
    x[4] = du * hb;
    x[5] = dw * ha;
    x[6] = dw * hb;
    x[7] = beta * ha;
    x[8] = beta * hb;
}

__device__ __forceinline__ float wave_max(float v) {
    for (int off = 32; off > 0; off >>= 1) v = fmaxf(v, __shfl_xor(v, off, 64));
    return v;
}

// *p = max(*p, bits of v >= 0).  A look first: all waves raise the same few
// words, and once a word is near its maximum almost none has to (16k surfels
// x 100 lights, 26,000 waves: pass 0 3.0 ms with an atomic per field and wave,
// 0.5 ms so).
__device__ __forceinline__ void raise(uint32_t *p, float v) {
    const uint32_t bits = __float_as_uint(v);
    if (bits > __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) atomicMax(p, bits);
}

// Pass 0 finds max |contribution| per field, pass 1 adds the contributions
// in 64-bit fixed point with a per-field power-of-two scale (integer adds
// commute: bit-identical between runs) into one copy per XCD.
template <int PASS>
struct FieldSink {
    float m[kFields];         // pass 0: largest |contribution| per field
    float qm;                 // pass 1: largest |scaled contribution| (INFINITY once one is not finite)
    unsigned long long *acc;
    const int *fx;
    int64_t n;
    __device__ __forceinline__ void init(unsigned long long *copies, const int *exps, int64_t surfels) {
#pragma unroll
        for (int f = 0; f < kFields; ++f) m[f] = 0.0f;
        qm = 0.0f;
        acc = copies + (int64_t)xcc_id() * kFields * surfels;
        fx = exps;
        n = surfels;
    }
    __device__ __forceinline__ void track(float q) {
        const float a = fabsf(q);
        qm = a <= 3.0e38f ? fmaxf(qm, a) : INFINITY;
    }
    __device__ __forceinline__ long long scaled(int f, float v) {
        const float q = v * __builtin_ldexpf(1.0f, fx[f]);
        track(q);
        return __float2ll_rn(q);
    }
    __device__ __forceinline__ void add_scaled(int f, uint32_t surfel, long long q) {
        __hip_atomic_fetch_add(acc + (int64_t)f * n + surfel, (unsigned long long)q, __ATOMIC_RELAXED,
                               __HIP_MEMORY_SCOPE_WORKGROUP);
    }
    __device__ __forceinline__ void add(int f, uint32_t surfel, float v) {
        if (PASS == 0) {
            m[f] = fmaxf(m[f], fabsf(v));
        } else {
            const long long q = scaled(f, v);
            if (q != 0) add_scaled(f, surfel, q);
        }
    }
    __device__ __forceinline__ void add3(int f, uint32_t surfel, float x, float y, float z) {
        add(f, surfel, x);
        add(f + 1, surfel, y);
        add(f + 2, surfel, z);
    }
    __device__ __forceinline__ void cross(uint32_t k, const SurfRec &r, float du, float dw, float beta, float hx,
                                          float hy, float hz) {
        float x[9];
        cross_terms(r, du, dw, beta, hx, hy, hz, x);
#pragma unroll
        for (int q = 0; q < 9; ++q) add(kFdu + q, k, x[q]);
    }
    // wave maxima to maxbits[f] (pass 0) or maxbits[2 kFields] (pass 1);
    // every lane of the wave calls this
    __device__ __forceinline__ void report(uint32_t *maxbits) {
        const int lane = (int)__lane_id();
        if (PASS == 0) {
            float mine = 0.0f;   // lane f's: field f
#pragma unroll
            for (int f = 0; f < kFields; ++f) {
                const float v = wave_max(m[f]);
                mine = lane == f ? v : mine;
            }
            if (lane < kFields) raise(maxbits + lane, mine);
        } else {
            const float v = wave_max(qm);
            if (lane == 0) raise(maxbits + 2 * kFields, v);
        }
    }
};

// Contributions of one thread to NF fields of one surfel that the whole
// wave shares (the row's receiver): summed per thread in the fields' 64-bit
// fixed point (exact), then over the wave, and added with one atomic per
// field instead of one per contribution to the same address.
template <int NF>
struct SharedSurfelAcc {
    long long q[NF];
    __device__ __forceinline__ void zero() {
#pragma unroll
        for (int f = 0; f < NF; ++f) q[f] = 0;
    }
    template <int PASS, typename Sink>
    __device__ __forceinline__ void add(Sink &sink, int slot, int field, float v) {
        if (PASS == 0) {
            sink.m[field] = fmaxf(sink.m[field], fabsf(v));
        } else {
            const float qv = v * __builtin_ldexpf(1.0f, sink.fx[field]);
            sink.track(qv);
            q[slot] += __float2ll_rn(qv);
        }
    }
    // every lane of the wave must call this (shuffles); lanes whose surfel
    // differs from lane 0's are not allowed
    template <int PASS>
    __device__ __forceinline__ void flush(unsigned long long *acc, int64_t n, uint32_t surfel, const int *fields) {
        if (PASS == 0) return;
#pragma unroll
        for (int f = 0; f < NF; ++f) {
            long long v = q[f];
            for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
            if (__lane_id() == 0 && v != 0)
                __hip_atomic_fetch_add(acc + (int64_t)fields[f] * n + surfel, (unsigned long long)v, __ATOMIC_RELAXED,
                                       __HIP_MEMORY_SCOPE_WORKGROUP);
        }
    }
};

// Crossings' sums of a workgroup in LDS: open addressing on the surfel, ten
// 64-bit fixed-point sums each (fields kFdu ... kFdu + 8 and kFo); a surfel
// that finds no place within kProbes adds to the global sums.
template <int SLOTS>
struct CrossTable {
    static constexpr int kProbes = 8, kSums = 10;
    uint32_t key[SLOTS];
    unsigned long long sum[kSums][SLOTS];
    static __device__ __forceinline__ int field(int q) { return q < 9 ? kFdu + q : kFo; }
    __device__ __forceinline__ void clear(int tid, int threads) {
        for (int z = tid; z < SLOTS; z += threads) {
            key[z] = kEmpty;
#pragma unroll
            for (int q = 0; q < kSums; ++q) sum[q][z] = 0;
        }
    }
    template <typename Sink>
    __device__ __forceinline__ void add(Sink &sink, uint32_t k, const float (&x)[kSums]) {
        const uint32_t h = (k * 0x9e3779b1u) >> 16;
        int at = -1;
        for (int p = 0; p < kProbes && at < 0; ++p) {
            const int z = (int)((h + (uint32_t)p) & (uint32_t)(SLOTS - 1));
            uint32_t old = key[z];
            if (old == kEmpty) old = atomicCAS(&key[z], kEmpty, k);
            if (old == kEmpty || old == k) at = z;
        }
#pragma unroll
        for (int q = 0; q < kSums; ++q) {
            const long long v = sink.scaled(field(q), x[q]);
            if (v == 0) continue;
            if (at >= 0) atomicAdd(&sum[q][at], (unsigned long long)v);
            else sink.add_scaled(field(q), k, v);
        }
    }
    template <typename Sink>
    __device__ __forceinline__ void flush(Sink &sink, int tid, int threads) {
        for (int z = tid; z < SLOTS; z += threads) {
            const uint32_t k = key[z];
            if (k == kEmpty) continue;
#pragma unroll
            for (int q = 0; q < kSums; ++q)
                if (sum[q][z] != 0) sink.add_scaled(field(q), k, (long long)sum[q][z]);
        }
    }
};

// One crossing of a segment o + t d with weight W: the crossed surfel's ten
// sums x, and the shares ge and gs of the segment's end and start.
__device__ __forceinline__ void crossing(const BvhDev &bv, const SurfRec &r, float ox, float oy, float oz,
                                         float dx, float dy, float dz, float W, float (&x)[10], float (&ge)[3],
                                               float (&gs)[3]) {
    const float ok = bv.raw_op[__float_as_uint(r.d.w)];
    const float gam = kernel_gamma(hit_r2_exact(r, ox, oy, oz, dx, dy, dz));
    const float qx = r.a.x - ox, qy = r.a.y - oy, qz = r.a.z - oz;
    const float den = dx * r.b.x + dy * r.b.y + dz * r.b.z;
    const float tk = (qx * r.b.x + qy * r.b.y + qz * r.b.z) / den;
    const float hx = tk * dx - qx, hy = tk * dy - qy, hz = tk * dz - qz;
    const float u = (hx * r.c.x + hy * r.c.y + hz * r.c.z) * r.a.w;
    const float w = (hx * r.d.x + hy * r.d.y + hz * r.d.z) * r.b.w;
    const float f = W * 3.4f * r.c.w * gam;
    const float fu = f * u * r.a.w, fw = f * w * r.b.w;
    const float ghx = fu * r.c.x + fw * r.d.x, ghy = fu * r.c.y + fw * r.d.y, ghz = fu * r.c.z + fw * r.d.z;
    const float beta = (ghx * dx + ghy * dy + ghz * dz) / den;
    const float gqx = beta * r.b.x - ghx, gqy = beta * r.b.y - ghy, gqz = beta * r.b.z - ghz;
    cross_terms(r, fu, fw, beta, hx, hy, hz, x);
    x[9] = ok > 0.0f && ok < kOpacityMax ? -W * gam / (1.0f - ok) : 0.0f;
    ge[0] = -tk * gqx;
    ge[1] = -tk * gqy;
    ge[2] = -tk * gqz;
    gs[0] = -(1.0f - tk) * gqx;
    gs[1] = -(1.0f - tk) * gqy;
    gs[2] = -(1.0f - tk) * gqz;
}

// The pair's own terms of a centre-to-centre segment: Phi = |a| |b| / r^4,
// kappa = lambda_j A_j / pi; the shares of p_j (-: of p_i), n_i and n_j and
// the term of the chain through lambda_j A_j.
struct PairTerm {
    float dp[3], ni[3], nj[3], chain;
    __device__ __forceinline__ PairTerm(const SurfRec &ri, const SurfRec &rj, const Segment &g, float G, float lambda_j,
                                        float A, float T) {
        const float a = ri.b.x * g.dx + ri.b.y * g.dy + ri.b.z * g.dz;
        const float bb = rj.b.x * g.dx + rj.b.y * g.dy + rj.b.z * g.dz;
        const float r2 = g.dx * g.dx + g.dy * g.dy + g.dz * g.dz;
        const float r4 = r2 * r2;
        const float aa = fabsf(a), ab = fabsf(bb);
        const float sa = a > 0.0f ? 1.0f : (a < 0.0f ? -1.0f : 0.0f);
        const float sb = bb > 0.0f ? 1.0f : (bb < 0.0f ? -1.0f : 0.0f);
        const float kT = G * lambda_j * A * T * kInvPi;
        const float c1 = kT * sa * ab / r4, c2 = kT * aa * sb / r4, c3 = 4.0f * kT * aa * ab / (r4 * r2);
        dp[0] = c1 * ri.b.x + c2 * rj.b.x - c3 * g.dx;
        dp[1] = c1 * ri.b.y + c2 * rj.b.y - c3 * g.dy;
        dp[2] = c1 * ri.b.z + c2 * rj.b.z - c3 * g.dz;
        ni[0] = c1 * g.dx;
        ni[1] = c1 * g.dy;
        ni[2] = c1 * g.dz;
        nj[0] = c2 * g.dx;
        nj[1] = c2 * g.dy;
        nj[2] = c2 * g.dz;
        chain = G * T * (aa * ab / r4) * kInvPi;
    }
};

// Crossings of the accumulating pass (64 bits), words after maxbits
constexpr int kCrossings = 3 * kFields + 3;
static_assert(kCrossings % 2 == 0, "aligned");

// What k_center_rows left of its rows (each from entry done[row]), a segment a
// lane.
template <int PASS>
__global__ void __launch_bounds__(kCenterThreads) k_center_bwd(BvhDev bv, const int64_t *__restrict__ row_ptr,
                                                               const int32_t *__restrict__ col,
                                                               const float *__restrict__ fval, int64_t n,
                                                               const float *__restrict__ lambda,
                                                               const float *__restrict__ gF, uint32_t *maxbits,
                                                               const int *fx, unsigned long long *acc,
                                                               int64_t nblocks, const int32_t *__restrict__ order,
                                                               int stride, const int32_t *__restrict__ done,
                                                               int *err) {
    extern __shared__ uint32_t stack_mem[];
    const int64_t idx = (xcd_block(blockIdx.x, nblocks) * (kCenterThreads / 64) + threadIdx.x / 64) * stride;
    if (idx >= n) return;
    const int64_t row = order ? (int64_t)order[idx] : idx;
    const int64_t b = row_ptr[row] + (int64_t)done[row], e = row_ptr[row + 1];
    if (b >= e) return;
    FieldSink<PASS> sink;
    sink.init(acc, fx, n);
    SharedSurfelAcc<6> accI;   // the row's receiver: p and n
    accI.zero();
    const uint32_t i = (uint32_t)row;
    unsigned long long hits = 0;
    const SurfRec ri = bv.rec[bv.inv[row]];
    for (int64_t kk = b + __lane_id(); kk < e; kk += 64) {
        const float G = gF[kk];
        if (G == 0.0f) continue;
        const uint32_t j = (uint32_t)col[kk];
        const SurfRec rj = bv.rec[bv.inv[j]];
        const Segment g = make_segment(ri, rj, bv.bounds[6]);
        const float W = G * fval[kk];
        float T = 1.0f;
        float gpi[3] = {0.0f, 0.0f, 0.0f}, gpj[3] = {0.0f, 0.0f, 0.0f};
        trace_segment(bv, g.ox, g.oy, g.oz, g.dx, g.dy, g.dz, i, j, g.t_lo, g.t_hi, stack_mem + threadIdx.x,
                                 kCenterThreads, err, [&](const SurfRec &r, int) {
                                     T = __fmul_rn(T, transmit(r.c.w, kernel_gamma(hit_r2_exact(r, g.ox, g.oy, g.oz,
                                                                                                g.dx, g.dy, g.dz))));
                                     float x[10], ge[3], gs[3];
                                     crossing(bv, r, g.ox, g.oy, g.oz, g.dx, g.dy, g.dz, W, x, ge, gs);
#pragma unroll
                                     for (int q = 0; q < 10; ++q)
                                         sink.add(CrossTable<1>::field(q), __float_as_uint(r.d.w), x[q]);
                                     // (pass 0: each share alone, as k_center_rows)
#pragma unroll
                                     for (int c = 0; c < 3; ++c) {
                                         gpi[c] = PASS == 0 ? fmaxf(gpi[c], fabsf(gs[c])) : gpi[c] + gs[c];
                                         gpj[c] = PASS == 0 ? fmaxf(gpj[c], fabsf(ge[c])) : gpj[c] + ge[c];
                                     }
                                     ++hits;
                                 });
        const PairTerm t(ri, rj, g, G, lambda[j], (float)bv.area[j], T);
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            if (PASS == 0) {
                sink.add(kFp + c, j, fmaxf(fabsf(t.dp[c]), fmaxf(gpi[c], gpj[c])));
            } else {
                sink.add(kFp + c, j, t.dp[c] + gpj[c]);
                accI.add<PASS>(sink, c, kFp + c, gpi[c] - t.dp[c]);
            }
            accI.add<PASS>(sink, 3 + c, kFn + c, t.ni[c]);
            sink.add(kFn + c, j, t.nj[c]);
        }
        sink.add(kFpair, j, t.chain);
    }
    const int fI[6] = {kFp, kFp + 1, kFp + 2, kFn, kFn + 1, kFn + 2};
    accI.flush<PASS>(sink.acc, n, i, fI);
    sink.report(maxbits);
    if (PASS == 1) {
        for (int off = 32; off > 0; off >>= 1) hits += __shfl_xor(hits, off, 64);
        if (__lane_id() == 0) atomicAdd(reinterpret_cast<unsigned long long *>(maxbits + kCrossings), hits);
    }
}

// A workgroup takes a row, kRowSegs entries of it at a
// time.  Rows of 16 lanes walk the segments and list their crossings (the
// segment and the surfel's sorted position) in kRowParts parts by a hash of
// the surfel; then part after part is dealt evenly to the lanes and summed in
// a table in LDS.  A row of 512 entries crosses some 1,900 surfels 17,000
// times, so ten sums per surfel and row go to memory instead of ten per
// crossing.  Bound by the walks (14.6 of 23.8 ms for 10 M segments of a 20k-surfel
// bowl, as long as k_ff_center), then by the LDS atomics.  A segment a lane
// and ten global atomics a crossing took 108 ms.
// The lists lie in the workgroup's own stretch of the workspace; a row that
// crosses more surfels than fit is left to k_center_bwd from there (done[row]).
constexpr int kCenterRowThreads = 512, kRowSegs = 512, kRowParts = 5, kRowSlots = 512;
constexpr int kRowPart = 13312;        // list places of a part
constexpr int64_t kCenterGroups = 512;   // workgroups, two a CU

struct RowShared {
    union {
        int32_t stack[kCenterRowThreads / 16][kCrossNodes + kCrossLeaves];
        CrossTable<kRowSlots> table;
    };
    float d[3][kRowSegs], W[kRowSegs], T[kRowSegs];
    unsigned long long end[3][kRowSegs];   // shares of the segments' ends, fixed point
    uint32_t count[kRowParts];
};

template <int PASS>
__global__ void __launch_bounds__(kCenterRowThreads, 4) k_center_rows(BvhDev bv, const int64_t *__restrict__ row_ptr,
                                                                   const int32_t *__restrict__ col,
                                                                   const float *__restrict__ fval, int64_t n,
                                                                   const float *__restrict__ lambda,
                                                                   const float *__restrict__ gF, uint32_t *maxbits,
                                                                   const int *fx, unsigned long long *acc,
                                                                   const int32_t *__restrict__ order, int stride,
                                                                   uint2 *__restrict__ lists,
                                                                   int32_t *__restrict__ done, int *err) {
    extern __shared__ __align__(16) char row_mem[];
    RowShared &sh = *reinterpret_cast<RowShared *>(row_mem);
    const int tid = threadIdx.x;
    uint2 *list = lists + (int64_t)blockIdx.x * kRowParts * kRowPart;
    FieldSink<PASS> sink;
    sink.init(acc, fx, n);
    unsigned long long hits = 0;
    for (int64_t idx = (int64_t)blockIdx.x * stride; idx < n; idx += (int64_t)gridDim.x * stride) {
        const int64_t row = order ? (int64_t)order[idx] : idx;
        const SurfRec ri = bv.rec[bv.inv[row]];
        const int64_t b = row_ptr[row], e = row_ptr[row + 1];
        SharedSurfelAcc<6> accI;   // the row's receiver: p and n
        accI.zero();
        int64_t k0 = b;
        for (; k0 < e; k0 += kRowSegs) {
            const int segs = (int)min<int64_t>(kRowSegs, e - k0);
            if (tid < kRowParts) sh.count[tid] = 0;
            __syncthreads();
            for (int q = tid / 16; q < segs; q += kCenterRowThreads / 16) {
                const float G = gF[k0 + q];
                const int32_t j = col[k0 + q];
                const Segment g = make_segment(ri, bv.rec[bv.inv[j]], bv.bounds[6]);
                float T = 1.0f;
                if (G != 0.0f)
                    T = row_crossings(bv, g, (uint32_t)row, (uint32_t)j, sh.stack[tid / 16], err, [&](int s) {
                        const uint32_t part = __umulhi((uint32_t)s * 0x85ebca6bu, (uint32_t)kRowParts);
                        const uint32_t at = atomicAdd(&sh.count[part], 1u);
                        if (at < (uint32_t)kRowPart) list[part * kRowPart + at] = make_uint2((uint32_t)q, (uint32_t)s);
                    });
                if ((tid & 15) == 0) {
                    sh.d[0][q] = g.dx;
                    sh.d[1][q] = g.dy;
                    sh.d[2][q] = g.dz;
                    sh.W[q] = G * fval[k0 + q];
                    sh.T[q] = T;
                }
            }
            __syncthreads();
            bool fits = true;
            for (int part = 0; part < kRowParts; ++part) fits = fits && sh.count[part] <= (uint32_t)kRowPart;
            if (!fits) break;
            if (tid < segs) {
                const float G = gF[k0 + tid];
                const uint32_t j = (uint32_t)col[k0 + tid];
                long long own[3] = {0, 0, 0};
                if (G != 0.0f) {
                    const SurfRec rj = bv.rec[bv.inv[j]];
                    const PairTerm t(ri, rj, make_segment(ri, rj, bv.bounds[6]), G, lambda[j], (float)bv.area[j],
                                     sh.T[tid]);
#pragma unroll
                    for (int c = 0; c < 3; ++c) {
                        if (PASS == 1) own[c] = sink.scaled(kFp + c, t.dp[c]);
                        accI.add<PASS>(sink, c, kFp + c, -t.dp[c]);
                        accI.add<PASS>(sink, 3 + c, kFn + c, t.ni[c]);
                        sink.add(kFn + c, j, t.nj[c]);
                    }
                    sink.add(kFpair, j, t.chain);
                }
#pragma unroll
                for (int c = 0; c < 3; ++c) sh.end[c][tid] = (unsigned long long)own[c];
            }
            // parts share the table while they cannot fill it
            bool open = false;
            uint32_t used = 0;
            for (int part = 0; part < kRowParts; ++part) {
                const uint32_t count = sh.count[part];
                hits += count;
                if (count == 0) continue;
                if (PASS == 1 && (!open || used + count > (uint32_t)kRowSlots)) {
                    if (open) {
                        __syncthreads();
                        sh.table.flush(sink, tid, kCenterRowThreads);
                        __syncthreads();
                    }
                    sh.table.clear(tid, kCenterRowThreads);
                    __syncthreads();
                    open = true;
                    used = 0;
                }
                used += count;
                for (uint32_t h = tid; h < count; h += kCenterRowThreads) {
                    const uint2 hit = list[part * kRowPart + h];
                    const SurfRec r = bv.rec[hit.y];
                    float x[10], ge[3], gs[3];
                    crossing(bv, r, ri.a.x, ri.a.y, ri.a.z, sh.d[0][hit.x], sh.d[1][hit.x], sh.d[2][hit.x],
                             sh.W[hit.x], x, ge, gs);
#pragma unroll
                    for (int c = 0; c < 3; ++c) {
                        accI.add<PASS>(sink, c, kFp + c, gs[c]);
                        if (PASS == 0) {
                            sink.add(kFp + c, 0, ge[c]);
                        } else {
                            const long long v = sink.scaled(kFp + c, ge[c]);
                            if (v != 0) atomicAdd(&sh.end[c][hit.x], (unsigned long long)v);
                        }
                    }
                    if (PASS == 0) {
#pragma unroll
                        for (int q = 0; q < 10; ++q) sink.add(sh.table.field(q), 0, x[q]);
                    } else {
                        sh.table.add(sink, __float_as_uint(r.d.w), x);
                    }
                }
            }
            if (open) {
                __syncthreads();
                sh.table.flush(sink, tid, kCenterRowThreads);
                __syncthreads();
            }
            if (PASS == 1 && tid < segs) {
                const uint32_t j = (uint32_t)col[k0 + tid];
#pragma unroll
                for (int c = 0; c < 3; ++c)
                    if (sh.end[c][tid] != 0) sink.add_scaled(kFp + c, j, (long long)sh.end[c][tid]);
            }
            __syncthreads();
        }
        if (tid == 0) done[row] = (int32_t)(min(k0, e) - b);
        const int fI[6] = {kFp, kFp + 1, kFp + 2, kFn, kFn + 1, kFn + 2};
        accI.flush<PASS>(sink.acc, n, (uint32_t)row, fI);
        __syncthreads();
    }
    sink.report(maxbits);
    if (PASS == 1 && tid == 0) atomicAdd(reinterpret_cast<unsigned long long *>(maxbits + kCrossings), hits);
}

// per-field exponent: (max contribution) * count * 2^margin < 2^62 (count
// bounds the contributions a surfel's field can receive; margin: headroom
// over a maximum estimated on sampled rows)
__global__ void k_fields_exp(const uint32_t *maxbits, int64_t count, int margin, int *fx) {
    const int f = threadIdx.x;
    if (f >= kFields) return;
    const float m = __uint_as_float(maxbits[f]);
    int e = 0;
    if (!(m <= 3.0e38f)) {
        e = kFxNonFinite;
    } else if (m > 0.0f) {
        int ex;
        (void)frexpf(m * (float)count, &ex);
        e = min(120, max(-120, 62 - ex - margin));
    }
    fx[f] = e;
}

// The gradients of the 15 surfel fields (and lambda) from the summed copies
// of the fields, one thread per surfel, FP64 up to the one rounding.
__global__ void __launch_bounds__(256) k_fields_finish(BvhDev bv, const unsigned long long *__restrict__ acc,
                                                       const int *fx, const float *__restrict__ lambda,
                                                       CenterOutputs out) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= bv.n) return;
    double v[kFields];
#pragma unroll
    for (int f = 0; f < kFields; ++f) {
        unsigned long long s = 0;
#pragma unroll
        for (int x = 0; x < 8; ++x) s += acc[((int64_t)x * kFields + f) * bv.n + i];
        const int e = fx[f];
        v[f] = e == kFxNonFinite ? (double)__builtin_nanf("") : ldexp((double)(long long)s, -e);
    }
    const SurfRec r = bv.rec[bv.inv[i]];
    const double tu[3] = {r.c.x, r.c.y, r.c.z}, tv[3] = {r.d.x, r.d.y, r.d.z}, nr[3] = {r.b.x, r.b.y, r.b.z};
    // the crossings' sums of du h, dw h, beta h with their third coordinate
    double duh[3], dwh[3], bh[3];
    auto expand = [&](int f, double (&h)[3]) {
        const int ax = plane_axis(r.b.x, r.b.y, r.b.z);
        const double a = v[f], b = v[f + 1];
        const double na = ax == 0 ? nr[1] : nr[0], nb = ax == 2 ? nr[1] : nr[2];
        const double nd = ax == 0 ? nr[0] : (ax == 1 ? nr[1] : nr[2]);
        const double c = a == 0.0 && b == 0.0 ? 0.0 : -(na * a + nb * b) / nd;
        h[0] = ax == 0 ? c : a;
        h[1] = ax == 1 ? c : (ax == 0 ? a : b);
        h[2] = ax == 2 ? c : b;
    };
    expand(kFduh, duh);
    expand(kFdwh, dwh);
    expand(kFbetah, bh);
    auto times = [](double s, double x) { return s == 0.0 ? 0.0 : s * x; };   // no crossing: 0 whatever the frame
    double su = 0.0, sv = 0.0;
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        if (out.p[c])
            out.p[c][i] = (float)(v[kFp + c] + times(v[kFbeta], nr[c]) - times(v[kFdu], tu[c]) - times(v[kFdw], tv[c]));
        if (out.p[3 + c]) out.p[3 + c][i] = (float)(v[kFtu + c] + duh[c]);
        if (out.p[6 + c]) out.p[6 + c][i] = (float)(v[kFtv + c] + dwh[c]);
        if (out.p[9 + c]) out.p[9 + c][i] = (float)(v[kFn + c] - bh[c]);
        su -= times(duh[c], tu[c]);
        sv -= times(dwh[c], tv[c]);
    }
    // through lambda_j A_j: dA/ds_u = A / s_u, dA/do as stored
    double lam = 0.0, o = v[kFo];
    if (lambda && v[kFpair] != 0.0) {
        const double A = (double)(float)bv.area[i], gA = v[kFpair] * lambda[i];
        lam = v[kFpair] * A;
        su += gA * A;
        sv += gA * A;
        o += gA * bv.dado[i];
    }
    if (out.p[12]) out.p[12][i] = (float)times(su, (double)r.a.w);
    if (out.p[13]) out.p[13][i] = (float)times(sv, (double)r.b.w);
    if (out.p[14]) out.p[14][i] = (float)o;
    if (out.p[15]) out.p[15][i] = (float)lam;
}

// ---------------------------------------------------------------------------
// geometry gradients through the ray-cast form factors (recorded hits)
// ---------------------------------------------------------------------------
// The compositing backward's dL/dalpha per recorded hit (as k_opacity_rec)
// chained to the hit surfel's centre, frame, scales and opacity and to the
// receiver's centre and frame (ray origin p_i, direction
// d = x t_u + y t_v + z n): alpha = 1 - e^(-c gamma), gamma = e^(-1.7 (u^2+w^2)),
// u = h . t_u / s_u, w = h . t_v / s_v, h = t d - q, q = p_k - p_i,
// t = (q . n_k)/(d . n_k).  The hit point is the FP64 intersection.  Sums in
// 64-bit fixed point with per-field scales from a first pass (bit-identical
// between runs), one copy per XCD; pass 1 lists a hit's ten contributions
// (hit_lists.h) and k_geometry_sum adds them: 107 M hits of a 30k-surfel bowl
// 33.6 ms with ten atomics a hit, 6.7 + 2.1 ms listed.

// zeroes a counter
__global__ void k_seg_reset(uint32_t *used) { used[threadIdx.x] = 0; }

template <int PASS, bool LISTED>
__global__ void __launch_bounds__(256) k_geometry_rec(BvhDev bv, int R, uint64_t seed, const uint2 *__restrict__ recs,
                                                      const uint32_t *__restrict__ rcnt, int rcap, int64_t s0, int64_t nblocks,
                                                      const int64_t *__restrict__ row_ptr,
                                                      const int32_t *__restrict__ col, const float *__restrict__ gF,
                                                      int max_row, uint32_t *maxbits, const int *fx,
                                                      unsigned long long *acc, int stride, HitLists lists) {
    extern __shared__ uint32_t sm4[];
    RowIndex row(sm4, max_row, bv.n);
    const int64_t b = s0 + xcd_block(blockIdx.x, nblocks) * stride;
    const int tid = threadIdx.x;
    const SurfRec ri = bv.rec[b];
    const uint32_t i = __float_as_uint(ri.d.w);
    const int64_t e0 = row_ptr[i];
    row.load(col + e0, gF + e0, (int)(row_ptr[i + 1] - e0), 1.0f / (float)R, tid, blockDim.x);
    FieldSink<PASS> sink;
    sink.init(acc, fx, bv.n);
    SharedSurfelAcc<12> accI;   // the receiver: p, t_u, t_v, n (fields 0-11)
    accI.zero();
    const int batches = (R + (int)blockDim.x - 1) / (int)blockDim.x;
    uint32_t *next = sm4 + row_index_bytes(max_row) / 4;
    for (int batch = 0; batch < batches; ++batch) {
        const int r = batch * (int)blockDim.x + tid;
        ListStretch list(lists, next, (int64_t)blockIdx.x * batches + batch);
        if (LISTED) {
            list.clear(tid, blockDim.x);
            __syncthreads();
        }
        uint32_t m = r < R ? rcnt[(int64_t)i * R + r] : 0u;
        if (m > (uint32_t)rcap) m = 0;
        const uint2 *in = recs + (int64_t)i * rcap * R + r;
        DF W{0.0f, 0.0f};
        float T = 1.0f;
        for (uint32_t q = 0; q < m; ++q) {
            const uint2 h = in[(int64_t)q * R];
            if (LISTED) list.count(h.x);
            const float gs = __uint_as_float(h.y);
            const float x = bv.c[h.x] * fabsf(gs);
            if (gs > 0.0f) {
                const float G = row.find(h.x);
                if (G != 0.0f) W = df_add(W, df_prod3(G, -expm1f(-x), T));
            }
            T = __fmul_rn(T, exp_fx(-x));
        }
        if (LISTED) list.open(tid, blockDim.x);
        if (W.hi == 0.0f) m = 0;
        float dx, dy, dz, sx, sy, sz;
        ray_direction(ri.c.x, ri.c.y, ri.c.z, ri.d.x, ri.d.y, ri.d.z, ri.b.x, ri.b.y, ri.b.z, (uint64_t)r,
                      (uint64_t)i, seed, 0, dx, dy, dz);
        ray_sample((uint64_t)r, (uint64_t)i, seed, 0, sx, sy, sz);
        float gd[3] = {0.0f, 0.0f, 0.0f}, gpi[3] = {0.0f, 0.0f, 0.0f};
        DF P{0.0f, 0.0f};
        T = 1.0f;
        for (uint32_t q = 0; q < m; ++q) {
            const uint2 h = in[(int64_t)q * R];
            const float gs = __uint_as_float(h.y);
            const float g = fabsf(gs);
            const uint32_t k = h.x;
            const float c = bv.c[k];
            const float x = c * g;
            const float f = exp_fx(-x);
            const float alpha = -expm1f(-x);
            const float G = gs > 0.0f ? row.find(k) : 0.0f;
            if (G != 0.0f) P = df_add(P, df_prod3(G, alpha, T));
            const DF Sd = df_add(W, DF{-P.hi, -P.lo});
            const float dLda = G * T - Sd.hi / f;
            T = __fmul_rn(T, f);
            if (dLda == 0.0f) continue;
            const float ok = bv.raw_op[k];
            float x10[10];
            x10[9] = ok > 0.0f && ok < kOpacityMax ? dLda * g * f / (1.0f - ok) : 0.0f;
            // the FP64 hit point of the FP32 ray on k's plane
            const SurfRec rk = bv.rec[bv.inv[k]];
            const double nx = rk.b.x, ny = rk.b.y, nz = rk.b.z;
            const double qx = (double)rk.a.x - ri.a.x, qy = (double)rk.a.y - ri.a.y, qz = (double)rk.a.z - ri.a.z;
            const double den = (double)dx * nx + (double)dy * ny + (double)dz * nz;
            const double tk = (qx * nx + qy * ny + qz * nz) / den;
            const float hx = (float)(tk * dx - qx), hy = (float)(tk * dy - qy), hz = (float)(tk * dz - qz);
            const float u = (hx * rk.c.x + hy * rk.c.y + hz * rk.c.z) * rk.a.w;
            const float w = (hx * rk.d.x + hy * rk.d.y + hz * rk.d.z) * rk.b.w;
            const float dLdg = dLda * c * f;
            const float du = dLdg * (-3.4f) * g * u * rk.a.w, dw = dLdg * (-3.4f) * g * w * rk.b.w;
            const float ghx = du * rk.c.x + dw * rk.d.x, ghy = du * rk.c.y + dw * rk.d.y, ghz = du * rk.c.z + dw * rk.d.z;
            const float beta = (ghx * dx + ghy * dy + ghz * dz) / (float)den;
            const float gqx = beta * rk.b.x - ghx, gqy = beta * rk.b.y - ghy, gqz = beta * rk.b.z - ghz;
            cross_terms(rk, du, dw, beta, hx, hy, hz, x10);
            if (LISTED && list.on) {
                float4 *e = reinterpret_cast<float4 *>(lists.entry) + 3 * (int64_t)list.place(k);
                e[0] = make_float4(x10[0], x10[1], x10[2], x10[3]);
                e[1] = make_float4(x10[4], x10[5], x10[6], x10[7]);
                e[2] = make_float4(x10[8], x10[9], __uint_as_float(k), 0.0f);
            } else {
#pragma unroll
                for (int z = 0; z < 10; ++z) sink.add(CrossTable<1>::field(z), k, x10[z]);
            }
            const float tf = (float)tk;
            gpi[0] -= gqx;
            gpi[1] -= gqy;
            gpi[2] -= gqz;
            gd[0] -= tf * gqx;
            gd[1] -= tf * gqy;
            gd[2] -= tf * gqz;
        }
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            accI.add<PASS>(sink, c, c, gpi[c]);
            accI.add<PASS>(sink, 3 + c, 3 + c, sx * gd[c]);
            accI.add<PASS>(sink, 6 + c, 6 + c, sy * gd[c]);
            accI.add<PASS>(sink, 9 + c, 9 + c, sz * gd[c]);
        }
        if (LISTED) list.close(tid, blockDim.x);
    }
    {
        const int fI[12] = {0, 1, 2, 3, 4, 5, 6, 7, 8, 9, 10, 11};
        accI.flush<PASS>(sink.acc, bv.n, i, fI);
    }
    sink.report(maxbits);
}

// The listed contributions of one chunk: workgroup (block of surfels, share of
// the stretches), 16 lanes per stretch; the ten sums of the block's surfels in
// LDS.
constexpr int kGeometryShift = 9;
constexpr int kGeometryEntry = 48;   // bytes
constexpr int kGeometryThreads = 512;
constexpr int kGeometryWgs = 1536;   // workgroups aimed at
// Blocks up to which the lists pay whatever the rays, and with 1 / 64 of a ray
// per block: 400k surfels (782 blocks), 16 / 128 rays each: a room 60 and 143 ms,
// added directly 79 and 449, a bowl 61 and 130, directly 73 and 344; 1 M, 16 / 32
// rays 196 and 228, directly 186 and 310; 260k, 4 / 16 rays 25 and 36, directly
// 23 and 53; 70k with 1, 2 and 4 rays 4.5, 5.3 and 6.1, directly 4.8, 5.6 and 6.4.
constexpr int64_t kGeometryAlways = 256, kGeometryBlocks = 2048;
constexpr double kGeometryShare = 1.0 / 64;

__global__ void __launch_bounds__(kGeometryThreads) k_geometry_sum(HitLists lists, int64_t stretches, int64_t n,
                                                                   uint32_t *maxbits, const int *fx,
                                                                   unsigned long long *acc) {
    constexpr int kPlaces = 1 << kGeometryShift;
    __shared__ unsigned long long table[10][kPlaces];
    const int tid = threadIdx.x;
    for (int z = tid; z < kPlaces; z += kGeometryThreads)
#pragma unroll
        for (int q = 0; q < 10; ++q) table[q][z] = 0;
    __syncthreads();
    FieldSink<1> sink;
    sink.init(acc, fx, n);
    const float4 *entry = reinterpret_cast<const float4 *>(lists.entry);
    const int block = blockIdx.x;
    constexpr int kRows = kGeometryThreads / 16;
    for (int64_t s = (int64_t)blockIdx.y * kRows + tid / 16; s < stretches; s += (int64_t)gridDim.y * kRows) {
        const uint2 p = lists.part[(s << lists.bits) + block];
        for (uint32_t k = p.x + (tid & 15); k < p.y; k += 16) {
            const float4 a = entry[3 * (int64_t)k], b = entry[3 * (int64_t)k + 1], c = entry[3 * (int64_t)k + 2];
            const uint32_t z = __float_as_uint(c.z) >> lists.bits;
            const float x[10] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w, c.x, c.y};
#pragma unroll
            for (int q = 0; q < 10; ++q) {
                const long long v = sink.scaled(CrossTable<1>::field(q), x[q]);
                if (v != 0) atomicAdd(&table[q][z], (unsigned long long)v);
            }
        }
    }
    __syncthreads();
    for (int z = tid; z < kPlaces; z += kGeometryThreads) {
        const int64_t j = ((int64_t)z << lists.bits) + block;
        if (j >= n) continue;
#pragma unroll
        for (int q = 0; q < 10; ++q)
            if (table[q][z] != 0) sink.add_scaled(CrossTable<1>::field(q), (uint32_t)j, (long long)table[q][z]);
    }
    sink.report(maxbits);
}

// ---------------------------------------------------------------------------
// direct-light gradients: light positions and intensities, albedo, surfel
// fields of the receivers and of the occluders on the shadow segments
// ---------------------------------------------------------------------------
// With v = x_l - p_i, r = |v|, ndot = n_i . v > 0,
// E_c = o a_c kappa I ndot T / r^3 (kappa = 2/sqrt(pi)),
// S = sum_c dL/dE_c a_c, Q = S o kappa I T:
//   dL/dI += S o kappa ndot T / r^3, dL/da_c += dL/dE_c o kappa I ndot T / r^3,
//   dL/do_i += S kappa I ndot T / r^3, g_v = Q (n/r^3 - 3 ndot v/r^5):
//   x_l += g_v, p_i -= g_v, n_i += Q v / r^3,
// and the shadow segment's occluders as for a centre-to-centre segment with
// W = S o kappa I ndot T / r^3.  The surfel fields are FieldSink's, the
// light's (x, y, z, I) have accumulators of their own; fixed point as above.
//
// Bound by the walks' latency and by the sums' atomics.  One lane per
// receiver that walked its lights in turn, twice in each of two passes, left
// most of the chip idle: 458 ms for 16k surfels x 100 lights.  Here
// k_light_walk walks every (receiver, light) segment once, 16 lanes to one,
// and keeps T and the positions of the surfels crossed (kSegHits places per
// lane and for the lanes with more a block of kSegMore from a pool); the two
// passes (largest contributions, then the sums) read those lists.  A segment
// crosses between none and some 130 surfels, so a workgroup's crossings are
// dealt out evenly to its lanes rather than each lane its own segment's.  Its
// segments start at neighbouring receivers in Morton order, end at one light
// and cross the same surfels (256 of them some 500, 27 a segment), so the sums
// are formed in a table in LDS first (CrossTable).  The lists hold one slice
// of the lights at a time (kSegLanes); more slices are walked once per pass.
constexpr int kLightFields = kFields + 4;
constexpr int kLightCrossings = 28;   // word of maxbits: crossings of pass 0 (64 bits)
constexpr uint32_t kSegAgain = 0xffffffffu;   // count of a lane whose list is not complete
constexpr int kSegHits = 64, kSegMore = 96, kSegShare = 8;   // a block for every eighth lane
constexpr int64_t kSegLanes = (int64_t)1 << 21;

// Lists of one slice: lane (light - first light) * pad + receiver slot
struct SegLists {
    float *T;          // [lanes] transmittance
    uint32_t *count;   // [lanes] surfels crossed
    uint32_t *hit;     // [lanes][kSegHits] their sorted positions
    uint32_t *block;   // [lanes] block of a lane with more than kSegHits
    uint32_t *more;    // [blocks][kSegMore]
    uint32_t *used;    // blocks given out (zeroed before each slice's walk)
    int64_t pad, lanes;
    uint32_t hits, blocks;   // kSegHits and lanes / kSegShare; without memory for lists 0, and every crossing is walked again
    static constexpr int64_t words_per_lane = 3 + kSegHits + kSegMore / kSegShare;
};

// The light's side of one (receiver, light): nothing to do where !on.
struct LightTerm {
    float dx, dy, dz, dd, ndot, len, S;
    bool on;
    __device__ __forceinline__ LightTerm(const SurfRec &rr, bool live, const float *lpos, int l, const float *ge,
                                         const float *a) {
        dx = __fsub_rn(lpos[3 * l + 0], rr.a.x);
        dy = __fsub_rn(lpos[3 * l + 1], rr.a.y);
        dz = __fsub_rn(lpos[3 * l + 2], rr.a.z);
        dd = __builtin_fmaf(dz, dz, __builtin_fmaf(dy, dy, __fmul_rn(dx, dx)));
        ndot = rr.b.x * dx + rr.b.y * dy + rr.b.z * dz;
        len = sqrt_rn(dd);
        S = live ? ge[0] * a[0] + ge[1] * a[1] + ge[2] * a[2] : 0.0f;
        on = live && ndot > 0.0f && dd > 0.0f && S != 0.0f;
    }
};

__global__ void __launch_bounds__(kRowThreads) k_light_walk(BvhDev bv, const float *__restrict__ albedo,
                                                            const float *__restrict__ lpos, int l0, int Lt, int K,
                                                            const float *__restrict__ gE, SegLists seg, int *err) {
    constexpr int kRows = kRowThreads / 16, kListed = kSegHits + kSegMore;
    __shared__ int32_t stack[kRows][kCrossNodes + kCrossLeaves];
    __shared__ uint32_t list[kRows][kListed], hits[kRows];
    const int row = threadIdx.x / 16, lane = threadIdx.x & 15;
    const int64_t slot = (int64_t)blockIdx.x * kRows + row;
    if (slot >= bv.n) return;
    const int l = l0 + (int)blockIdx.y;
    const int64_t at = (int64_t)blockIdx.y * seg.pad + slot;
    const SurfRec rr = bv.rec[slot];
    const uint32_t i = __float_as_uint(rr.d.w);
    const LightTerm t(rr, true, lpos, l, gE + (((int64_t)i * Lt + l) * K) * 3, albedo + 3 * (int64_t)i);
    float T = 1.0f;
    if (lane == 0) hits[row] = 0;
    __builtin_amdgcn_wave_barrier();
    if (t.on) {
        const Segment g{rr.a.x, rr.a.y, rr.a.z, t.dx, t.dy, t.dz, __fdiv_rn(bv.bounds[6], t.len), 1.0f};
        T = row_crossings(bv, g, i, i, stack[row], err, [&](int s) {
            const uint32_t h = atomicAdd(&hits[row], 1u);
            if (h < (uint32_t)kListed) list[row][h] = (uint32_t)s;
        });
    }
    __builtin_amdgcn_wave_barrier();
    uint32_t count = hits[row];
    for (uint32_t h = lane; h < min(count, seg.hits); h += 16) seg.hit[at * kSegHits + h] = list[row][h];
    if (count > seg.hits) {
        uint32_t block = kSegAgain;
        if (seg.blocks > 0 && count <= (uint32_t)kListed) {
            if (lane == 0) block = atomicAdd(seg.used, 1u);
            block = (uint32_t)__shfl((int)block, (int)__lane_id() & 48);
        }
        if (block >= seg.blocks) {
            count = kSegAgain;
        } else {
            for (uint32_t h = kSegHits + lane; h < count; h += 16)
                seg.more[(int64_t)block * kSegMore + (h - kSegHits)] = list[row][h];
            if (lane == 0) seg.block[at] = block;
        }
    }
    if (lane == 0) {
        seg.T[at] = T;
        seg.count[at] = count;
    }
}

constexpr int kTermThreads = 256;
constexpr int kLightSlots = 512;   // 43 KB

// A lane's terms of a light's fields: its segment's own, and the shares of the
// light's position of the crossings it takes.  Which lane takes a crossing
// depends on which lists found a block, so each share enters the fixed-point
// sum by itself: an FP32 sum of a lane's shares would round differently from
// run to run.
template <int PASS>
struct LightSum {
    float own[4], top[3];   // top: largest |share| (pass 0)
    long long q[3];         // the shares' sums (pass 1)
    __device__ __forceinline__ LightSum() : own{}, top{}, q{} {}
    __device__ __forceinline__ void share(const float (&ge)[3], const int *fx) {
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            if (PASS == 0) top[c] = fmaxf(top[c], fabsf(ge[c]));
            else q[c] += __float2ll_rn(ge[c] * __builtin_ldexpf(1.0f, fx[kFields + c]));
        }
    }
};

// The light's fields: largest |value| of the wave's lanes (pass 0), or one
// wave sum and one fixed-point add per field
template <int PASS>
__device__ __forceinline__ void add_light(const LightSum<PASS> &gl, uint32_t *maxbits, const int *fx,
                                          unsigned long long *lacc, int Lt, int l) {
    unsigned long long *lsum = lacc + (int64_t)xcc_id() * 4 * Lt;   // this XCD's light fields [4][Lt]
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        if (PASS == 0) {
            const float v = wave_max(fmaxf(fabsf(gl.own[q]), q < 3 ? gl.top[q < 3 ? q : 0] : 0.0f));
            if (__lane_id() == 0) raise(maxbits + kFields + q, v);
        } else {
            unsigned long long tot =
                (unsigned long long)__float2ll_rn(gl.own[q] * __builtin_ldexpf(1.0f, fx[kFields + q]));
            if (q < 3) tot += (unsigned long long)gl.q[q < 3 ? q : 0];
            for (int off = 32; off > 0; off >>= 1) tot += (unsigned long long)__shfl_xor((long long)tot, off, 64);
            if (__lane_id() == 0 && tot != 0)
                __hip_atomic_fetch_add(lsum + (int64_t)q * Lt + l, tot, __ATOMIC_RELAXED,
                                       __HIP_MEMORY_SCOPE_WORKGROUP);
        }
    }
}

// What a workgroup's segments share with the lanes that take their crossings
struct SegShared {
    float o[3][kTermThreads], d[3][kTermThreads], W[kTermThreads];
    uint32_t first[kTermThreads + 1];        // crossings of the segments before
    unsigned long long own[3][kTermThreads];   // the crossings' share of the receiver's centre, fixed point
};

template <int PASS>
__global__ void __launch_bounds__(kTermThreads) k_light_terms(BvhDev bv, const float *__restrict__ albedo,
                                                              const float *__restrict__ lpos,
                                                              const float *__restrict__ lI, int l0, int Lt, int K,
                                                              const float *__restrict__ gE, SegLists seg,
                                                              uint32_t *maxbits, const int *fx,
                                                              unsigned long long *acc, unsigned long long *lacc) {
    __shared__ CrossTable<PASS == 1 ? kLightSlots : 1> table;
    __shared__ SegShared sh;
    const int tid = threadIdx.x;
    const int64_t slot = (int64_t)blockIdx.x * kTermThreads + tid;
    const int l = l0 + (int)blockIdx.y;
    const int64_t at0 = (int64_t)blockIdx.y * seg.pad + (int64_t)blockIdx.x * kTermThreads;
    FieldSink<PASS> sink;
    sink.init(acc, fx, bv.n);
    const bool live = slot < bv.n;
    const SurfRec rr = bv.rec[live ? slot : 0];
    const uint32_t i = __float_as_uint(rr.d.w);
    const LightTerm t(rr, live, lpos, l, gE + (((int64_t)i * Lt + l) * K) * 3, albedo + 3 * (int64_t)i);
    if (PASS == 1) table.clear(tid, kTermThreads);
    LightSum<PASS> gl;
    uint32_t count = 0;
    sh.W[tid] = 0.0f;
    if (t.on) {
        const float T = seg.T[at0 + tid], oc = bv.op[i], oraw = bv.raw_op[i];
        count = seg.count[at0 + tid];
        if (count == kSegAgain) count = 0;   // k_light_again's
        const float r3 = t.dd * t.len, r5 = r3 * t.dd;
        const float kI = 1.1283791670955126f * lI[l];
        const float base = kI * t.ndot * T / r3;
        gl.own[3] = t.S * oc * 1.1283791670955126f * t.ndot * T / r3;
        if (oraw > 0.0f && oraw < kOpacityMax) sink.add(kFo, i, t.S * base);
        const float Q = t.S * oc * kI * T;
        gl.own[0] = Q * (rr.b.x / r3 - 3.0f * t.ndot * t.dx / r5);
        gl.own[1] = Q * (rr.b.y / r3 - 3.0f * t.ndot * t.dy / r5);
        gl.own[2] = Q * (rr.b.z / r3 - 3.0f * t.ndot * t.dz / r5);
        sink.add3(kFp, i, -gl.own[0], -gl.own[1], -gl.own[2]);
        sink.add3(kFn, i, Q * t.dx / r3, Q * t.dy / r3, Q * t.dz / r3);
        sh.W[tid] = t.S * oc * base;
    }
    sh.o[0][tid] = rr.a.x;
    sh.o[1][tid] = rr.a.y;
    sh.o[2][tid] = rr.a.z;
    sh.d[0][tid] = t.dx;
    sh.d[1][tid] = t.dy;
    sh.d[2][tid] = t.dz;
#pragma unroll
    for (int c = 0; c < 3; ++c) sh.own[c][tid] = 0;
    // exclusive sums of the counts
    uint32_t sum = count;
    for (int off = 1; off < 64; off <<= 1) {
        const uint32_t o = __shfl_up(sum, off, 64);
        if ((int)__lane_id() >= off) sum += o;
    }
    __shared__ uint32_t wave_total[kTermThreads / 64];
    if (__lane_id() == 63) wave_total[tid / 64] = sum;
    __syncthreads();
    uint32_t before = 0, total = 0;
#pragma unroll
    for (int w = 0; w < kTermThreads / 64; ++w) {
        if (w < tid / 64) before += wave_total[w];
        total += wave_total[w];
    }
    sh.first[tid] = before + sum - count;
    if (tid == 0) sh.first[kTermThreads] = total;
    __syncthreads();
    for (uint32_t e = tid; e < total; e += kTermThreads) {
        int g = 0;
#pragma unroll
        for (int step = kTermThreads / 2; step > 0; step >>= 1)
            if (sh.first[g + step] <= e) g += step;
        const uint32_t h = e - sh.first[g];
        const uint32_t s = h < (uint32_t)kSegHits
                               ? seg.hit[(at0 + g) * kSegHits + h]
                               : seg.more[(int64_t)seg.block[at0 + g] * kSegMore + (h - kSegHits)];
        const SurfRec r = bv.rec[s];
        float x[10], ge[3], gp[3];
        crossing(bv, r, sh.o[0][g], sh.o[1][g], sh.o[2][g], sh.d[0][g], sh.d[1][g], sh.d[2][g], sh.W[g], x, ge, gp);
        gl.share(ge, fx);
        if (PASS == 0) {
#pragma unroll
            for (int c = 0; c < 3; ++c) sink.add(kFp + c, 0, gp[c]);
#pragma unroll
            for (int q = 0; q < 10; ++q) sink.add(table.field(q), 0, x[q]);
        } else {
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                const long long v = sink.scaled(kFp + c, gp[c]);
                if (v != 0) atomicAdd(&sh.own[c][g], (unsigned long long)v);
            }
            table.add(sink, __float_as_uint(r.d.w), x);
        }
    }
    add_light<PASS>(gl, maxbits, fx, lacc, Lt, l);
    if (PASS == 0) {
        sink.report(maxbits);
        if (tid == 0 && total != 0)
            atomicAdd(reinterpret_cast<unsigned long long *>(maxbits + kLightCrossings), (unsigned long long)total);
    } else {
        __syncthreads();
#pragma unroll
        for (int c = 0; c < 3; ++c)
            if (live && sh.own[c][tid] != 0) sink.add_scaled(kFp + c, i, (long long)sh.own[c][tid]);
        table.flush(sink, tid, kTermThreads);
    }
}

// The crossings of the segments whose lists are not complete (kSegAgain),
// walked again, a lane each
template <int PASS>
__global__ void __launch_bounds__(kCenterThreads) k_light_again(BvhDev bv, const float *__restrict__ albedo,
                                                                const float *__restrict__ lpos,
                                                                const float *__restrict__ lI, int l0, int Lt, int K,
                                                                const float *__restrict__ gE, SegLists seg,
                                                                uint32_t *maxbits, const int *fx,
                                                                unsigned long long *acc, unsigned long long *lacc,
                                                                int *err) {
    extern __shared__ uint32_t stack_mem[];
    const int64_t slot = (int64_t)blockIdx.x * kCenterThreads + threadIdx.x;
    const int l = l0 + (int)blockIdx.y;
    const int64_t at = (int64_t)blockIdx.y * seg.pad + slot;
    const bool mine = slot < bv.n && seg.count[at] == kSegAgain;
    if (!__any(mine)) return;
    FieldSink<PASS> sink;
    sink.init(acc, fx, bv.n);
    LightSum<PASS> gl;
    unsigned long long hits = 0;
    if (mine) {
        const SurfRec rr = bv.rec[slot];
        const uint32_t i = __float_as_uint(rr.d.w);
        const LightTerm t(rr, true, lpos, l, gE + (((int64_t)i * Lt + l) * K) * 3, albedo + 3 * (int64_t)i);
        const float W = t.S * bv.op[i] * (1.1283791670955126f * lI[l] * t.ndot * seg.T[at] / (t.dd * t.len));
        trace_segment(bv, rr.a.x, rr.a.y, rr.a.z, t.dx, t.dy, t.dz, i, i, __fdiv_rn(bv.bounds[6], t.len),
                                 1.0f, stack_mem + threadIdx.x, kCenterThreads, err, [&](const SurfRec &r, int) {
                                     float x[10], ge[3], gp[3];
                                     crossing(bv, r, rr.a.x, rr.a.y, rr.a.z, t.dx, t.dy, t.dz, W, x, ge, gp);
                                     gl.share(ge, fx);
                                     ++hits;
                                     sink.add3(kFp, i, gp[0], gp[1], gp[2]);
#pragma unroll
                                     for (int q = 0; q < 10; ++q)
                                         sink.add(CrossTable<1>::field(q), __float_as_uint(r.d.w), x[q]);
                                 });
    }
    add_light<PASS>(gl, maxbits, fx, lacc, Lt, l);
    if (PASS == 0) {
        sink.report(maxbits);
        for (int off = 32; off > 0; off >>= 1) hits += __shfl_xor(hits, off, 64);
        if (__lane_id() == 0)
            atomicAdd(reinterpret_cast<unsigned long long *>(maxbits + kLightCrossings), hits);
    }
}

// dL/dalbedo of a slice's lights, in their order (added to the earlier
// slices' where l0 > 0)
__global__ void __launch_bounds__(256) k_light_albedo(BvhDev bv, const float *__restrict__ albedo,
                                                      const float *__restrict__ lpos, const float *__restrict__ lI,
                                                      int l0, int l1, int Lt, int K, const float *__restrict__ gE,
                                                      SegLists seg, float *__restrict__ g_alb) {
    const int64_t slot = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (slot >= bv.n) return;
    const SurfRec rr = bv.rec[slot];
    const int64_t i = (int64_t)__float_as_uint(rr.d.w);
    const float oc = bv.op[i];
    float ga[3] = {0.0f, 0.0f, 0.0f};
    if (l0 > 0)
        for (int c = 0; c < 3; ++c) ga[c] = g_alb[3 * i + c];
    for (int l = l0; l < l1; ++l) {
        const float *ge = gE + ((i * Lt + l) * K) * 3;
        const LightTerm t(rr, true, lpos, l, ge, albedo + 3 * i);
        if (!t.on) continue;
        const float base = 1.1283791670955126f * lI[l] * t.ndot * seg.T[(int64_t)(l - l0) * seg.pad + slot] /
                           (t.dd * t.len);
        for (int c = 0; c < 3; ++c) ga[c] += ge[c] * oc * base;
    }
    for (int c = 0; c < 3; ++c) g_alb[3 * i + c] = ga[c];
}

__global__ void k_light_exp(const uint32_t *maxbits, int64_t count_surfel, int64_t count_light, int *fx) {
    const int f = threadIdx.x;
    if (f >= kLightFields) return;
    // (a crossing adds to its light's position once)
    count_light += 2 * (int64_t)*reinterpret_cast<const unsigned long long *>(maxbits + kLightCrossings);
    const float m = __uint_as_float(maxbits[f]);
    int e = 0;
    if (!(m <= 3.0e38f)) {
        e = kFxNonFinite;
    } else if (m > 0.0f) {
        int ex;
        (void)frexpf(m * (float)(f < kFields ? count_surfel : count_light), &ex);
        e = min(120, max(-120, 62 - ex));
    }
    fx[f] = e;
}

__global__ void k_light_finish(const unsigned long long *__restrict__ lacc, const int *fx, int Lt, float *g_lpos,
                               float *g_lI) {
    const int t = threadIdx.x + blockIdx.x * blockDim.x;
    if (t >= 4 * Lt) return;
    const int q = t / Lt, l = t % Lt;
    unsigned long long s = 0;
    for (int x = 0; x < 8; ++x) s += lacc[((int64_t)x * 4 + q) * Lt + l];
    const int e = fx[kFields + q];
    const float v = e == kFxNonFinite ? __builtin_nanf("") : __builtin_ldexpf(__ll2float_rn((long long)s), -e);
    if (q < 3) {
        if (g_lpos) g_lpos[3 * l + q] = v;
    } else if (g_lI) {
        g_lI[l] = v;
    }
}

}  // namespace

// ---------------------------------------------------------------------------
// host launchers
// ---------------------------------------------------------------------------
gsrad_status launch_ff_center(const BvhDev &bv, const Csr &P, const float *lambda, float *val, int *err,
                              hipStream_t st) {
    if (P.n == 0) return GSRAD_OK;
    each_launch(P.n, kRowThreads, [&](int64_t first, unsigned blocks) {
        hipLaunchKernelGGL(k_ff_center, dim3(blocks), dim3(kRowThreads), 0, st, bv, P.row_ptr, P.col, P.n, lambda, val,
                           first, P.n, P.order, err);
    });
    return check_hip(hipGetLastError(), "centre-to-centre form factor launch");
}


// The fixed-point exponents come from the largest contributions on every
// kScaleStride-th row, with 2^kScaleMargin headroom; the accumulating pass
// records the true maxima, and where one could overflow its field's sums the
// pass runs again with the exact exponents (the host reads one flag).
constexpr int kScaleStride = 64;
constexpr int kScaleMargin = 12;

size_t geometry_list_bytes(int64_t n, int R) {
    const int threads = R >= 256 ? 256 : ((R + 63) / 64) * 64;
    const bool pay = lists_pay(n, R, kGeometryShift, kGeometryAlways, 0.0) ||
                     lists_pay(n, R, kGeometryShift, kGeometryBlocks, kGeometryShare);
    return pay ? (size_t)ListLayout(n, R, threads, kGeometryShift, kGeometryEntry).bytes : 0;
}

size_t center_group_bytes() { return (size_t)kRowParts * kRowPart * sizeof(uint2); }
size_t center_list_bytes(int64_t n) { return (size_t)std::min(n, kCenterGroups) * center_group_bytes(); }

size_t center_acc_bytes(int64_t n) { return (size_t)8 * kFields * n * 8 + 512; }

// accumulator layout: [8 XCD copies][kFields][n] u64, then maxbits[kFields],
// fx[kFields], the largest scaled contribution of the accumulating pass (as
// float bits) at maxbits[2 kFields], its crossings at maxbits[kCrossings]
static gsrad_status center_scaled_passes(int64_t n, int64_t count, void *acc, hipStream_t st,
                                         const std::function<void(int pass, int stride)> &run) {
    unsigned long long *a = static_cast<unsigned long long *>(acc);
    uint32_t *maxbits = reinterpret_cast<uint32_t *>(a + (size_t)8 * kFields * n);
    int *fx = reinterpret_cast<int *>(maxbits + kFields);
    run(0, kScaleStride);
    hipLaunchKernelGGL(k_fields_exp, dim3(1), dim3(64), 0, st, maxbits, count, kScaleMargin, fx);
    run(1, 1);
    uint32_t words[kCrossings + 2 - 2 * kFields];
    gsrad_status e = check_hip(hipMemcpyAsync(words, maxbits + 2 * kFields, sizeof(words), hipMemcpyDeviceToHost, st),
                               "scale check copy");
    if (e != GSRAD_OK) return e;
    if ((e = check_hip(hipStreamSynchronize(st), "scale check sync")) != GSRAD_OK) return e;
    // every |scaled contribution| times the count below 2^62: no sum overflows
    const double qmax = (double)reinterpret_cast<const float &>(words[0]);
    uint64_t crossings;
    memcpy(&crossings, words + (kCrossings - 2 * kFields), 8);
    count += (int64_t)crossings;   // a crossing adds to its segment's ends once
    if (!(qmax * (double)count < 4.6e18)) {
        // the sampled rows missed the largest contributions: exact maxima from
        // every row, then the sums again
        if ((e = check_hip(hipMemsetAsync(a, 0, center_acc_bytes(n), st), "accumulators zero")) != GSRAD_OK) return e;
        run(0, 1);
        hipLaunchKernelGGL(k_fields_exp, dim3(1), dim3(64), 0, st, maxbits, count, 0, fx);
        run(1, 1);
    }
    return check_hip(hipGetLastError(), "scaled passes");
}

gsrad_status launch_center_backward(const BvhDev &bv, const Csr &F, const float *lambda, const float *gF, void *acc,
                                    int32_t *done, void *lists, size_t list_bytes, const CenterOutputs &out, int *err,
                                    hipStream_t st) {
    if (F.n == 0) return GSRAD_OK;
    unsigned long long *a = static_cast<unsigned long long *>(acc);
    uint32_t *maxbits = reinterpret_cast<uint32_t *>(a + (size_t)8 * kFields * F.n);
    int *fx = reinterpret_cast<int *>(maxbits + kFields);
    static bool attr_set = false;
    if (!attr_set) {
        for (const void *fn : {reinterpret_cast<const void *>(&k_center_rows<0>),
                               reinterpret_cast<const void *>(&k_center_rows<1>)})
            (void)hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)sizeof(RowShared));
        attr_set = true;
    }
    const size_t smem = kWalkBytes;
    // as many workgroups as have lists; with none, every row is k_center_bwd's
    const int64_t groups = std::min(std::min(F.n, kCenterGroups), (int64_t)(list_bytes / center_group_bytes()));
    if (groups == 0) {
        const gsrad_status e = check_hip(hipMemsetAsync(done, 0, (size_t)F.n * 4, st), "rows zero");
        if (e != GSRAD_OK) return e;
    }
    auto run = [&](int pass, int stride) {
        const int64_t rows = (F.n + stride - 1) / stride;
        const int64_t nb = (rows + 1) / 2;
        const unsigned grid = (unsigned)std::min(rows, groups);
        uint2 *lp = static_cast<uint2 *>(lists);
        if (pass == 0) {
            if (groups > 0)
                hipLaunchKernelGGL(k_center_rows<0>, dim3(grid), dim3(kCenterRowThreads), sizeof(RowShared), st, bv,
                                   F.row_ptr, F.col, F.val, F.n, lambda, gF, maxbits, fx, a, F.order, stride, lp, done,
                                   err);
            hipLaunchKernelGGL(k_center_bwd<0>, dim3((unsigned)nb), dim3(kCenterThreads), smem, st, bv, F.row_ptr,
                               F.col, F.val, F.n, lambda, gF, maxbits, fx, a, nb, F.order, stride, done, err);
        } else {
            if (groups > 0)
                hipLaunchKernelGGL(k_center_rows<1>, dim3(grid), dim3(kCenterRowThreads), sizeof(RowShared), st, bv,
                                   F.row_ptr, F.col, F.val, F.n, lambda, gF, maxbits, fx, a, F.order, stride, lp, done,
                                   err);
            hipLaunchKernelGGL(k_center_bwd<1>, dim3((unsigned)nb), dim3(kCenterThreads), smem, st, bv, F.row_ptr,
                               F.col, F.val, F.n, lambda, gF, maxbits, fx, a, nb, F.order, stride, done, err);
        }
    };
    gsrad_status e = center_scaled_passes(F.n, 2 * F.nnz + 2, acc, st, run);
    if (e != GSRAD_OK) return e;
    hipLaunchKernelGGL(k_fields_finish, dim3((unsigned)((F.n + 255) / 256)), dim3(256), 0, st, bv, a, fx, lambda, out);
    return check_hip(hipGetLastError(), "centre-to-centre backward launch");
}

gsrad_status launch_geometry_rec(const BvhDev &bv, int R, uint64_t seed, const uint2 *recs, const uint32_t *rcnt,
                                 int rcap, const int64_t *row_ptr, const int32_t *col, const float *gF, int max_row,
                                 void *acc, void *ws, const CenterOutputs &out, hipStream_t st) {
    const int threads = R >= 256 ? 256 : ((R + 63) / 64) * 64;
    const size_t smem = row_index_bytes(max_row);
    if (max_row > kRowIndexMax) {
        set_error("geometry backward: row of %d entries is too long for the LDS row table", max_row);
        return GSRAD_EINVAL;
    }
    static bool attr_set = false;
    if (!attr_set) {
        for (const void *fn : {reinterpret_cast<const void *>(&k_geometry_rec<0, false>),
                               reinterpret_cast<const void *>(&k_geometry_rec<1, false>),
                               reinterpret_cast<const void *>(&k_geometry_rec<1, true>)})
            (void)hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024 - 4096);
        attr_set = true;
    }
    unsigned long long *a = static_cast<unsigned long long *>(acc);
    uint32_t *maxbits = reinterpret_cast<uint32_t *>(a + (size_t)8 * kFields * bv.n);
    int *fx = reinterpret_cast<int *>(maxbits + kFields);
    const int64_t batches = (R + threads - 1) / threads;
    const ListLayout lay(bv.n, R, threads, kGeometryShift, kGeometryEntry);
    const HitLists none{}, lists = ws ? lay.view(ws) : none;
    auto run = [&](int pass, int stride) {
        if (pass == 0) {
            const int64_t nb = (bv.n + stride - 1) / stride;
            hipLaunchKernelGGL((k_geometry_rec<0, false>), dim3((unsigned)nb), dim3(threads), smem, st, bv, R, seed, recs, rcnt,
                               rcap, (int64_t)0, nb, row_ptr, col, gF, max_row, maxbits, fx, a, stride, none);
            return;
        }
        const int64_t chunk = ws ? lay.stretches / batches : bv.n;
        for (int64_t s0 = 0; s0 < bv.n; s0 += chunk) {
            const int64_t m = std::min(chunk, bv.n - s0);
            if (ws) hipLaunchKernelGGL(k_seg_reset, dim3(1), dim3(2), 0, st, reinterpret_cast<uint32_t *>(lists.used));
            const auto kernel = ws ? k_geometry_rec<1, true> : k_geometry_rec<1, false>;
            hipLaunchKernelGGL(kernel, dim3((unsigned)m), dim3(threads),
                               smem + (ws ? (size_t)lists.blocks() * 4 : 0), st, bv, R, seed, recs, rcnt, rcap, s0, m,
                               row_ptr, col, gF, max_row, maxbits, fx, a, 1, lists);
            if (ws) {
                const int64_t rows = (m * batches + kGeometryThreads / 16 - 1) / (kGeometryThreads / 16);
                const unsigned split =
                    (unsigned)std::max<int64_t>(1, std::min<int64_t>(rows, kGeometryWgs / lists.blocks()));
                hipLaunchKernelGGL(k_geometry_sum, dim3((unsigned)lists.blocks(), split), dim3(kGeometryThreads), 0, st,
                                   lists, m * batches, bv.n, maxbits, fx, a);
            }
        }
    };
    gsrad_status e = center_scaled_passes(bv.n, bv.n * (int64_t)R + bv.n, acc, st, run);
    if (e != GSRAD_OK) return e;
    CenterOutputs o15 = out;
    o15.p[15] = nullptr;
    hipLaunchKernelGGL(k_fields_finish, dim3((unsigned)((bv.n + 255) / 256)), dim3(256), 0, st, bv, a, fx, nullptr,
                       o15);
    return check_hip(hipGetLastError(), "geometry backward launch");
}

// receivers padded to the workgroups of k_light_terms, lights of a slice
static int64_t light_pad(int64_t n) { return (n + kTermThreads - 1) / kTermThreads * kTermThreads; }
static int light_slice(int64_t n, int Lt) {
    return (int)std::min<int64_t>({(int64_t)Lt, 32768, std::max<int64_t>(1, kSegLanes / light_pad(n))});
}

// [8 XCD copies][kFields][n] u64, the lights' [8][4][Lt] u64, maxbits[32],
// fx[32]; behind them a light's T, counts and blocks, for where there is no
// memory for its lists
static size_t light_sum_bytes(int64_t n, int Lt) { return (size_t)8 * kFields * n * 8 + (size_t)8 * 4 * Lt * 8 + 256; }
size_t light_acc_bytes(int64_t n, int Lt) { return light_sum_bytes(n, Lt) + (size_t)light_pad(n) * 12; }
size_t light_one_bytes(int64_t n) { return (size_t)light_pad(n) * SegLists::words_per_lane * 4; }
size_t light_list_bytes(int64_t n, int Lt) { return (size_t)light_slice(n, Lt) * light_one_bytes(n); }

gsrad_status launch_direct_backward(const BvhDev &bv, const float *albedo, const float *lpos, const float *lI, int Lt,
                                    int K, const float *gE, void *acc, void *lists, size_t list_bytes, float *g_lpos,
                                    float *g_lI, float *g_alb, const CenterOutputs &out, int *err, hipStream_t st) {
    static_assert(kLightFields <= kLightCrossings && kLightCrossings % 2 == 0,
                  "maxbits and fx hold 32 entries each; crossings are counted at kLightCrossings, blocks in the last");
    unsigned long long *a = static_cast<unsigned long long *>(acc);
    unsigned long long *la = a + (size_t)8 * kFields * bv.n;
    uint32_t *maxbits = reinterpret_cast<uint32_t *>(la + (size_t)8 * 4 * Lt);
    int *fx = reinterpret_cast<int *>(maxbits + 32);
    // as many lights a slice as have lists
    const bool listed = list_bytes >= light_one_bytes(bv.n);
    const int slice =
        listed ? (int)std::min<int64_t>(light_slice(bv.n, Lt), (int64_t)(list_bytes / light_one_bytes(bv.n))) : 1;
    SegLists seg;
    seg.pad = light_pad(bv.n);
    seg.lanes = seg.pad * slice;
    seg.hits = listed ? kSegHits : 0;
    seg.blocks = listed ? (uint32_t)(seg.lanes / kSegShare) : 0;
    seg.T = listed ? static_cast<float *>(lists) : reinterpret_cast<float *>(fx + 32);
    seg.count = reinterpret_cast<uint32_t *>(seg.T + seg.lanes);
    seg.block = seg.count + seg.lanes;
    seg.hit = seg.block + seg.lanes;
    seg.more = seg.hit + (int64_t)kSegHits * seg.lanes;
    seg.used = maxbits + 31;
    const unsigned gw = (unsigned)((bv.n + kCenterThreads - 1) / kCenterThreads), gt = (unsigned)(seg.pad / kTermThreads);
    auto walk = [&](int l0) {
        const int m = std::min(slice, Lt - l0);
        hipLaunchKernelGGL(k_seg_reset, dim3(1), dim3(1), 0, st, seg.used);
        hipLaunchKernelGGL(k_light_walk, dim3((unsigned)((bv.n + kRowThreads / 16 - 1) / (kRowThreads / 16)), (unsigned)m),
                           dim3(kRowThreads), 0, st, bv, albedo, lpos, l0, Lt, K, gE, seg, err);
        return m;
    };
    for (int l0 = 0; l0 < Lt; l0 += slice) {
        const int m = walk(l0);
        if (g_alb)
            hipLaunchKernelGGL(k_light_albedo, dim3((unsigned)((bv.n + 255) / 256)), dim3(256), 0, st, bv, albedo, lpos,
                               lI, l0, l0 + m, Lt, K, gE, seg, g_alb);
        hipLaunchKernelGGL(k_light_terms<0>, dim3(gt, (unsigned)m), dim3(kTermThreads), 0, st, bv, albedo, lpos, lI, l0,
                           Lt, K, gE, seg, maxbits, fx, a, la);
        hipLaunchKernelGGL(k_light_again<0>, dim3(gw, (unsigned)m), dim3(kCenterThreads), kWalkBytes, st,
                           bv, albedo, lpos, lI, l0, Lt, K, gE, seg, maxbits, fx, a, la, err);
    }
    hipLaunchKernelGGL(k_light_exp, dim3(1), dim3(64), 0, st, maxbits,
                       2 * (bv.n * (int64_t)Lt + bv.n), 2 * seg.pad, fx);
    for (int l0 = 0; l0 < Lt; l0 += slice) {
        const int m = slice < Lt ? walk(l0) : Lt;
        hipLaunchKernelGGL(k_light_terms<1>, dim3(gt, (unsigned)m), dim3(kTermThreads), 0, st, bv, albedo, lpos, lI, l0,
                           Lt, K, gE, seg, maxbits, fx, a, la);
        hipLaunchKernelGGL(k_light_again<1>, dim3(gw, (unsigned)m), dim3(kCenterThreads), kWalkBytes, st,
                           bv, albedo, lpos, lI, l0, Lt, K, gE, seg, maxbits, fx, a, la, err);
    }
    CenterOutputs o15 = out;
    o15.p[15] = nullptr;
    hipLaunchKernelGGL(k_fields_finish, dim3((unsigned)((bv.n + 255) / 256)), dim3(256), 0, st, bv, a, fx, nullptr,
                       o15);
    hipLaunchKernelGGL(k_light_finish, dim3((unsigned)((4 * Lt + 63) / 64)), dim3(64), 0, st, la, fx, Lt, g_lpos, g_lI);
    return check_hip(hipGetLastError(), "direct light backward launch");
}

}  // namespace gsrad
