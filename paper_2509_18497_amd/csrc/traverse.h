// Device-side traversal helpers shared by the ray-cast, gradient and
// Monte-Carlo kernels: the k-buffer all-hit walk (trace_sorted), the segment
// walks (trace_segment by a lane, row_segment and row_crossings by 16), a row
// of dL/dF in LDS (RowIndex), the slot hash of surfel indices, and the
// double-float and fixed-point helpers of the deterministic gradient sums.
// Everything sits in an unnamed namespace: each kernel source gets its own
// inlined copy.
#pragma once

#include <utility>

#include "gsrad_internal.h"

namespace gsrad {

namespace {

// Traversal stack entries per lane of the walks over binary nodes: covers any
// LBVH of 30-bit Morton codes plus 32 index bits.
constexpr int kStackDeep = 64;
constexpr int kKB = 20;   // k-buffer entries per traversal round (measured best of 8-32)
constexpr uint32_t kEmpty = 0xffffffffu;

// Stack of the segment walks that take a lane each, kStackDeep entries: the
// first kWalkHead in LDS (column `lds`, entries `stride` apart), the deeper
// ones, which few walks reach (an LBVH of 100k surfels is some 20 levels high),
// in the lane's private memory.  The walks wait for dependent node and leaf
// loads, so waves in flight count: all 64 entries in LDS hold a CU to ten waves
// (10 M segments of a 20k-surfel bowl: F 29.6 ms, with a head of 20 24.2 ms).
constexpr int kWalkHead = 20;

template <int HEAD>
struct WalkStack {
    uint32_t *lds;
    int stride;
    uint32_t tail[kStackDeep - HEAD];
    __device__ __forceinline__ WalkStack(uint32_t *column, int stride_) : lds(column), stride(stride_) {}
    __device__ __forceinline__ void put(int k, uint32_t v) {
        if (k < HEAD) lds[k * stride] = v;
        else tail[k - HEAD] = v;
    }
    __device__ __forceinline__ uint32_t get(int k) const { return k < HEAD ? lds[k * stride] : tail[k - HEAD]; }
};
// all of it in LDS
template <>
struct WalkStack<kStackDeep> {
    uint32_t *lds;
    int stride;
    __device__ __forceinline__ WalkStack(uint32_t *column, int stride_) : lds(column), stride(stride_) {}
    __device__ __forceinline__ void put(int k, uint32_t v) { lds[k * stride] = v; }
    __device__ __forceinline__ uint32_t get(int k) const { return lds[k * stride]; }
};

// Workgroups are dispatched round-robin over the 8 XCDs; give each XCD a
// contiguous range of receivers so its L2 sees one region of the scene.
__device__ __forceinline__ int64_t xcd_block(int64_t b, int64_t g) {
    const int64_t x = b & 7, q = b >> 3, per = g >> 3, rem = g & 7;
    return x * per + (x < rem ? x : rem) + q;
}

// Keys (t bits, j) of the k-buffer.  t > 0 is a finite FP32 value, so the
// 64-bit key has a clear sign bit and an exponent field below all ones: read
// as an FP64 number it is a positive finite double, and positive finite
// doubles order exactly as their bit patterns.  The sorted insertion then
// takes one FP64 min and one max per entry instead of a 64-bit compare and
// four selects.  The empty entry is the largest finite double.
constexpr uint64_t kKeyEmpty = 0x7fefffffffffffffull;

__device__ __forceinline__ uint64_t key_bits(double k) { return (uint64_t)__double_as_longlong(k); }

// One step of the insertion: (a, x) <- (min(a, x), max(a, x)).  Written as
// the two VALU instructions: keys are never NaN, so the input quieting the
// compiler would add before an IEEE min/max is not needed.
__device__ __forceinline__ void key_insert_step(double &a, double &x) {
    double hi;
    asm volatile("v_max_f64 %1, %0, %2\n\tv_min_f64 %0, %0, %2" : "+v"(a), "=&v"(hi) : "v"(x));
    x = hi;
}

// Leaf visit of the sorted traversal: FP32 hit decision, then insertion
// into the ascending k-buffer of keys (t bits, j).  The kernel value and
// the face of a hit are found only for the hits that end up buffered.
template <int KB>
__device__ __forceinline__ void visit_leaf(const SurfRec *__restrict__ rec, int s, uint32_t self, float ox, float oy,
                                           float oz, float dx, float dy, float dz, float t_eps, uint64_t last,
                                           double (&key)[KB], int &found, float &t1) {
    const SurfRec r = rec[s];
    // all four 16-byte parts of the record are requested together: left to
    // itself the compiler loads the part holding j first and the rest only
    // after the self test, a second memory latency per leaf
    asm volatile("" : : "v"(r.a.x), "v"(r.b.x), "v"(r.c.x), "v"(r.d.w));
    const uint32_t j = __float_as_uint(r.d.w);
    if (j == self) return;
    float t, r2;
    bool front;
    if (!hit_test(r, ox, oy, oz, dx, dy, dz, t_eps, 0.0f, false, t, r2, front)) return;
    const uint64_t kk = ((uint64_t)__float_as_uint(t) << 32) | (uint64_t)j;
    if (kk <= last) return;
    ++found;
    if (kk >= key_bits(key[KB - 1])) return;
    double x = __longlong_as_double((long long)kk);
#pragma unroll
    for (int k = 0; k < KB; ++k) key_insert_step(key[k], x);
    if (found >= KB) t1 = __uint_as_float((uint32_t)(key_bits(key[KB - 1]) >> 32)) * 1.00001f + 1e-30f;
}

// All hits of one ray in (t, j) order, composited front to back until the
// transmittance drops below t_min; on_hit(j, alpha, T_before, front, gamma)
// is called for every composited hit (plus its depth t).  Returns the final
// transmittance.
template <int KB, int STK = kStackDeep, typename OnHit>
__device__ __forceinline__ float trace_sorted(const BvhDev &bv, float ox, float oy, float oz, float dx, float dy,
                                              float dz, uint32_t self, float t_eps, float t_min,
                                              uint32_t *stack, int stride, int *err, OnHit &&on_hit) {
    const float ix = safe_inv(dx), iy = safe_inv(dy), iz = safe_inv(dz);
    uint64_t last = 0;
    float T = 1.0f;
    for (;;) {
        double key[KB];
#pragma unroll
        for (int k = 0; k < KB; ++k) key[k] = __longlong_as_double((long long)kKeyEmpty);
        int found = 0;
        const float tlo = last ? __uint_as_float((uint32_t)(last >> 32)) : t_eps;
        const float t0 = tlo * 0.99999f;
        float t1 = INFINITY;
        if (bv.n == 1) {
            visit_leaf<KB>(bv.rec, 0, self, ox, oy, oz, dx, dy, dz, t_eps, last, key, found, t1);
        } else {
            int sp = 0, node = 0;
            bool ovf = false;
            for (;;) {
                const Node nd = bv.nodes[node];
                float tn0, tn1;
                bool h0 = slab(nd.b0.x, nd.b0.y, nd.b0.z, nd.b0.w, nd.b1.x, nd.b1.y, ox, oy, oz, ix, iy, iz, t0, t1, tn0);
                bool h1 = slab(nd.b1.z, nd.b1.w, nd.b2.x, nd.b2.y, nd.b2.z, nd.b2.w, ox, oy, oz, ix, iy, iz, t0, t1, tn1);
                const int c0 = nd.ch.x, c1 = nd.ch.y;
                if (h0 && c0 < 0) {
                    visit_leaf<KB>(bv.rec, ~c0, self, ox, oy, oz, dx, dy, dz, t_eps, last, key, found, t1);
                    h0 = false;
                }
                if (h1 && c1 < 0) {
                    visit_leaf<KB>(bv.rec, ~c1, self, ox, oy, oz, dx, dy, dz, t_eps, last, key, found, t1);
                    h1 = false;
                }
                // descend into the nearer hit child and push the other; with
                // no child left, pop.  A push past the stack's end ends the
                // walk with an error.
                const bool both = h0 && h1;
                const bool n0 = !h1 || (h0 && tn0 <= tn1);
                ovf = both && sp >= STK;
                if (both) stack[min(sp, STK - 1) * stride] = (uint32_t)(n0 ? c1 : c0);
                sp += both ? 1 : 0;
                node = n0 ? c0 : c1;
                if (!h0 && !h1) {
                    if (sp == 0) break;
                    --sp;
                    node = (int)stack[sp * stride];
                }
                if (ovf) break;
            }
            if (ovf) {
                atomicOr(err, kErrStack);
                return T;
            }
        }
        const int m = found < KB ? found : KB;
        // kernel values (FP64 hit point) and faces of the buffered hits only
        float gam[KB];
#pragma unroll
        for (int k = 0; k < KB; ++k) {
            gam[k] = 0.0f;
            if (k < m) {
                const SurfRec r = bv.rec[bv.inv[(uint32_t)key_bits(key[k])]];
                const float den = __builtin_fmaf(dz, r.b.z, __builtin_fmaf(dy, r.b.y, __fmul_rn(dx, r.b.x)));
                const float g = kernel_gamma(hit_r2_exact(r, ox, oy, oz, dx, dy, dz));
                gam[k] = den < 0.0f ? g : -g;
            }
        }
#pragma unroll
        for (int k = 0; k < KB; ++k) {
            if (k < m) {
                const uint32_t j = (uint32_t)key_bits(key[k]);
                const float g = fabsf(gam[k]);
                const bool front = gam[k] > 0.0f;
                const float x = __fmul_rn(bv.c[j], g);
                const float alpha = -expm1f(-x);
                on_hit(j, alpha, T, front, g, __uint_as_float((uint32_t)(key_bits(key[k]) >> 32)));
                T = __fmul_rn(T, exp_fx(-x));
                if (T < t_min) return T;
            }
        }
        // a full buffer pruned every box beyond its last entry, so more hits
        // may exist: only a buffer that did not fill ends the ray
        if (found < KB) return T;
        last = key_bits(key[KB - 1]);
    }
}

// Slot of surfel j in an open-addressing table of 2^log2h entries.  A full
// avalanche mixer (the 32-bit finaliser of "lowbias32"), not a single
// golden-ratio multiply: surfels laid out on Fibonacci lattices have index
// differences that are Fibonacci numbers, which golden-ratio hashing sends
// to nearly the same slot.
__device__ __forceinline__ uint32_t hash_slot(uint32_t j, int log2h) {
    uint32_t h = j;
    h ^= h >> 16;
    h *= 0x7feb352du;
    h ^= h >> 15;
    h *= 0x846ca68bu;
    h ^= h >> 16;
    return h >> (32 - log2h);
}

// Double-float pairs (error-free FP32 sums and products) and 64-bit
// fixed-point accumulation with atomics of workgroup scope (each XCD adds
// into its own copy of the accumulators, held in its L2).
struct DF {
    float hi, lo;
};

__device__ __forceinline__ DF df_add(DF x, DF y) {
    const float s = x.hi + y.hi;
    const float bb = s - x.hi;
    const float e = ((x.hi - (s - bb)) + (y.hi - bb)) + (x.lo + y.lo);
    const float hi = s + e;
    return {hi, e - (hi - s)};
}

// G * alpha * T as an unevaluated pair (relative error about 2^-46)
__device__ __forceinline__ DF df_prod3(float G, float a, float T) {
    const float p = a * T;
    const float pe = __builtin_fmaf(a, T, -p);
    const float h = G * p;
    return {h, __builtin_fmaf(G, p, -h) + G * pe};
}

__device__ __forceinline__ int xcc_id() {
    return __builtin_amdgcn_s_getreg((3 << 11) | (0 << 6) | 20) & 7;   // HW_REG_XCC_ID
}

__device__ __forceinline__ void fx_add(unsigned long long *acc, float v, float scale) {
    const long long q = __float2ll_rn(v * scale);
    if (q != 0)
        __hip_atomic_fetch_add(acc, (unsigned long long)q, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// Exponent marker of a non-finite upstream gradient: the fixed-point sums
// then yield NaN.
constexpr int kFxNonFinite = 1 << 20;

__device__ __forceinline__ uint32_t wave_incl_scan_u32(uint32_t v) {
    const int lane = __lane_id();
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const uint32_t u = __shfl_up(v, o, 64);
        if (lane >= o) v += u;
    }
    return v;
}

// A row of dL/dF in LDS: its columns (ascending), their values, and the first
// position of each of up to kRowBuckets ranges of columns (about two an entry),
// from which find() searches on.  An open-addressing table needs twice the row,
// rounded up to a power of two: the rows of a 16k-surfel room (2,544 entries, the
// longest 4,369) left a CU one workgroup of four waves, now four workgroups
// (opacity gradient 14.5 ms and 10.0 ms, each with direct adds).
constexpr int kRowBuckets = 512;
// bytes of LDS for rows of up to max_row entries
constexpr size_t row_index_bytes(int64_t max_row) { return (size_t)max_row * 8 + (kRowBuckets + 2) * 2; }
// longest row (start positions are 16 bits, and the LDS of a CU)
constexpr int kRowIndexMax = 8192;

struct RowIndex {
    uint32_t *col;
    float *val;
    uint16_t *start;
    int len, shift;
    __device__ __forceinline__ RowIndex(uint32_t *lds, int max_row, int64_t n)
        : col(lds), val(reinterpret_cast<float *>(lds + max_row)),
          start(reinterpret_cast<uint16_t *>(lds + 2 * max_row)), len(0), shift(0) {
        while (((n - 1) >> shift) >= kRowBuckets) ++shift;
    }
    // whole workgroup; ends with a barrier
    __device__ __forceinline__ void load(const int32_t *cols, const float *vals, int entries, float scale, int tid,
                                         int threads) {
        len = entries;
        int buckets = kRowBuckets;
        for (; buckets > 64 && buckets > 2 * len; buckets >>= 1) ++shift;
        for (int k = tid; k < len; k += threads) {
            col[k] = (uint32_t)cols[k];
            val[k] = vals[k] * scale;
        }
        __syncthreads();
        for (int q = tid; q <= buckets; q += threads) start[q] = (uint16_t)lower(0, len, (uint32_t)q << shift);
        __syncthreads();
    }
    __device__ __forceinline__ int lower(int lo, int hi, uint32_t j) const {
        while (lo < hi) {
            const int mid = (lo + hi) >> 1;
            if (col[mid] < j) lo = mid + 1;
            else hi = mid;
        }
        return lo;
    }
    // value of column j, 0 when absent
    __device__ __forceinline__ float find(uint32_t j) const {
        const uint32_t q = j >> shift;
        const int hi = start[q + 1], k = lower(start[q], hi, j);
        return k < hi && col[k] == j ? val[k] : 0.0f;
    }
};

// Every surfel other than skip_a and skip_b whose support the segment
// o + t d, t in (t_lo, t_hi), crosses (D_hit, both faces occlude);
// on_hit(record, sorted position) per crossing, in traversal order.
template <int HEAD = kWalkHead, typename OnHit>
__device__ __forceinline__ void trace_segment(const BvhDev &bv, float ox, float oy, float oz, float dx, float dy,
                                              float dz, uint32_t skip_a, uint32_t skip_b, float t_lo, float t_hi,
                                              uint32_t *column, int stride, int *err, OnHit &&on_hit) {
    const float ix = safe_inv(dx), iy = safe_inv(dy), iz = safe_inv(dz);
    const float t0 = t_lo * 0.99999f, t1 = t_hi * 1.00001f;
    auto leaf = [&](int s) {
        const SurfRec r = bv.rec[s];
        asm volatile("" : : "v"(r.a.x), "v"(r.b.x), "v"(r.c.x), "v"(r.d.w));   // whole record in one latency
        const uint32_t j = __float_as_uint(r.d.w);
        if (j == skip_a || j == skip_b) return;
        float t, r2;
        bool front;
        if (!hit_test(r, ox, oy, oz, dx, dy, dz, t_lo, t_hi, true, t, r2, front)) return;
        on_hit(r, s);
    };
    if (bv.n == 1) {
        leaf(0);
        return;
    }
    WalkStack<HEAD> stack(column, stride);
    int sp = 0, node = 0;
    bool ovf = false;
    for (;;) {
        const Node nd = bv.nodes[node];
        float tn0, tn1;
        bool h0 = slab(nd.b0.x, nd.b0.y, nd.b0.z, nd.b0.w, nd.b1.x, nd.b1.y, ox, oy, oz, ix, iy, iz, t0, t1, tn0);
        bool h1 = slab(nd.b1.z, nd.b1.w, nd.b2.x, nd.b2.y, nd.b2.z, nd.b2.w, ox, oy, oz, ix, iy, iz, t0, t1, tn1);
        const int c0 = nd.ch.x, c1 = nd.ch.y;
        if (h0 && c0 < 0) {
            leaf(~c0);
            h0 = false;
        }
        if (h1 && c1 < 0) {
            leaf(~c1);
            h1 = false;
        }
        // descend (first child first), push the other; none left: pop.  A
        // push past the stack's end ends the walk with an error.
        const bool both = h0 && h1;
        ovf = both && sp >= kStackDeep;
        if (both) stack.put(min(sp, kStackDeep - 1), (uint32_t)c1);
        sp += both ? 1 : 0;
        node = h0 ? c0 : c1;
        if (!h0 && !h1) {
            if (sp == 0) break;
            --sp;
            node = (int)stack.get(sp);
        }
        if (ovf) break;
    }
    if (ovf) atomicOr(err, kErrStack);
}

constexpr int kCenterThreads = 128;   // two rows (waves) per workgroup
constexpr size_t kWalkBytes = (size_t)kWalkHead * kCenterThreads * sizeof(uint32_t);   // LDS of its walks
constexpr float kInvPi = 0.318309886183790672f;

struct Segment {
    float ox, oy, oz, dx, dy, dz, t_lo, t_hi;
};

// The segment between the centres of ri and rj, its ends trimmed by t_eps
__device__ __forceinline__ Segment make_segment(const SurfRec &ri, const SurfRec &rj, float t_eps) {
    Segment g;
    g.ox = ri.a.x;
    g.oy = ri.a.y;
    g.oz = ri.a.z;
    g.dx = __fsub_rn(rj.a.x, ri.a.x);
    g.dy = __fsub_rn(rj.a.y, ri.a.y);
    g.dz = __fsub_rn(rj.a.z, ri.a.z);
    const float len = sqrt_rn(__builtin_fmaf(g.dz, g.dz, __builtin_fmaf(g.dy, g.dy, __fmul_rn(g.dx, g.dx))));
    g.t_lo = __fdiv_rn(t_eps, len);
    g.t_hi = __fsub_rn(1.0f, g.t_lo);
    return g;
}

// Lane N's value in every lane of its row of 16 lanes
template <int N>
__device__ __forceinline__ float row_bcast(float v) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x150 + N, 0xf, 0xf, true));
}
template <int... I, typename Fn>
__device__ __forceinline__ void each_lane(std::integer_sequence<int, I...>, float v, Fn &&fn) {
    (fn(I, row_bcast<I>(v)), ...);
}

// Transmittance of a segment by a row of 16 lanes, bit by bit as from
// trace_segment.  The row keeps the walk's stack in LDS, next entry on top: a
// node to open, a leaf to test, or the factor of a crossing found while nodes
// before it were still closed.  A round takes the top entries, one per lane,
// with one load for nodes and leaves alike (both are 64 bytes); what they leave
// goes back in their order, and the factors that have come to the top are
// multiplied in.  The loads that trace_segment waits for one by one are up to
// 16 at a time, and a wave waits for the longest of four segments, not of 64.
// 50k segments across a bowl of 50k surfels: 1.0 ms with a lane each (whether
// 64 or 16 of them share a wave), 0.24 ms with a row each (with
// WideNodes the same).
// A tree no higher than trace_segment takes never fills the stack: near its
// end a round opens one entry only, which needs kStackDeep more of them.
constexpr int kRowThreads = 256;   // 16 rows a workgroup
constexpr int kRowStack = 192;

__device__ __forceinline__ float row_segment(const BvhDev &bv, const Segment &g, uint32_t skip_a, uint32_t skip_b,
                                             uint64_t *stack, int *err) {
    constexpr auto kRow = std::make_integer_sequence<int, 16>{};
    constexpr uint32_t kNode = 0, kLeaf = 1, kFactor = 2;
    auto entry = [](uint32_t kind, uint32_t v) { return (uint64_t)kind << 32 | v; };
    auto child = [&](int c) { return c < 0 ? entry(kLeaf, (uint32_t)~c) : entry(kNode, (uint32_t)c); };
    const int l = threadIdx.x & 15, row = (int)__lane_id() & 48;
    const float ix = safe_inv(g.dx), iy = safe_inv(g.dy), iz = safe_inv(g.dz);
    const float t0 = g.t_lo * 0.99999f, t1 = g.t_hi * 1.00001f;
    float T = 1.0f;
    if (l == 0) stack[0] = entry(bv.n == 1 ? kLeaf : kNode, 0);
    int sp = 1;
    while (sp > 0) {
        const int m = sp + 16 <= kRowStack - kStackDeep ? min(sp, 16) : 1;
        if (sp >= kRowStack) {
            if (l == 0) atomicOr(err, kErrStack);
            break;
        }
        uint64_t e = entry(kFactor, __float_as_uint(1.0f));
        __builtin_amdgcn_wave_barrier();
        if (l < m) e = stack[sp - 1 - l];
        __builtin_amdgcn_wave_barrier();
        const uint32_t kind = (uint32_t)(e >> 32), v = (uint32_t)e;
        uint64_t keep0 = 0, keep1 = 0;   // what the entry leaves, keep0 first
        int keep = 0;
        float f = 1.0f;
        if (kind == kFactor) {
            f = __uint_as_float(v);
        } else {
            const float4 *q = kind == kNode ? reinterpret_cast<const float4 *>(bv.nodes + v)
                                            : reinterpret_cast<const float4 *>(bv.rec + v);
            const float4 q0 = q[0], q1 = q[1], q2 = q[2], q3 = q[3];
            if (kind == kNode) {
                float tn;
                const bool h0 = slab(q0.x, q0.y, q0.z, q0.w, q1.x, q1.y, g.ox, g.oy, g.oz, ix, iy, iz, t0, t1, tn);
                const bool h1 = slab(q1.z, q1.w, q2.x, q2.y, q2.z, q2.w, g.ox, g.oy, g.oz, ix, iy, iz, t0, t1, tn);
                const int c0 = __float_as_int(q3.x), c1 = __float_as_int(q3.y);
                const bool swap = c0 >= 0 && c1 < 0;   // a node's leaves come before its nodes
                keep = (h0 ? 1 : 0) + (h1 ? 1 : 0);
                keep0 = child(h0 && !(h1 && swap) ? c0 : c1);
                keep1 = child(swap ? c0 : c1);
            } else {
                SurfRec r;
                r.a = q0;
                r.b = q1;
                r.c = q2;
                r.d = q3;
                const uint32_t j = __float_as_uint(r.d.w);
                float t, r2;
                bool front;
                if (j != skip_a && j != skip_b &&
                    hit_test(r, g.ox, g.oy, g.oz, g.dx, g.dy, g.dz, g.t_lo, g.t_hi, true, t, r2, front))
                    f = transmit(r.c.w, kernel_gamma(hit_r2_exact(r, g.ox, g.oy, g.oz, g.dx, g.dy, g.dz)));
            }
        }
        // lanes before the row's first node: their factors are next in order
        const uint32_t nodes = (uint32_t)(__ballot(kind == kNode) >> row) & 0xffffu;
        const int first = nodes ? __ffs((int)nodes) - 1 : 16;
        if (kind != kNode && l >= first && __float_as_uint(f) != __float_as_uint(1.0f)) {
            keep = 1;
            keep0 = entry(kFactor, __float_as_uint(f));
        }
        each_lane(kRow, l < first ? f : 1.0f, [&](int, float x) { T = __fmul_rn(T, x); });
        const uint32_t k1 = (uint32_t)(__ballot(keep >= 1) >> row) & 0xffffu;
        const uint32_t k2 = (uint32_t)(__ballot(keep >= 2) >> row) & 0xffffu;
        int at = sp - m + __popc(k1 >> (l + 1)) + __popc(k2 >> (l + 1));
        if (keep >= 2) stack[at++] = keep1;
        if (keep >= 1) stack[at] = keep0;
        sp += __popc(k1) + __popc(k2) - m;
    }
    return T;
}

// The crossings of a segment by a row of 16 lanes, in no order: on_hit(sorted
// position) in the lane that finds one; returns the transmittance, e to the
// minus sum of c gamma.  The sum is in steps of 2^-40, so that it does not
// depend on the order (which the other rows of the wave have a part in).  Nodes
// are WideNodes; a round opens up to 16 nodes or tests up to 16 leaves, and the
// rows of a wave do the same kind, so that a wave does not step through both.
// Bound by the vector instructions of the tests: 10 M segments of a 20k-surfel bowl (200 binary nodes and 96 leaves
// each) 24.2 ms with a lane each, 19.4 ms with a row each taking nodes and
// leaves as they come, 17.5 ms with WideNodes, 14.6 ms with rounds of one kind.
// The stack never fills in a tree no higher than trace_segment takes: near its
// end a round opens fewer nodes, at last one, which needs kWideReserve more.
constexpr int kCrossNodes = 224, kCrossLeaves = 160;   // 1.5 KB a row
constexpr int kWideReserve = 96;                       // three a level of four grandchildren

template <typename OnHit>
__device__ __forceinline__ float row_crossings(const BvhDev &bv, const Segment &g, uint32_t skip_a, uint32_t skip_b,
                                               int32_t *nodes, int *err, OnHit &&on_hit) {
    int32_t *leaves = nodes + kCrossNodes;
    const int l = threadIdx.x & 15, row = (int)__lane_id() & 48;
    const float ix = wide_inv(g.dx), iy = wide_inv(g.dy), iz = wide_inv(g.dz);
    const float t0 = g.t_lo * 0.99999f, t1 = g.t_hi * 1.00001f;
    long long depth = 0;
    int sp = bv.n > 1 ? 1 : 0, nl = 1 - sp;
    if (l == 0) {
        nodes[0] = 0;
        leaves[0] = 0;
    }
    while (sp > 0 || nl > 0) {
        // (sp and nl are the row's; rows that are done take no part)
        const int rows = __popcll(__ballot(true)), want = __popcll(__ballot(nl >= 16 || sp == 0));
        __builtin_amdgcn_wave_barrier();
        if (2 * want >= rows || __any(nl > kCrossLeaves - 64)) {
            const int m = min(nl, 16);
            if (l < m) {
                const int s = leaves[nl - 1 - l];
                const SurfRec r = bv.rec[s];
                asm volatile("" : : "v"(r.a.x), "v"(r.b.x), "v"(r.c.x), "v"(r.d.w));   // whole record in one latency
                const uint32_t j = __float_as_uint(r.d.w);
                float t, r2;
                bool front;
                if (j != skip_a && j != skip_b &&
                    hit_test(r, g.ox, g.oy, g.oz, g.dx, g.dy, g.dz, g.t_lo, g.t_hi, true, t, r2, front)) {
                    const float x = __fmul_rn(r.c.w, kernel_gamma(hit_r2_exact(r, g.ox, g.oy, g.oz, g.dx, g.dy, g.dz)));
                    depth += __float2ll_rn(x * 0x1p40f);
                    on_hit(s);
                }
            }
            nl -= m;
        } else {
            if (sp > kCrossNodes - 4) {
                if (l == 0) atomicOr(err, kErrStack);
                break;
            }
            const int m = min(min(sp, 16), max(1, (kCrossNodes - kWideReserve - sp) / 3));
            int c[4] = {};
            bool h[4] = {};
            if (l < m) {
                const uint4 *q = reinterpret_cast<const uint4 *>(bv.wide + nodes[sp - 1 - l]);
                const float4 q0 = *reinterpret_cast<const float4 *>(q);
                const uint4 q1 = q[1], q2 = q[2];
                const int4 q3 = *reinterpret_cast<const int4 *>(q + 3);
                c[0] = q3.x;
                c[1] = q3.y;
                c[2] = q3.z;
                c[3] = q3.w;
                float tn[4];
                wide_slab(q0, q1, q2, q3, g.ox, g.oy, g.oz, ix, iy, iz, t0, t1, h, tn);
            }
            __builtin_amdgcn_wave_barrier();
            // (counts of the lanes before and of all, through the counts' bits)
            int cn = 0, cl = 0;
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                cn += h[k] && c[k] >= 0 ? 1 : 0;
                cl += h[k] && c[k] < 0 ? 1 : 0;
            }
            const uint32_t below = (1u << l) - 1u;
            int an = 0, al = 0, tn = 0, tl = 0;
#pragma unroll
            for (int b = 0; b < 3; ++b) {
                const uint32_t kn = (uint32_t)(__ballot((cn >> b) & 1) >> row) & 0xffffu;
                const uint32_t kl = (uint32_t)(__ballot((cl >> b) & 1) >> row) & 0xffffu;
                an += __popc(kn & below) << b;
                al += __popc(kl & below) << b;
                tn += __popc(kn) << b;
                tl += __popc(kl) << b;
            }
            an += sp - m;
            al += nl;
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                if (!h[k]) continue;
                if (c[k] >= 0) nodes[an++] = c[k];
                else leaves[al++] = ~c[k];
            }
            sp += tn - m;
            nl += tl;
        }
    }
#pragma unroll
    for (int off = 8; off > 0; off >>= 1) depth += __shfl_xor(depth, off);
    return exp_fx(-(__ll2float_rn(depth) * 0x1p-40f));
}

}  // namespace

}  // namespace gsrad
