// FP32 row products of the transport: B <- E + rho (F B), its adjoint on F^T
// and the sampled products lambda_i . B_j at F's entries.
//
// Rows of B, E and the gradients hold C = 3 M contiguous floats, M = Lt K
// RGB coefficients.  A lane owns one coefficient of a chunk (its three colours
// in one 12-byte load, so no lane masks a colour) and G lanes a gathered row:
// G = 1 for M = 1, 4 for M <= 4, else 16, more than 16 coefficients in chunks
// of equal width.  A wave owns an output row and reads its entries 64 at a
// time, one a lane; each of its 64 / G groups takes G of them, broadcast to
// its lanes by DPP, and the groups' sums are added at the end.  Shorter rows, and
// rows of chunks that a wave had better gather side by side, take 16 or 32 lanes
// (row_lanes_of); the sums are the same.
//
// What bounds them is where the gathered rows come from and how many gathers
// are in flight.  Measured on rows of 192 bytes: one instruction gathering
// four rows takes a CU some 18 cycles, 25 TB/s over the chip, while the rows
// come from the XCDs' L2, and 6.3 TB/s from the Infinity Cache; one row per
// instruction takes 7.8 cycles, 15 TB/s.  So an instruction gathers 64 / G
// rows, sixteen are in flight per lane with the next entries read ahead, and
// the order keeps the rows in L2: rows in the receivers' Morton order, each
// XCD a contiguous part, and the workgroups of one chunk of columns after the
// other (100 lights: 1/57 of a row is in use at a time).
//   16k-surfel room, 41.7 M entries, C = 27: bounce 0.87 -> 0.52 ms
//   100k bowl, 50.5 M entries, C = 48: bounce 0.81 -> 0.77 ms
// In L2 they run near its request rate (0.83 of one 64-byte request a cycle
// and channel at C = 540, 96 % hits); the 100k bowl's bounce misses on 39 % of
// its requests and runs at what the Infinity Cache gives.
// Launches per tile of senders that fits L2, the row's position kept between
// them, were slower (bowl: 1.27 ms a bounce with eight tiles): a row has too
// few entries in a tile to pay for its start.
#include <algorithm>
#include <type_traits>
#include <utility>

#include "gsrad_internal.h"
#include "rows.h"

namespace gsrad {

namespace {

constexpr int kThreads = 256;

__device__ __forceinline__ int64_t xcd_block(int64_t b, int64_t g) {
    const int64_t x = b & 7, q = b >> 3, per = g >> 3, rem = g & 7;
    return x * per + (x < rem ? x : rem) + q;
}

// three floats at any 4-byte alignment
struct __attribute__((packed, aligned(4))) F3 {
    float x, y, z;
};

// chunks of a row of M coefficients and their width
__host__ __device__ inline int row_chunks(int M, int g) { return (M + g - 1) / g; }
__host__ __device__ inline int row_width(int M, int g) {
    const int c = row_chunks(M, g);
    return (M + c - 1) / c;
}

// The coefficient that the lane of coefficient m reads: m, or past its chunk
// (from m0 on) or row the last one of these, whose line the chunk touches
// anyway.  (The row's first one was a line more for every entry of the later
// chunks: 20k surfels, 90 coefficients in six chunks of 15, a bounce 0.99 ms.)
__device__ __forceinline__ int near(int m0, int m, int M, int g) { return min(m, min(m0 + row_width(M, g), M) - 1); }

// Lane N's value in every lane of its row of 16 lanes, or of its quad
template <int CTRL>
__device__ __forceinline__ int dpp(int v) {
    return __builtin_amdgcn_update_dpp(0, v, CTRL, 0xf, 0xf, true);
}
template <int N, int W>
__device__ __forceinline__ int bcast(int v) {
    if constexpr (W == 16) return dpp<0x150 + N>(v);   // row_newbcast:N
    else return dpp<N * 0x55>(v);                      // quad_perm [N, N, N, N]
}
template <int... I, typename Fn>
__device__ __forceinline__ void unroll_seq(std::integer_sequence<int, I...>, Fn &&fn) {
    (fn(std::integral_constant<int, I>{}), ...);
}
// fn(integral_constant 0) ... fn(integral_constant N - 1)
template <int N, typename Fn>
__device__ __forceinline__ void unroll(Fn &&fn) {
    unroll_seq(std::make_integer_sequence<int, N>{}, fn);
}

// One entry a lane of the 64 entries from k on (the last one past e), of
// which the group takes the G at `off`
struct Entries {
    int j;
    float w;
    __device__ __forceinline__ void read(const int32_t *__restrict__ col, const float *__restrict__ val, int64_t k,
                                         int64_t e) {
        const int64_t q = min(k, e - 1);
        j = col[q];
        w = val[q];
    }
    template <int N, int G>
    __device__ __forceinline__ int column() const {
        if constexpr (G == 1) return j;
        else return bcast<N, G>(j);
    }
    template <int N, int G>
    __device__ __forceinline__ float weight() const {
        if constexpr (G == 1) return w;
        else return __int_as_float(bcast<N, G>(__float_as_int(w)));
    }
};

// acc += w_e * in[col_e] over the group's first m <= N entries
template <int G, int U0, int N, bool ALL>
__device__ __forceinline__ void take(const Entries &now, int m, const float *__restrict__ in, int C, float (&acc)[3]) {
    F3 x[N];
    unroll<N>([&](auto u) {
        const int j = now.column<U0 + u(), G>();
        x[u()] = *reinterpret_cast<const F3 *>(in + (int64_t)j * C);   // past m: the row's last entry
    });
    unroll<N>([&](auto u) {
        const float w = now.weight<U0 + u(), G>();
        if (ALL || U0 + u() < m) {
            acc[0] = __builtin_fmaf(w, x[u()].x, acc[0]);
            acc[1] = __builtin_fmaf(w, x[u()].y, acc[1]);
            acc[2] = __builtin_fmaf(w, x[u()].z, acc[2]);
        }
    });
}

// Ends one of several sums' part of a loop: left to itself the compiler issues
// all parts' loads first, in 230 registers
__device__ __forceinline__ void hold(float (&sum)[3]) {
    asm volatile("" : "+v"(sum[0]), "+v"(sum[1]), "+v"(sum[2]) : : "memory");
}

// Sum of v over the groups of a row's LPR lanes, in every lane
template <int G, int LPR>
__device__ __forceinline__ float over_groups(float v) {
#pragma unroll
    for (int o = G; o < LPR; o <<= 1) v += __shfl_xor(v, o, 64);
    return v;
}

struct RowArgs {
    const int64_t *row_ptr;
    const int32_t *col;
    const float *val;
    const int32_t *order;   // rows of a scene in the order they are taken, or NULL
    RowScene one;           // the scene, when tab is NULL
    const RowScene *tab;
    const int64_t *first;
    int count;
    int64_t block0;         // first workgroup of this launch
    const float *rho;
};

// The scene of this workgroup, and the workgroup's number in it
__device__ __forceinline__ int64_t find_scene(const RowArgs &a, RowScene &s) {
    const int64_t b = a.block0 + blockIdx.x;
    if (!a.tab) {
        s = a.one;
        return b;
    }
    int lo = 0, hi = a.count - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (a.first[mid] <= b) lo = mid;
        else hi = mid - 1;
    }
    s = a.tab[lo];
    return b - a.first[lo];
}

// The scene and the (chunk, row) of this lane; false past the scene's rows
template <int G, int LPR>
__device__ __forceinline__ bool find_row(const RowArgs &a, RowScene &s, int &m0, int64_t &row) {
    const int64_t b = find_scene(a, s);
    constexpr int R = kThreads / LPR;
    const int chunks = row_chunks(s.C / 3, G);
    // 16 lanes: a row's chunks side by side, together they gather whole rows;
    // more: one chunk of all rows after the other
    const int64_t items = s.n * chunks, per = (s.n + R - 1) / R;
    int chunk = 0;
    int64_t idx;
    if (LPR == 16) {
        idx = xcd_block(b, (items + R - 1) / R) * R + threadIdx.x / LPR;
        if (chunks > 1) {
            const int64_t item = idx;
            idx = items < (int64_t)1 << 32 ? (int64_t)((uint32_t)item / (uint32_t)chunks) : item / chunks;
            chunk = (int)(item - idx * chunks);
        }
    } else {
        if (chunks > 1) chunk = items < (int64_t)1 << 32 ? (int)((uint32_t)b / (uint32_t)per) : (int)(b / per);
        idx = xcd_block(b - (int64_t)chunk * per, per) * R + threadIdx.x / LPR;
    }
    m0 = chunk * row_width(s.C / 3, G);
    if (idx >= s.n) return false;
    row = a.order ? (int64_t)a.order[s.row0 + idx] : s.row0 + idx;
    return true;
}

// ADJ false: out = E + rho acc.  ADJ true: out = acc, p_out = rho acc,
// gE += acc (out, p_out where not NULL).  LPR lanes per row: 64, or with
// G = 16 also 32 or 16, which take the sums of two or four of the 64-entry
// reading's groups one after the other; the sums are the same.
template <int G, int LPR, bool ADJ>
__global__ void __launch_bounds__(kThreads) k_rows(RowArgs a, const float *__restrict__ in,
                                                   const float *__restrict__ E, float *__restrict__ out,
                                                   float *__restrict__ p_out, float *__restrict__ gE) {
    RowScene s;
    int m0;
    int64_t row;
    if (!find_row<G, LPR>(a, s, m0, row)) return;
    constexpr int A = 64 / LPR;   // groups of a reading that one group of lanes takes
    const int M = s.C / 3, l = threadIdx.x % G, m = m0 + l;
    const int sub = (threadIdx.x % LPR) / G;
    const bool on = l < row_width(M, G) && m < M;
    const int64_t b = a.row_ptr[row], e = a.row_ptr[row + 1];
    float acc[A][3];
#pragma unroll
    for (int q = 0; q < A; ++q) acc[q][0] = acc[q][1] = acc[q][2] = 0.0f;
    if (b < e) {
        const float *src = in + s.vbase - s.row0 * s.C + 3 * near(m0, m, M, G);
        Entries next[A];
        auto first_of = [&](int64_t k, int q) { return k + (q * (LPR / G) + sub) * G; };
#pragma unroll
        for (int q = 0; q < A; ++q) next[q].read(a.col, a.val, first_of(b, q) + l, e);
        int64_t k = b;
        for (; k + 64 <= e; k += 64) {
#pragma unroll
            for (int q = 0; q < A; ++q) {
                const Entries now = next[q];
                if (k + 64 < e) next[q].read(a.col, a.val, first_of(k + 64, q) + l, e);
                if constexpr (G == 16 && A == 4) {
                    take<G, 0, 8, true>(now, G, src, s.C, acc[q]);
                    hold(acc[q]);
                    take<G, 8, 8, true>(now, G, src, s.C, acc[q]);
                } else {
                    take<G, 0, G, true>(now, G, src, s.C, acc[q]);
                }
                if (A > 1) hold(acc[q]);
            }
        }
#pragma unroll
        for (int q = 0; q < A; ++q) {
            const int n = (int)max<int64_t>(0, min<int64_t>(G, e - first_of(k, q)));
            if constexpr (G == 16) {
                if constexpr (A == 4) {
                    if (n > 0) take<G, 0, 8, false>(next[q], n, src, s.C, acc[q]);
                    hold(acc[q]);
                    if (n > 8) take<G, 8, 8, false>(next[q], n, src, s.C, acc[q]);
                } else if (n > 8) {
                    take<G, 0, 16, false>(next[q], n, src, s.C, acc[q]);
                } else if (n > 0) {
                    take<G, 0, 8, false>(next[q], n, src, s.C, acc[q]);
                }
            } else if (n > 0) {
                take<G, 0, G, false>(next[q], n, src, s.C, acc[q]);
            }
            if (A > 1) hold(acc[q]);
        }
    }
    // the groups' sums in one order whatever LPR: pairs at distance one
    // group, then two, ...
    float t[3];
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        float x[A];
#pragma unroll
        for (int q = 0; q < A; ++q) x[q] = over_groups<G, LPR>(acc[q][c]);
        if constexpr (A == 1) t[c] = x[0];
        else if constexpr (A == 2) t[c] = x[0] + x[1];
        else t[c] = (x[0] + x[1]) + (x[2] + x[3]);
    }
    if (!on || sub != 0) return;
    const int64_t at = s.vbase + (row - s.row0) * s.C + 3 * m;
    const float r0 = a.rho[row * 3 + 0], r1 = a.rho[row * 3 + 1], r2 = a.rho[row * 3 + 2];
    if (ADJ) {
        if (out) *reinterpret_cast<F3 *>(out + at) = F3{t[0], t[1], t[2]};
        if (p_out) *reinterpret_cast<F3 *>(p_out + at) = F3{r0 * t[0], r1 * t[1], r2 * t[2]};
        const F3 g = *reinterpret_cast<const F3 *>(gE + at);
        *reinterpret_cast<F3 *>(gE + at) = F3{g.x + t[0], g.y + t[1], g.z + t[2]};
    } else {
        const F3 x = *reinterpret_cast<const F3 *>(E + at);
        *reinterpret_cast<F3 *>(out + at) = F3{__builtin_fmaf(r0, t[0], x.x), __builtin_fmaf(r1, t[1], x.y),
                                               __builtin_fmaf(r2, t[2], x.z)};
    }
}

// Sum over the G lanes of a group, in every lane (rotations within a row of
// 16 lanes, or a quad)
template <int G>
__device__ __forceinline__ float group_sum(float v) {
    auto add = [&](auto ctrl) { v += __int_as_float(dpp<decltype(ctrl)::value>(__float_as_int(v))); };
    if constexpr (G == 16) {
        add(std::integral_constant<int, 0x128>{});   // row_ror:8
        add(std::integral_constant<int, 0x124>{});   // row_ror:4
        add(std::integral_constant<int, 0x122>{});   // row_ror:2
        add(std::integral_constant<int, 0x121>{});   // row_ror:1
    } else if constexpr (G == 4) {
        add(std::integral_constant<int, 0x4e>{});   // quad_perm [2,3,0,1]
        add(std::integral_constant<int, 0xb1>{});   // quad_perm [1,0,3,2]
    }
    return v;
}

// For each stored entry e = (row, j), over NQ bounces and one chunk of columns
// or, with CP > 1, all of them, CP at a time side by side:
//   s_c = sum_k sum_{columns of colour c} lambda^(k+1)[row] B^(k)[j]
//   grad_F[e] (+)= sum_c rho[row, c] s_c;  grad_rho[row, c] (+)= sum_e F[e] s_c
// LPR lanes per row, the row's lambda in registers; a group gathers two of its
// entries' NQ rows at a time.  Both results are linear in the lanes' shares of
// s_c, so only the one value of dL/dF is summed over a group's lanes for each
// entry; dL/drho's three are summed over the row's lanes once per chunk.
template <int G, int LPR, int CP, int NQ>
__global__ void __launch_bounds__(kThreads) k_sddmm3(RowArgs a, int chunk, int64_t stride,
                                                     const float *__restrict__ Bt, const float *__restrict__ Lt,
                                                     float *__restrict__ grad_F, float *__restrict__ grad_rho,
                                                     bool fresh) {
    RowScene s;
    constexpr int R = kThreads / LPR;
    const int64_t block = find_scene(a, s);
    if (CP == 1 && chunk * row_width(s.C / 3, G) >= s.C / 3) return;
    const int64_t idx = xcd_block(block, (s.n + R - 1) / R) * R + threadIdx.x / LPR;
    if (idx >= s.n) return;
    const int64_t row = a.order ? (int64_t)a.order[s.row0 + idx] : s.row0 + idx;
    const int M = s.C / 3, width = row_width(M, G), l = threadIdx.x % G, lane = threadIdx.x % LPR;
    const int64_t b = a.row_ptr[row], e = a.row_ptr[row + 1];
    static_assert(CP == 1 || (G == 16 && LPR == 16 * CP), "a row of 16 lanes a chunk");
    constexpr int kRead = CP == 1 ? LPR : G;   // entries of a reading
    const int at_e = CP == 1 ? lane : l;       // this lane's
    auto one = [&](int m0, bool first) {
        const int m = m0 + l;
        const bool on = l < width && m < M;
        float gr[3] = {0.0f, 0.0f, 0.0f};
        if (b < e) {
            const float r[3] = {a.rho[row * 3 + 0], a.rho[row * 3 + 1], a.rho[row * 3 + 2]};
            float lam[NQ][3];
            const int64_t at = s.vbase + (row - s.row0) * s.C + 3 * near(m0, m, M, G);
#pragma unroll
            for (int q = 0; q < NQ; ++q) {
                const F3 x = *reinterpret_cast<const F3 *>(Lt + q * stride + at);
                lam[q][0] = x.x;
                lam[q][1] = x.y;
                lam[q][2] = x.z;
            }
            const float *base = Bt + s.vbase - s.row0 * s.C + 3 * near(m0, m, M, G);
            Entries next;
            next.read(a.col, a.val, b + at_e, e);
            for (int64_t k = b; k < e; k += kRead) {
                const Entries now = next;
                if (k + kRead < e) next.read(a.col, a.val, k + kRead + at_e, e);
                const int n = (int)max<int64_t>(0, min<int64_t>(G, e - (k + at_e - l)));
                float keep = 0.0f;   // dL/dF of the entry this lane read
                constexpr int P = G == 1 ? 1 : 2;
                unroll<G / P>([&](auto h) {
                    constexpr int u0 = h() * P;
                    if (u0 < n) {
                        F3 x[P][NQ];
                        unroll<P>([&](auto u) {
                            const float *src = base + (int64_t)now.column<u0 + u(), G>() * s.C;
#pragma unroll
                            for (int q = 0; q < NQ; ++q) x[u()][q] = *reinterpret_cast<const F3 *>(src + q * stride);
                        });
                        unroll<P>([&](auto u) {
                            float t[3] = {0.0f, 0.0f, 0.0f};
#pragma unroll
                            for (int q = 0; q < NQ; ++q) {
                                t[0] = __builtin_fmaf(lam[q][0], x[u()][q].x, t[0]);
                                t[1] = __builtin_fmaf(lam[q][1], x[u()][q].y, t[1]);
                                t[2] = __builtin_fmaf(lam[q][2], x[u()][q].z, t[2]);
                            }
                            float g = r[0] * t[0] + r[1] * t[1] + r[2] * t[2];
                            if (G > 1) g = group_sum<G>(on ? g : 0.0f);
                            const float f = now.weight<u0 + u(), G>();
                            if (l == u0 + u()) keep = g;
                            if (u0 + u() < n) {
#pragma unroll
                                for (int c = 0; c < 3; ++c) gr[c] = __builtin_fmaf(f, t[c], gr[c]);
                            }
                        });
                    }
                });
                if constexpr (CP > 1) keep = over_groups<16, LPR>(keep);
                if (grad_F && lane == at_e && k + at_e < e)
                    grad_F[k + at_e] = first ? keep : grad_F[k + at_e] + keep;
            }
        }
        if (!grad_rho) return;
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            const float t = over_groups<1, LPR>(on ? gr[c] : 0.0f);
            if (lane == 0) grad_rho[row * 3 + c] = first ? t : grad_rho[row * 3 + c] + t;
        }
    };
    if constexpr (CP == 1) {
        one(chunk * width, fresh);
    } else {
        for (int c = 0; c < row_chunks(M, G); c += CP) one((c + lane / 16) * width, fresh && c == 0);
    }
}

// The adjoint's start, a lane per coefficient: lam = gE = in (in may be gE),
// p = rho in
__device__ __forceinline__ void seed(int64_t row, int64_t at, const float *in, const float *__restrict__ rho,
                                     float *__restrict__ lam, float *gE, float *__restrict__ p) {
    const F3 x = *reinterpret_cast<const F3 *>(in + at);
    *reinterpret_cast<F3 *>(lam + at) = x;
    *reinterpret_cast<F3 *>(gE + at) = x;
    *reinterpret_cast<F3 *>(p + at) = F3{rho[row * 3] * x.x, rho[row * 3 + 1] * x.y, rho[row * 3 + 2] * x.z};
}

__global__ void __launch_bounds__(256) k_seed(int64_t lanes, int M, int64_t block0, const float *in,
                                              const float *__restrict__ rho, float *__restrict__ lam, float *gE,
                                              float *__restrict__ p) {
    const int64_t t = (block0 + blockIdx.x) * 256 + threadIdx.x;
    if (t < lanes) seed(t / M, 3 * t, in, rho, lam, gE, p);
}

// on all scenes of a batch (tab[count], in order)
__global__ void __launch_bounds__(256) k_seed_batch(const RowScene *__restrict__ tab, int count, int64_t lanes,
                                                    int64_t block0, const float *in, const float *__restrict__ rho,
                                                    float *__restrict__ lam, float *gE, float *__restrict__ p) {
    const int64_t t = (block0 + blockIdx.x) * 256 + threadIdx.x;
    if (t >= lanes) return;
    int lo = 0, hi = count - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (tab[mid].vbase <= 3 * t) lo = mid;
        else hi = mid - 1;
    }
    seed(tab[lo].row0 + (3 * t - tab[lo].vbase) / tab[lo].C, 3 * t, in, rho, lam, gE, p);
}

int row_lanes(int C) { return C == 3 ? 1 : C <= 12 ? 4 : 16; }

int64_t rows_blocks(int64_t n, int C, int lanes) {
    const int64_t r = kThreads / lanes, chunks = row_chunks(C / 3, row_lanes(C));
    return lanes == 16 ? (n * chunks + r - 1) / r : (n + r - 1) / r * chunks;
}

// Bounces per launch of the sampled products.  One launch of all takes the
// fewest instructions, but the chunk of all rows and bounces that it gathers
// from has to stay in the XCDs' L2: with two against eight per launch 100k
// rows of 192 bytes take 8.3 against 10.9 ms, 8k rows in 12 chunks 6.2
// against 10.1, while 8k rows of 108 bytes take 0.33 against 0.27 and 16k
// (four: 3.9) 4.5 against 3.9.  The line lies where these cross.
constexpr int64_t kSddmmBytes = (int64_t)7 << 20;
int sddmm_bounces(int64_t n, int width) {
    return (int)std::min<int64_t>(8, std::max<int64_t>(2, kSddmmBytes / (n * width * 12)));
}

RowArgs row_args(const Csr &F, const float *rho) {
    RowArgs a{};
    a.row_ptr = F.row_ptr;
    a.col = F.col;
    a.val = F.val;
    a.order = F.order;
    a.rho = rho;
    return a;
}

// Lanes per row of a scene's products.  64 where the mean row has more than
// kShortRow entries; a wave with a shorter row leaves lanes without an entry, so
// 16 (20k rows of 32 entries, 27 coefficients: bounce 20 -> 15 us), or 32 where
// 16 would fill less than two waves a SIMD.  The adjoint's rows, F's columns,
// vary more in length: 16 up to kShortColumn.
// Rows of several chunks: with 16 lanes a wave gathers four chunks of an entry
// side by side, with 64 all workgroups one chunk after the other.  The latter
// pays where the rows' one chunk fits an XCD's L2 and the whole rows do not (20k
// rows of 512 entries, 270 coefficients: 2.1 against 3.1 ms a bounce).  The
// former up to kWholeBytes and kWholeChunks (8k rows, 90 coefficients: 224 against
// 257 us; 540 coefficients: 2.6 against 1.4 ms), for two chunks further (100k
// rows of 17 coefficients, whose halves share their lines: 1.1 against 1.4 ms),
// and again where one chunk is past kChunkBytes (100k rows of 128 entries, 90
// coefficients: 1.8 against 2.1 ms; of 512 both 5.8).
constexpr int64_t kShortRow = 40, kShortColumn = 12, kManyItems = 8192;
constexpr int64_t kWholeBytes = (int64_t)18 << 20, kWholeBytesTwo = (int64_t)64 << 20, kChunkBytes = (int64_t)16 << 20;
constexpr int kWholeChunks = 12;
int row_lanes_of(const RowScene &s, bool adjoint) {
    const int64_t chunks = row_chunks(s.C / 3, row_lanes(s.C)), len = s.nnz / std::max<int64_t>(s.n, 1);
    const bool many = s.n * chunks >= kManyItems;
    if (adjoint && !many) return 64;
    if (chunks == 1) return len > (adjoint ? kShortColumn : kShortRow) ? 64 : many ? 16 : 32;
    if (len <= kShortRow) return many && chunks > kWholeChunks && len > 24 ? 32 : 16;
    const bool whole = many && chunks <= kWholeChunks && s.n * s.C * 4 <= (chunks == 2 ? kWholeBytesTwo : kWholeBytes);
    if (whole && (!adjoint || len <= 100)) return 16;
    return s.n * row_width(s.C / 3, row_lanes(s.C)) * 12 > kChunkBytes && len <= 256 ? 16 : 64;
}

template <bool ADJ>
gsrad_status run_rows(RowArgs a, int g, int lanes, int64_t blocks, const float *in, const float *E, float *out,
                      float *p_out, float *gE, hipStream_t st) {
    auto run = [&](auto kernel) {
        each_launch(blocks, kThreads, [&](int64_t first, unsigned groups) {
            a.block0 = first;
            hipLaunchKernelGGL(kernel, dim3(groups), dim3(kThreads), 0, st, a, in, E, out, p_out, gE);
        });
    };
    auto with = [&](auto width) {
        constexpr int G = decltype(width)::value;
        if (lanes == 16) run(k_rows<G, 16, ADJ>);
        else if (lanes == 32) run(k_rows<G, 32, ADJ>);
        else run(k_rows<G, 64, ADJ>);
    };
    if (g == 1) with(std::integral_constant<int, 1>{});
    else if (g == 4) with(std::integral_constant<int, 4>{});
    else with(std::integral_constant<int, 16>{});
    return check_hip(hipGetLastError(), ADJ ? "adjoint launch" : "bounce launch");
}

template <bool ADJ>
gsrad_status run_scene(const Csr &F, const RowScene &s, const float *in, const float *E, const float *rho, float *out,
                       float *p_out, float *gE, hipStream_t st) {
    if (s.n == 0) return GSRAD_OK;
    RowArgs a = row_args(F, rho);
    a.one = s;
    const int lanes = row_lanes_of(s, ADJ);
    return run_rows<ADJ>(a, row_lanes(s.C), lanes, rows_blocks(s.n, s.C, lanes), in, E, out, p_out, gE, st);
}

// The scenes of a batch: a launch for each G among them.
template <bool ADJ>
gsrad_status run_batch(const Csr &F, const RowTable &t, int lanes, const float *in, const float *E, const float *rho,
                       float *out, float *p_out, float *gE, hipStream_t st) {
    if (lanes != 16 && lanes != 32 && lanes != 64) {
        set_error("ragged product: lanes per row must be 16, 32 or 64");
        return GSRAD_EINVAL;
    }
    for (const RowTable::Part &p : t.rows[lanes == 16 ? 0 : lanes == 32 ? 1 : 2]) {
        RowArgs a = row_args(F, rho);
        a.tab = reinterpret_cast<const RowScene *>(t.base + p.tab);
        a.first = reinterpret_cast<const int64_t *>(t.base + p.first);
        a.count = p.count;
        const gsrad_status e = run_rows<ADJ>(a, p.g, lanes, p.blocks, in, E, out, p_out, gE, st);
        if (e != GSRAD_OK) return e;
    }
    return GSRAD_OK;
}

}  // namespace

gsrad_status rows_bounce(const Csr &F, const RowScene &s, const float *Bin, const float *E, const float *rho,
                         float *Bout, hipStream_t st) {
    return run_scene<false>(F, s, Bin, E, rho, Bout, nullptr, nullptr, st);
}

gsrad_status rows_adjoint(const Csr &FT, const RowScene &s, const float *p, const float *rho, float *lam,
                          float *p_out, float *gE, hipStream_t st) {
    return run_scene<true>(FT, s, p, nullptr, rho, lam, p_out, gE, st);
}

gsrad_status rows_bounce_batch(const Csr &F, const RowTable &t, int lanes, const float *Bin, const float *E,
                               const float *rho, float *Bout, hipStream_t st) {
    return run_batch<false>(F, t, lanes, Bin, E, rho, Bout, nullptr, nullptr, st);
}

gsrad_status rows_adjoint_batch(const Csr &FT, const RowTable &t, int lanes, const float *p, const float *rho,
                                float *lam, float *p_out, float *gE, hipStream_t st) {
    return run_batch<true>(FT, t, lanes, p, nullptr, rho, lam, p_out, gE, st);
}

gsrad_status rows_seed(const RowScene &s, const float *grad_B, const float *rho, float *lam, float *gE, float *p,
                       hipStream_t st) {
    const int64_t lanes = s.n * (s.C / 3);
    each_launch((lanes + 255) / 256, 256, [&](int64_t first, unsigned blocks) {
        hipLaunchKernelGGL(k_seed, dim3(blocks), dim3(256), 0, st, lanes, s.C / 3, first, grad_B, rho, lam, gE, p);
    });
    return check_hip(hipGetLastError(), "adjoint seed launch");
}

gsrad_status rows_seed_batch(const RowTable &t, const float *grad_B, const float *rho, float *lam, float *gE, float *p,
                             hipStream_t st) {
    const int64_t lanes = t.vals / 3;
    each_launch((lanes + 255) / 256, 256, [&](int64_t first, unsigned blocks) {
        hipLaunchKernelGGL(k_seed_batch, dim3(blocks), dim3(256), 0, st, reinterpret_cast<const RowScene *>(t.base),
                           t.scenes, lanes, first, grad_B, rho, lam, gE, p);
    });
    return check_hip(hipGetLastError(), "adjoint seed launch");
}

namespace {

// How the sampled products take a scene's rows.  Several chunks: side by side in
// one launch where the mean row is short (20k rows of 8 entries, 90
// coefficients, three bounces: 72 us, one launch per chunk 227; of 64 entries
// 471 and 449, but 8k rows 130 and 163) or there are two of at most twelve (50k
// rows of 512, 20 coefficients: 1.8 and 2.3 ms; 20k of 32: 1.8 and 1.5; 2k of
// 20: 107 and 67 us).  One chunk: 16 lanes per short row (20k rows of 8 entries,
// 27 coefficients, six bounces: 27 us, with 64 lanes 48).
RowTable::Part sampled_part(const RowScene &s) {
    RowTable::Part p;
    p.g = row_lanes(s.C);
    const int chunks = row_chunks(s.C / 3, p.g);
    const bool short_rows = s.nnz <= (s.n > kManyItems || chunks == 1 ? kShortRow : 100) * s.n;
    if (chunks > 1 && (short_rows || (chunks == 2 && s.n >= kManyItems && s.C <= 72))) p.cp = chunks == 2 ? 2 : 4;
    p.lanes = p.cp > 1 ? 16 * p.cp : chunks == 1 && s.n >= kManyItems && short_rows ? 16 : 64;
    p.chunks = p.cp > 1 ? 1 : chunks;
    p.per = p.cp > 1 ? 8 : sddmm_bounces(s.n, row_width(s.C / 3, p.g));
    p.blocks = (s.n + kThreads / p.lanes - 1) / (kThreads / p.lanes);
    return p;
}

gsrad_status run_sampled(RowArgs a, const RowTable::Part &p, int nb, int64_t stride, const float *Btape,
                         const float *Ltape, float *grad_F, float *grad_rho, hipStream_t st) {
    for (int chunk = 0; chunk < p.chunks; ++chunk) {
        for (int q0 = 0; q0 < nb; q0 += p.per) {
            const float *B = Btape + q0 * stride, *L = Ltape + q0 * stride;
            // (a scene's first chunk and bounces write, the others add)
            const bool write = chunk == 0 && q0 == 0;
            auto run = [&](auto kernel) {
                each_launch(p.blocks, kThreads, [&](int64_t first, unsigned groups) {
                    a.block0 = first;
                    hipLaunchKernelGGL(kernel, dim3(groups), dim3(kThreads), 0, st, a, chunk, stride, B, L, grad_F,
                                       grad_rho, write);
                });
            };
            auto with = [&](auto bounces) {
                constexpr int N = decltype(bounces)::value;
                if (p.cp == 2) run(k_sddmm3<16, 32, 2, N>);
                else if (p.cp == 4) run(k_sddmm3<16, 64, 4, N>);
                else if (p.g == 1) run(p.lanes == 16 ? k_sddmm3<1, 16, 1, N> : k_sddmm3<1, 64, 1, N>);
                else if (p.g == 4) run(p.lanes == 16 ? k_sddmm3<4, 16, 1, N> : k_sddmm3<4, 64, 1, N>);
                else run(p.lanes == 16 ? k_sddmm3<16, 16, 1, N> : k_sddmm3<16, 64, 1, N>);
            };
            switch (std::min(p.per, nb - q0)) {
                case 1: with(std::integral_constant<int, 1>{}); break;
                case 2: with(std::integral_constant<int, 2>{}); break;
                case 3: with(std::integral_constant<int, 3>{}); break;
                case 4: with(std::integral_constant<int, 4>{}); break;
                case 5: with(std::integral_constant<int, 5>{}); break;
                case 6: with(std::integral_constant<int, 6>{}); break;
                case 7: with(std::integral_constant<int, 7>{}); break;
                case 8: with(std::integral_constant<int, 8>{}); break;
            }
        }
    }
    return check_hip(hipGetLastError(), "sddmm launch");
}

}  // namespace

gsrad_status rows_sddmm(const Csr &F, const RowScene &s, int nb, int64_t stride, const float *Btape,
                        const float *Ltape, const float *rho, float *grad_F, float *grad_rho, hipStream_t st) {
    if (s.n == 0 || nb == 0) return GSRAD_OK;
    RowArgs a = row_args(F, rho);
    a.one = s;
    return run_sampled(a, sampled_part(s), nb, stride, Btape, Ltape, grad_F, grad_rho, st);
}

gsrad_status rows_sddmm_batch(const Csr &F, const RowTable &t, int nb, const float *Btape, const float *Ltape,
                              const float *rho, float *grad_F, float *grad_rho, hipStream_t st) {
    if (nb == 0) return GSRAD_OK;
    for (const RowTable::Part &p : t.sampled) {
        RowArgs a = row_args(F, rho);
        a.tab = reinterpret_cast<const RowScene *>(t.base + p.tab);
        a.first = reinterpret_cast<const int64_t *>(t.base + p.first);
        a.count = p.count;
        const gsrad_status e = run_sampled(a, p, nb, t.vals, Btape, Ltape, grad_F, grad_rho, st);
        if (e != GSRAD_OK) return e;
    }
    for (const RowScene &s : t.alone) {
        const gsrad_status e = rows_sddmm(F, s, nb, t.vals, Btape, Ltape, rho, grad_F, grad_rho, st);
        if (e != GSRAD_OK) return e;
    }
    return GSRAD_OK;
}

// Scenes whose sampled products share launches: up to kJoined rows times chunks.
// A launch of a small one ends before it has filled the chip (64 scenes of 512
// rows, 8 lights, K = 9, six bounces: 6.7 ms with launches of their own, 2.4
// joined; 1,000 of 64 rows 8.1 and 0.2).  Large ones have the same chunk of
// columns in L2 longer by themselves (16 scenes of 4,096 rows, 30 lights: 21.3
// and 22.2 ms).
constexpr int64_t kJoined = 32768;
static bool joined(const RowScene &s) { return s.n * row_chunks(s.C / 3, row_lanes(s.C)) <= kJoined; }

size_t rows_table_bytes(size_t scenes) { return scenes * 3 * sizeof(RowScene) + scenes * 4 * sizeof(int64_t); }

void rows_table(const std::vector<RowScene> &scenes, RowTable *t, std::vector<char> *image) {
    *t = RowTable{};
    image->clear();
    auto put = [&](const void *p, size_t bytes) {
        const size_t at = image->size();
        image->insert(image->end(), static_cast<const char *>(p), static_cast<const char *>(p) + bytes);
        return at;
    };
    put(scenes.data(), scenes.size() * sizeof(RowScene));
    t->scenes = (int)scenes.size();
    double work = 0.0, whole = 0.0;
    for (const RowScene &s : scenes) {
        const double w = (double)s.nnz * s.C;
        t->vals += s.n * s.C;
        work += w;
        if (row_lanes_of(s, false) < 64 || row_lanes_of(s, true) < 64) whole += w;
    }
    t->whole = 2.0 * whole > work;
    for (int g : {1, 4, 16}) {
        std::vector<RowScene> of;
        for (const RowScene &s : scenes)
            if (row_lanes(s.C) == g) of.push_back(s);
        if (of.empty()) continue;
        const size_t tab = put(of.data(), of.size() * sizeof(RowScene));
        for (int k = 0; k < 3; ++k) {
            RowTable::Part p;
            p.g = g;
            p.lanes = 16 << k;
            std::vector<int64_t> first;
            for (const RowScene &s : of) {
                first.push_back(p.blocks);
                p.blocks += rows_blocks(s.n, s.C, p.lanes);
            }
            p.count = (int)of.size();
            p.tab = tab;
            p.first = put(first.data(), first.size() * sizeof(int64_t));
            t->rows[k].push_back(p);
        }
    }
    // joined: scenes of one kernel and as many bounces a launch
    std::vector<bool> taken(scenes.size(), false);
    for (size_t i = 0; i < scenes.size(); ++i) {
        if (taken[i]) continue;
        if (!joined(scenes[i])) {
            t->alone.push_back(scenes[i]);
            continue;
        }
        RowTable::Part p = sampled_part(scenes[i]);
        std::vector<RowScene> of;
        std::vector<int64_t> first;
        int64_t blocks = 0;
        for (size_t k = i; k < scenes.size(); ++k) {
            if (taken[k] || !joined(scenes[k])) continue;
            const RowTable::Part q = sampled_part(scenes[k]);
            if (q.g != p.g || q.lanes != p.lanes || q.cp != p.cp || q.per != p.per) continue;
            taken[k] = true;
            first.push_back(blocks);
            blocks += q.blocks;
            of.push_back(scenes[k]);
            p.chunks = std::max(p.chunks, q.chunks);
        }
        p.blocks = blocks;
        p.count = (int)of.size();
        p.tab = put(of.data(), of.size() * sizeof(RowScene));
        p.first = put(first.data(), first.size() * sizeof(int64_t));
        t->sampled.push_back(p);
    }
}

}  // namespace gsrad
