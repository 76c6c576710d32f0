// Contributions of recorded hits to their surfels' sums, listed by block of
// surfels and summed in LDS.  (trace.hip: opacity, grad.hip: geometry.)
//
// A sum per surfel in global memory takes an atomic per contribution; a 100k
// surfel scene's opacity gradient has 356 M of them (34 G/s: 11 of its 17 ms),
// the geometry gradient ten times as many a hit (28 of 34 ms for 30k surfels).
// Here a workgroup that makes contributions writes them to its own stretch of a
// list, ordered by block of surfels, and a second kernel gives every block to
// workgroups that read its parts of all stretches and add in a table in LDS, one
// place per surfel.  Integer sums: the order does not matter.  A block is every
// 2^bits-th surfel, not a range: neighbours are hit alike, and ranges had up to
// ten times the mean (the second kernel on a 100k-surfel bowl 2.85 ms, now
// 0.39 ms a chunk).
#pragma once

#include <algorithm>

#include "gsrad_internal.h"
#include "traverse.h"

namespace gsrad {

// Device view of a list for one chunk of stretches
struct HitLists {
    unsigned long long *used;   // places given out (zeroed before each chunk)
    uint2 *part;                // [stretches][blocks] first and end place
    char *entry;                // [capacity] entries
    int64_t capacity;           // places; 0: no list, contributions are added where they are made
    int bits;                   // 2^bits blocks
    __host__ __device__ int blocks() const { return 1 << bits; }
};

// Rule: listed where the rays reach kListRays, the surfels make at most `most`
// blocks of 2^shift, and a stretch has `share` times as many rays as there are
// blocks: with fewer its parts are a few contributions each, and the parts'
// table costs more than the atomics.  1,024 receivers of 128 rays (131k rays):
// opacity 402 us and geometry 744 us listed, 508 and 2,122 us added directly;
// 512 of 64 rays, the opacity's 37 us of direct adds leave nothing to gain.
constexpr int64_t kListRays = (int64_t)1 << 16;
// Bytes of a chunk's entries, and its stretches at most.  A chunk's two launches
// end with a few workgroups each, so few large chunks: 30k surfels' geometry
// 11.0 ms with 1 GiB, 8.8 with 2, 7.4 with 4; 100k surfels' opacity 12.7, 11.9
// and 11.3 ms.  An allocation of 4 GiB took up to 1.6 s at a handle's first
// call, of 2 GiB it is not seen.  Scenes of few rays take less.
constexpr int64_t kListBytes = (int64_t)1 << 31;
constexpr int64_t kListStretches = 1 << 16;

inline bool lists_pay(int64_t n, int R, int shift, int64_t most, double share) {
    const int64_t blocks = ((n - 1) >> shift) + 1;
    return n * R >= kListRays && blocks <= most && std::min(R, 256) >= share * (double)blocks;
}

// Host layout of the workspace: used, parts, entries
struct ListLayout {
    int64_t stretches, capacity, bytes;
    int bits = 0;
    // 64 contributions a ray expected: what does not fit is added directly
    ListLayout(int64_t n, int R, int threads, int shift, int entry_bytes) {
        while (((n - 1) >> shift) >> bits) ++bits;
        const int64_t batches = (R + threads - 1) / threads, per = (int64_t)threads * 64;
        const int64_t fit = std::max<int64_t>(batches, kListBytes / (per * entry_bytes) / batches * batches);
        stretches = std::min({n * batches, fit, kListStretches / batches * batches});
        capacity = std::min<int64_t>(stretches * per, (int64_t)1 << 31);
        bytes = entries() + capacity * entry_bytes;
    }
    int64_t entries() const { return (256 + (stretches * 8 << bits) + 255) / 256 * 256; }
    HitLists view(void *ws) const {
        char *p = static_cast<char *>(ws);
        HitLists l;
        l.used = reinterpret_cast<unsigned long long *>(p);
        l.part = reinterpret_cast<uint2 *>(p + 256);
        l.entry = p + entries();
        l.capacity = capacity;
        l.bits = bits;
        return l;
    }
};

namespace {

// One stretch: count(j) for every contribution to come, open(), place(j) for
// each (at most as often as counted), close().  open and close are called by
// the whole workgroup; `lds` holds blocks words.
struct ListStretch {
    const HitLists &list;
    uint32_t *next;   // [blocks] counts, then the next place
    uint2 *part;      // this stretch's parts
    bool on;
    __device__ __forceinline__ ListStretch(const HitLists &l, uint32_t *lds, int64_t stretch)
        : list(l), next(lds), part(l.part + (stretch << l.bits)), on(l.capacity > 0) {}
    // (before a barrier and the counts)
    __device__ __forceinline__ void clear(int tid, int threads) {
        if (!on) return;
        for (int b = tid; b < list.blocks(); b += threads) next[b] = 0;
    }
    __device__ __forceinline__ void count(uint32_t j) {
        if (on) atomicAdd(next + (j & (uint32_t)(list.blocks() - 1)), 1u);
    }
    __device__ __forceinline__ void open(int tid, int threads) {
        if (!on) return;
        __shared__ unsigned long long base;
        __syncthreads();
        if (tid < 64) {
            uint32_t total = 0;
            for (int b0 = 0; b0 < list.blocks(); b0 += 64) {
                const int b = b0 + tid;
                const uint32_t v = b < list.blocks() ? next[b] : 0u;
                const uint32_t sum = wave_incl_scan_u32(v);
                if (b < list.blocks()) next[b] = total + sum - v;
                total += (uint32_t)__shfl((int)sum, 63);
            }
            if (tid == 0) base = atomicAdd(list.used, (unsigned long long)total);
            if (tid == 0 && base + total > (unsigned long long)list.capacity) base = ~0ull;
        }
        __syncthreads();
        on = base != ~0ull;
        for (int b = tid; b < list.blocks(); b += threads) {
            const uint32_t first = on ? (uint32_t)base + next[b] : 0u;
            next[b] = first;
            part[b] = make_uint2(first, first);
        }
        __syncthreads();
    }
    __device__ __forceinline__ uint32_t place(uint32_t j) { return atomicAdd(next + (j & (uint32_t)(list.blocks() - 1)), 1u); }
    __device__ __forceinline__ void close(int tid, int threads) {
        if (!on) return;
        __syncthreads();
        for (int b = tid; b < list.blocks(); b += threads) part[b].y = next[b];
    }
};

}  // namespace

}  // namespace gsrad
