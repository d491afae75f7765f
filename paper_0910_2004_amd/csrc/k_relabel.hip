// Locality relabelling (Section 3.3: the preliminary partition by recursive
// coordinate bisection of nodes with 2D coordinates).
//
//   rcb order:  depth by depth, every box of more than `leaf` points is sorted
//               stably by x (even depths) or y (odd depths) and cut after its
//               first half.  Sorting a box again by an axis gives the order of
//               one global sort by that axis: stable sorts make it (x, index)
//               at depth 0, (y, x, index) at odd depths and (x, y, index) at
//               even ones from 2 on.  So three lists are sorted once, boxes are
//               contiguous ranges of each, and a depth only marks the points
//               in the second half of their box in the depth's list and splits
//               every box of the other list stably by that mark.  Boxes of up
//               to RCB_BOX points go through all their further depths in LDS.
//   relabel:    node x of the new numbering is node order[x] of the old one;
//               rows move, neighbours are renamed through the inverse, and the
//               entries are ordered by (row, new neighbour): within a wave for
//               rows of up to RL_SHORT entries, with two stable radix sorts
//               (by neighbour, then by row) for the entries of longer rows.
//
// 2^20 points, leaf 32, and a graph of 8.4 M entries: 6.7 ms with a sort of all
// points for every depth (64-bit key, then box) and sorts of all entries, now
// 0.83 ms, of which the order is 0.6 (8 sort passes of 28 us, 9 depths of 24 us,
// 43 us for the last 7) and the rows in order 0.12.
//
// The sorts are the library's own stable LSD radix sorts (k_sort.hip), the
// offsets its device scans.
#include <algorithm>

#include "kappa_internal.h"

namespace kappa {

// Order-preserving 64-bit key of a double (-0.0 as +0.0).
__device__ __forceinline__ uint64_t sortable(double x) {
    if (x == 0.0) x = 0.0;
    const uint64_t b = (uint64_t)__double_as_longlong(x);
    return (b >> 63) ? ~b : (b | 0x8000000000000000ull);
}

constexpr int RCB_THREADS = 512;
constexpr int RCB_ITEMS = 8;
constexpr int RCB_BOX = RCB_THREADS * RCB_ITEMS;   // points of a box kept in LDS
constexpr int RCB_RUN = 64;                        // longest run of equal short keys put in order

// The box of position i after `depth` cuts (or fewer: a box of up to leaf
// points is not cut); returns the cuts made.
__device__ __forceinline__ int rcb_box(int32_t n, int32_t leaf, int depth, int32_t i, int32_t &b,
                                       int32_t &len) {
    b = 0;
    len = n;
    for (int d = 0; d < depth; ++d) {
        if (len <= leaf) return d;
        const int32_t mid = len >> 1;
        if (i - b < mid) {
            len = mid;
        } else {
            b += mid;
            len -= mid;
        }
    }
    return depth;
}

// mm: smallest and largest key of x, then of y (start: ~0, 0, ~0, 0).
__global__ void __launch_bounds__(BLOCK) rcb_range_k(const double *xy, int32_t n, uint64_t *mm) {
    __shared__ uint64_t sh[4][BLOCK / WAVE];
    uint64_t v[4] = {~0ull, 0ull, ~0ull, 0ull};
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x) {
#pragma unroll
        for (int a = 0; a < 2; ++a) {
            const uint64_t k = sortable(xy[2 * i + a]);
            v[2 * a] = min(v[2 * a], k);
            v[2 * a + 1] = max(v[2 * a + 1], k);
        }
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        for (int o = WAVE / 2; o > 0; o >>= 1) {
            const uint64_t u = __shfl_xor((unsigned long long)v[q], o, WAVE);
            v[q] = (q & 1) ? max(v[q], u) : min(v[q], u);
        }
        if (lane_id() == 0) sh[q][threadIdx.x / WAVE] = v[q];
    }
    __syncthreads();
    if (threadIdx.x < 4) {
        const int q = threadIdx.x;
        uint64_t r = sh[q][0];
        for (int w = 1; w < BLOCK / WAVE; ++w) r = (q & 1) ? max(r, sh[q][w]) : min(r, sh[q][w]);
        if (q & 1) atomicMax((unsigned long long *)&mm[q], (unsigned long long)r);
        else atomicMin((unsigned long long *)&mm[q], (unsigned long long)r);
    }
}

// Short keys: the top 32 bits of a key's distance from the smallest, which do
// not decrease with the key.  from: the list in whose order to write (null:
// 0 .. n-1, which goes to val).
__global__ void rcb_short_keys_k(const double *xy, int32_t n, int axis, const uint64_t *mm,
                                 const int32_t *from, uint32_t *key, int32_t *val) {
    const uint64_t lo = mm[2 * axis], span = mm[2 * axis + 1] - lo;
    const int bits = span ? 64 - (int)__clzll((long long)span) : 0, sh = bits > 32 ? bits - 32 : 0;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x) {
        const int64_t v = from ? from[i] : i;
        key[i] = (uint32_t)((sortable(xy[2 * v + axis]) - lo) >> sh);
        if (!from) val[i] = (int32_t)i;
    }
}

// Runs of equal short keys into the order of their full keys, stably, by the
// thread at the run's first position; flag bit 0: a run longer than RCB_RUN is
// out of order; bit 1: two full keys are equal.
__global__ void rcb_runs_k(const double *xy, int32_t n, int axis, const uint32_t *key, int32_t *v,
                           uint32_t *flag) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i + 1 < n;
         i += (int64_t)gridDim.x * blockDim.x) {
        const uint32_t k = key[i];
        if (key[i + 1] != k) continue;
        int64_t b = i, e = i + 2;   // the run, as far as it decides
        while (b > 0 && i - b <= RCB_RUN && key[b - 1] == k) --b;
        while (e < n && e - b <= RCB_RUN && key[e] == k) ++e;
        if (e - b > RCB_RUN) {   // (no thread moves this run)
            const uint64_t x = sortable(xy[2 * (int64_t)v[i] + axis]),
                           y = sortable(xy[2 * (int64_t)v[i + 1] + axis]);
            if (x > y) atomicOr(flag, 1u);
            else if (x == y) atomicOr(flag, 2u);
        } else if (b == i) {
            uint32_t bits = 0;
            for (int64_t p = b + 1; p < e; ++p) {
                const int32_t m = v[p];
                const uint64_t f = sortable(xy[2 * (int64_t)m + axis]);
                int64_t q = p;
                while (q > b) {
                    const uint64_t g = sortable(xy[2 * (int64_t)v[q - 1] + axis]);
                    if (g == f) bits = 2u;
                    if (g <= f) break;
                    v[q] = v[q - 1];
                    --q;
                }
                v[q] = m;
            }
            if (bits) atomicOr(flag, bits);
        }
    }
}

// Full keys in the order of `from` (null: 0 .. n-1, which goes to val).
__global__ void rcb_full_keys_k(const double *xy, int32_t n, int axis, const int32_t *from,
                                uint64_t *key, int32_t *val) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x) {
        const int64_t v = from ? from[i] : i;
        key[i] = sortable(xy[2 * v + axis]);
        if (!from) val[i] = (int32_t)i;
    }
}

// Dense rank of the x keys along the list by x, to the points.
struct RankF {
    const double *xy;
    const int32_t *list;
    int64_t len;
    __device__ int64_t size() const { return len; }
    __device__ int64_t operator()(int64_t i) const {
        return i > 0 && sortable(xy[2 * (int64_t)list[i]]) != sortable(xy[2 * (int64_t)list[i - 1]]);
    }
    __device__ void post(int64_t) const {}
};
struct RankW {
    const int32_t *list;
    uint32_t *rank;
    struct Pre {};
    struct Bound {
        const int32_t *list;
        uint32_t *rank;
        __device__ Pre prefetch(int64_t, int64_t) const { return Pre{}; }
        __device__ void operator()(int64_t i, int64_t pre, int64_t val, const Pre &) const {
            rank[list[i]] = (uint32_t)(pre + val);
        }
    };
    __device__ Bound bind() const { return Bound{list, rank}; }
};

__global__ void gather_i32_k(const int32_t *src, const int32_t *idx, int64_t n, int32_t *dst) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x)
        dst[i] = src[idx[i]];
}

__global__ void iota_k(int32_t *p, int64_t n) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x)
        p[i] = (int32_t)i;
}

// side[v]: v lies in the second half of its box of the list, which is cut.
__global__ void rcb_mark_k(const int32_t *list, int32_t n, int32_t leaf, int depth, uint8_t *side) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x) {
        int32_t b, len;
        rcb_box(n, leaf, depth, (int32_t)i, b, len);
        side[list[i]] = len > leaf && (int32_t)i - b >= (len >> 1);
    }
}

// Bit i of first: the point at position i of the list is not marked.  A block
// takes RCB_TILE positions; before[w]: the bits of its words before word w,
// tiles[t]: all of its bits (scanned next; scanned word by word, 17 us of the
// 40 us of a depth at 2^20 points, now 5).
constexpr int RCB_TILE = WAVE * WAVE;
__global__ void __launch_bounds__(RCB_THREADS) rcb_first_k(const int32_t *list, int32_t n,
                                                           const uint8_t *side, uint64_t *first,
                                                           int32_t *before, int32_t *tiles) {
    static_assert(RCB_TILE == RCB_THREADS * RCB_ITEMS, "a thread's items");
    __shared__ uint64_t words[WAVE];
    const int64_t nt = ((int64_t)n + RCB_TILE - 1) / RCB_TILE;
    for (int64_t t = blockIdx.x; t < nt; t += gridDim.x) {   // block-uniform
        uint8_t m[RCB_ITEMS];
#pragma unroll
        for (int q = 0; q < RCB_ITEMS; ++q) {
            const int64_t i = t * RCB_TILE + q * RCB_THREADS + threadIdx.x;
            m[q] = i < n ? side[list[i]] : 1;
        }
#pragma unroll
        for (int q = 0; q < RCB_ITEMS; ++q) {
            const uint64_t b = __ballot(m[q] == 0);
            if (lane_id() == 0) words[(q * RCB_THREADS + threadIdx.x) / WAVE] = b;
        }
        __syncthreads();
        if (threadIdx.x < WAVE) {
            const int64_t w = t * WAVE + threadIdx.x;
            const uint64_t b = words[threadIdx.x];
            const int32_t c = (int32_t)__popcll(b);
            int32_t incl = c;
            for (int s = 1; s < WAVE; s <<= 1) {
                const int32_t up = __shfl_up(incl, s, WAVE);
                if (lane_id() >= s) incl += up;
            }
            if (w * WAVE < n) {
                first[w] = b;
                before[w] = incl - c;
            }
            if (threadIdx.x == WAVE - 1) tiles[t] = incl;
        }
        __syncthreads();   // words are written again
    }
}

// The tiles' sums to the sums before them, in place.
struct TileF {
    int32_t *tiles;
    int64_t count;
    __device__ int64_t size() const { return count; }
    __device__ int64_t operator()(int64_t t) const { return tiles[t]; }
    __device__ void post(int64_t) const {}
};
struct TileW {
    int32_t *tiles;
    struct Pre {};
    struct Bound {
        int32_t *tiles;
        __device__ Pre prefetch(int64_t, int64_t) const { return Pre{}; }
        __device__ void operator()(int64_t t, int64_t pre, int64_t, const Pre &) const {
            tiles[t] = (int32_t)pre;
        }
    };
    __device__ Bound bind() const { return Bound{tiles}; }
};

// Every box of the list that is cut at this depth, split stably: unmarked
// points, then marked ones.  side (may be null): the marks of the next depth,
// whose list this is.
__global__ void rcb_split_k(const int32_t *list, int32_t n, int32_t leaf, int depth,
                            const uint64_t *first, const int32_t *before, const int32_t *tiles,
                            int32_t *out, uint8_t *side) {
    auto firsts = [&](int32_t i) {   // unmarked points before position i
        return tiles[i / RCB_TILE] + before[i >> 6] +
               (int32_t)__popcll(first[i >> 6] & (((uint64_t)1 << (i & 63)) - 1));
    };
    for (int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; t < n;
         t += (int64_t)gridDim.x * blockDim.x) {
        const int32_t i = (int32_t)t, v = list[i];
        int32_t b, len, j = i;
        rcb_box(n, leaf, depth, i, b, len);
        if (len > leaf) {
            const int32_t mid = len >> 1, z = firsts(i) - firsts(b);
            if ((first[i >> 6] >> (i & 63)) & 1) {
                j = b + z;
                len = mid;
            } else {
                j = b + mid + (i - b - z);
                b += mid;
                len -= mid;
            }
        }
        out[j] = v;
        if (side) side[v] = len > leaf && j - b >= (len >> 1);
    }
}

// The list that holds the order of a box after D cuts.
__device__ __forceinline__ const int32_t *rcb_list(int D, const int32_t *x0, const int32_t *x,
                                                   const int32_t *y) {
    return D == 1 ? x0 : ((D - 1) & 1) ? y : x;
}

// The order where no box is left to cut (n > leaf).
__global__ void rcb_out_k(const int32_t *x0, const int32_t *x, const int32_t *y, int32_t n,
                          int32_t leaf, int32_t *order) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x) {
        int32_t b, len;
        order[i] = rcb_list(rcb_box(n, leaf, 32, (int32_t)i, b, len), x0, x, y)[i];
    }
}

// The boxes after `depth` cuts (>= 1), a block each, of at most RCB_BOX points
// or not to be cut: all further depths in LDS, then the order.  Both lists are
// kept as positions in the box's part of x (loc: a point's, n entries); a depth
// is four barriers and a few LDS accesses per point, and one box per compute
// unit is in flight at 2^20 points, so the depths' latency bounds it.
__global__ void __launch_bounds__(RCB_THREADS) rcb_block_k(const int32_t *x0, const int32_t *x,
                                                           const int32_t *y, int32_t n, int32_t leaf,
                                                           int depth, uint16_t *loc, int32_t *order) {
    __shared__ uint16_t list[2][RCB_BOX];
    __shared__ uint8_t side[RCB_BOX];
    __shared__ uint64_t first[RCB_BOX / WAVE];
    __shared__ int32_t before[RCB_BOX / WAVE];
    static_assert(RCB_BOX / WAVE == WAVE, "one wave scans the words");
    int32_t b = 0, len = n;
    int D = 0;
    for (; D < depth && len > leaf; ++D) {
        const int32_t mid = len >> 1;
        if ((blockIdx.x >> (depth - 1 - D)) & 1u) {
            b += mid;
            len -= mid;
        } else {
            len = mid;
        }
    }
    if (D < depth && (blockIdx.x & ((1u << (depth - D)) - 1))) return;   // no box of that path
    if (len <= leaf) {
        const int32_t *src = rcb_list(D, x0, x, y);
        for (int32_t i = threadIdx.x; i < len; i += RCB_THREADS) order[b + i] = src[b + i];
        return;
    }
    int32_t ib[RCB_ITEMS], il[RCB_ITEMS], iD[RCB_ITEMS];   // the item's box and its cuts
#pragma unroll
    for (int q = 0; q < RCB_ITEMS; ++q) {
        const int32_t i = q * RCB_THREADS + threadIdx.x;
        ib[q] = 0;
        il[q] = i < len ? len : 0;
        iD[q] = depth;
        if (i < len) {
            loc[x[b + i]] = (uint16_t)i;
            list[0][i] = (uint16_t)i;
        }
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < RCB_ITEMS; ++q) {
        const int32_t i = q * RCB_THREADS + threadIdx.x;
        if (i < len) list[1][i] = loc[y[b + i]];
    }
    __syncthreads();
    int d = depth;
    for (int32_t most = len; most > leaf; most -= most >> 1, ++d) {   // most: the largest box
        const uint16_t *a = list[d & 1];
        uint16_t *o = list[1 - (d & 1)];
#pragma unroll
        for (int q = 0; q < RCB_ITEMS; ++q) {
            const int32_t i = q * RCB_THREADS + threadIdx.x;
            if (il[q] > leaf) side[a[i]] = i - ib[q] >= (il[q] >> 1);
        }
        __syncthreads();
        uint16_t v[RCB_ITEMS];
#pragma unroll
        for (int q = 0; q < RCB_ITEMS; ++q) {
            const int32_t i = q * RCB_THREADS + threadIdx.x;
            v[q] = il[q] > 0 ? o[i] : (uint16_t)0;
            const uint64_t m = __ballot(il[q] > leaf && side[v[q]] == 0);
            if (lane_id() == 0) first[i / WAVE] = m;
        }
        __syncthreads();
        if (threadIdx.x < WAVE) {
            const int32_t c = (int32_t)__popcll(first[threadIdx.x]);
            int32_t incl = c;
            for (int s = 1; s < WAVE; s <<= 1) {
                const int32_t up = __shfl_up(incl, s, WAVE);
                if (lane_id() >= s) incl += up;
            }
            before[threadIdx.x] = incl - c;
        }
        __syncthreads();
        auto firsts = [&](int32_t i) {
            return before[i >> 6] + (int32_t)__popcll(first[i >> 6] & (((uint64_t)1 << (i & 63)) - 1));
        };
#pragma unroll
        for (int q = 0; q < RCB_ITEMS; ++q) {
            const int32_t i = q * RCB_THREADS + threadIdx.x;
            if (il[q] <= leaf) continue;
            const int32_t mid = il[q] >> 1, z = firsts(i) - firsts(ib[q]);
            o[(first[i >> 6] >> (i & 63)) & 1 ? ib[q] + z : ib[q] + mid + (i - ib[q] - z)] = v[q];
            if (i - ib[q] < mid) {   // position i's box from here on
                il[q] = mid;
            } else {
                ib[q] += mid;
                il[q] -= mid;
            }
            iD[q] = d + 1;
        }
        __syncthreads();
    }
#pragma unroll
    for (int q = 0; q < RCB_ITEMS; ++q) {
        const int32_t i = q * RCB_THREADS + threadIdx.x;
        if (i < len) order[b + i] = x[b + list[(iD[q] - 1) & 1][i]];
    }
}

// --- relabel ----------------------------------------------------------------
constexpr int RL_SHORT = WAVE;   // entries of a row put in order within a wave
constexpr int RL_GROUP = 16;     // lanes of a row where four rows share a wave

// inv[order[x]] = x; longs: the entries of rows longer than RL_SHORT.
__global__ void __launch_bounds__(BLOCK) relabel_inverse_k(DevGraph g, const int32_t *order,
                                                           int32_t *inv, uint64_t *longs) {
    __shared__ uint64_t sh[BLOCK / WAVE + 1];
    uint64_t sum = 0;
    for (int64_t x = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; x < g.n;
         x += (int64_t)gridDim.x * blockDim.x) {
        const int64_t deg = g.xadj[x + 1] - g.xadj[x];
        if (deg > RL_SHORT) sum += (uint64_t)deg;
        const int32_t v = order[x];
        if ((uint32_t)v < (uint32_t)g.n) inv[v] = (int32_t)x;
    }
    sum = block_sum(sum, sh);
    if (threadIdx.x == 0 && sum) atomicAdd((unsigned long long *)longs, (unsigned long long)sum);
}

// flag: order is not a permutation of 0 .. n-1 (a value out of range, or one
// of two equal values does not find its own position in inv).
__global__ void relabel_check_k(const int32_t *order, int32_t n, const int32_t *inv, uint32_t *flag) {
    bool bad = false;
    for (int64_t x = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; x < n;
         x += (int64_t)gridDim.x * blockDim.x) {
        const int32_t v = order[x];
        bad = bad || (uint32_t)v >= (uint32_t)n || inv[v] != (int32_t)x;
    }
    if (__ballot(bad) && lane_id() == 0) atomicOr(flag, 1u);
}

// New degree and node weight of every new node (deg[n] = 0 closes the scan).
// longs: only the degrees, 0 for a row of at most RL_SHORT entries.
__global__ void relabel_rows_k(DevGraph g, const int32_t *order, int64_t *deg, uint32_t *vw,
                               int longs) {
    for (int64_t x = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; x <= g.n;
         x += (int64_t)gridDim.x * blockDim.x) {
        if (x == g.n) {
            deg[x] = 0;
            continue;
        }
        const int32_t v = order[x];
        const int64_t d = g.xadj[v + 1] - g.xadj[v];
        deg[x] = longs && d <= RL_SHORT ? 0 : d;
        if (!longs) vw[x] = g.vw[v];
    }
}

// Rows of up to RL_SHORT entries, renamed and put in order: a wave takes four
// rows, 16 lanes each, or one after the other where one of them is longer; an
// entry's place is the number of entries before it by (neighbour, position).
// Bound by the gathers of inv and the rows' chain of loads (order, offsets,
// entries); no pass writes what another reads back.
__global__ void __launch_bounds__(BLOCK) relabel_short_k(DevGraph g, const int32_t *order,
                                                         const int32_t *inv, const int64_t *nx,
                                                         int32_t *adj, uint32_t *ew) {
    constexpr int ROWS = WAVE / RL_GROUP;
    const int64_t w0 = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) / WAVE;
    const int64_t nw = (int64_t)gridDim.x * blockDim.x / WAVE;
    const int lane = lane_id(), sub = lane % RL_GROUP, row0 = lane - sub;
    for (int64_t w = w0; w * ROWS < g.n; w += nw) {   // wave-uniform
        const int64_t x = w * ROWS + lane / RL_GROUP;
        int64_t b = 0, d = 0, deg = 0;
        if (x < g.n) {
            const int32_t v = order[x];
            b = g.xadj[v];
            deg = g.xadj[v + 1] - b;
            d = nx[x];
        }
        if (__ballot(deg > RL_GROUP) == 0) {
            uint32_t key = 0xFFFFFFFFu, wt = 0;
            if (sub < deg) {
                key = (uint32_t)inv[g.adj[b + sub]];
                wt = g.ew[b + sub];
            }
            int rank = 0;
#pragma unroll
            for (int l = 0; l < RL_GROUP; ++l) {
                const uint32_t o = __shfl(key, row0 + l, WAVE);
                rank += o < key || (o == key && l < sub);
            }
            if (sub < deg) {
                adj[d + rank] = (int32_t)key;
                ew[d + rank] = wt;
            }
            continue;
        }
        for (int r = 0; r < ROWS; ++r) {
            const int64_t rb = __shfl((long long)b, r * RL_GROUP, WAVE),
                          rd = __shfl((long long)d, r * RL_GROUP, WAVE),
                          rn = __shfl((long long)deg, r * RL_GROUP, WAVE);
            if (rn > RL_SHORT) continue;   // wave-uniform
            uint32_t key = 0xFFFFFFFFu, wt = 0;
            if (lane < rn) {
                key = (uint32_t)inv[g.adj[rb + lane]];
                wt = g.ew[rb + lane];
            }
            int rank = 0;
            for (int l = 0; l < (int)rn; ++l) {
                const uint32_t o = __shfl(key, l, WAVE);
                rank += o < key || (o == key && l < lane);
            }
            if (lane < rn) {
                adj[rd + rank] = (int32_t)key;
                ew[rd + rank] = wt;
            }
        }
    }
}

// The entries of the longer rows in the old order, renamed, with their row and
// position (one wave per row; lx: the rows' first positions).
__global__ void relabel_fill_k(DevGraph g, const int32_t *order, const int32_t *inv,
                               const int64_t *lx, int32_t *adj, uint32_t *ew, uint32_t *row,
                               int32_t *pos) {
    const int64_t w0 = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) / WAVE;
    const int64_t nw = (int64_t)gridDim.x * blockDim.x / WAVE;
    for (int64_t x = w0; x < g.n; x += nw) {
        const int32_t v = order[x];
        const int64_t b = g.xadj[v], e = g.xadj[v + 1], d = lx[x];
        if (e - b <= RL_SHORT) continue;
        for (int64_t j = b + lane_id(); j < e; j += WAVE) {
            const int64_t t = d + (j - b);
            adj[t] = inv[g.adj[j]];
            ew[t] = g.ew[j];
            row[t] = (uint32_t)x;
            pos[t] = (int32_t)t;
        }
    }
}

// Sorted entry j of the longer rows (row row[j]) to its place.
__global__ void relabel_gather_k(const int32_t *adj0, const uint32_t *ew0, const int32_t *idx,
                                 const uint32_t *row, const int64_t *lx, const int64_t *nx,
                                 int64_t m, int32_t *adj, uint32_t *ew) {
    for (int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; j < m;
         j += (int64_t)gridDim.x * blockDim.x) {
        const int32_t s = idx[j];
        const int64_t r = row[j], t = nx[r] + (j - lx[r]);
        adj[t] = adj0[s];
        ew[t] = ew0[s];
    }
}

static int bits_for(int64_t count) {   // bits of the largest value count - 1
    int b = 1;
    while (b < 63 && ((int64_t)1 << b) < count) ++b;
    return b;
}

#define HCHK(expr)                                    \
    do {                                              \
        if ((expr) != hipSuccess) return KAPPA_E_HIP; \
    } while (0)

static size_t al256(size_t x) { return (x + 255) & ~(size_t)255; }

// The scan workspace of launch_scan for n items.
static size_t scan_ws_bytes(int64_t n) { return al256(8 * (scan_tiles(n) + 1)) + 4 * ARRIVE_WORDS; }

// ws == nullptr: only *need is set.  hflag: a pinned host word.  Synchronous.
kappa_status rcb_order_impl(const double *xy, int32_t n, int32_t leaf, int32_t *order,
                            hipStream_t s, char *ws, size_t ws_bytes, size_t *need,
                            uint32_t *hflag) {
    const size_t nn = (size_t)std::max(n, 1), words = (nn + WAVE - 1) / WAVE;
    // the sorts' keys, and when those are done the lists' other halves and the
    // marks (side, loc, first, before, tiles)
    const size_t o_side = 0, o_loc = al256(nn), o_first = al256(o_loc + 2 * nn),
                 o_before = al256(o_first + 8 * words), o_tiles = al256(o_before + 4 * words),
                 marks = al256(o_tiles + 4 * (nn / RCB_TILE + 1));
    const size_t o_k0 = 0, o_k1 = al256(o_k0 + std::max(8 * nn, 2 * al256(4 * nn))),
                 o_x0 = al256(o_k1 + std::max(8 * nn, marks)), o_x = al256(o_x0 + 4 * nn),
                 o_y = al256(o_x + 4 * nn), o_mm = al256(o_y + 4 * nn), o_tmp = o_mm + 256,
                 total = al256(o_tmp + std::max({radix_sort_ws_bytes((int64_t)nn, 8),
                                                 radix_sort_ws_bytes((int64_t)nn, 4),
                                                 scan_ws_bytes((int64_t)nn)}));
    *need = total;
    if (!ws) return KAPPA_OK;
    if (ws_bytes < total) return KAPPA_E_NOMEM;
    if (n <= 0) return KAPPA_OK;
    const dim3 grid(grid_for(n, BLOCK, 4096)), blk(BLOCK);
    if (n <= leaf) {
        hipLaunchKernelGGL(iota_k, grid, blk, 0, s, order, (int64_t)n);
        HCHK(hipGetLastError());
        HCHK(hipStreamSynchronize(s));
        return KAPPA_OK;
    }
    uint64_t *K0 = (uint64_t *)(ws + o_k0), *K1 = (uint64_t *)(ws + o_k1);
    uint32_t *q0 = (uint32_t *)K0, *q1 = (uint32_t *)K1;
    int32_t *x0 = (int32_t *)(ws + o_x0), *x = (int32_t *)(ws + o_x), *y = (int32_t *)(ws + o_y);
    uint64_t *mm = (uint64_t *)(ws + o_mm);
    uint32_t *flag = (uint32_t *)(mm + 4);   // [2]: by x, by y
    char *tmp = ws + o_tmp;
    int64_t *partials = (int64_t *)tmp;
    unsigned *arrive = (unsigned *)(tmp + al256(8 * (scan_tiles((int64_t)nn) + 1)));
    auto by_short = [&](int axis, const int32_t *from, int32_t *out) -> kappa_status {
        // x holds 0 .. n-1 where there is no list to start from
        hipLaunchKernelGGL(rcb_short_keys_k, grid, blk, 0, s, xy, n, axis, mm, from, q0, x);
        const kappa_status st = radix_sort_pairs<uint32_t>(q0, q1, (const uint32_t *)(from ? from : x),
                                                           (uint32_t *)out, n, 0, 32, tmp, s);
        if (st != KAPPA_OK) return st;
        hipLaunchKernelGGL(rcb_runs_k, grid, blk, 0, s, xy, n, axis, q1, out, flag + axis);
        return KAPPA_OK;
    };
    auto by_full = [&](int axis, const int32_t *from, int32_t *out) -> kappa_status {
        hipLaunchKernelGGL(rcb_full_keys_k, grid, blk, 0, s, xy, n, axis, from, K0, x);
        return radix_sort_pairs<uint64_t>(K0, K1, (const uint32_t *)(from ? from : x),
                                          (uint32_t *)out, n, 0, 64, tmp, s);
    };
    // (x, index) and (y, x, index).  32-bit keys sort in half the passes and
    // bytes of the full ones and leave short runs to put in order, unless the
    // coordinates crowd: then the full keys.
    ZeroRanges z;
    z.add(mm, 10);
    launch_zero(z, s);
    launch_fill_u64(mm, 1, ~0ull, s);
    launch_fill_u64(mm + 2, 1, ~0ull, s);
    hipLaunchKernelGGL(rcb_range_k, dim3(grid_for(n, BLOCK * 8, 256)), blk, 0, s, xy, n, mm);
    kappa_status st = by_short(0, nullptr, x0);
    if (st == KAPPA_OK) st = by_short(1, x0, y);
    if (st != KAPPA_OK) return st;
    HCHK(hipMemcpyAsync(hflag, flag, 8, hipMemcpyDeviceToHost, s));
    HCHK(hipStreamSynchronize(s));
    const bool full_x = hflag[0] & 1u, full_y = full_x || (hflag[1] & 1u);
    if (full_x) st = by_full(0, nullptr, x0);
    if (st == KAPPA_OK && full_y) st = by_full(1, x0, y);
    if (st != KAPPA_OK) return st;
    // (x, y, index): the same as (x, index) where no two x are equal, else
    // (y, x, index) sorted by the rank of x
    const int32_t *lx = x0, *ly = y;
    if (hflag[0]) {
        uint32_t *rank = (uint32_t *)(ws + o_k0 + al256(4 * nn));
        ZeroRanges za;
        za.add(arrive, ARRIVE_WORDS);
        launch_zero(za, s);
        launch_scan(n, RankF{xy, x0, n}, RankW{x0, rank}, partials, arrive, nullptr, s);
        hipLaunchKernelGGL(gather_i32_k, grid, blk, 0, s, (const int32_t *)rank, y, (int64_t)n,
                           (int32_t *)q0);
        st = radix_sort_pairs<uint32_t>(q0, q1, (const uint32_t *)y, (uint32_t *)x, n, 0,
                                        bits_for(n), tmp, s);
        if (st != KAPPA_OK) return st;
        lx = x;
    }
    uint8_t *side = (uint8_t *)(ws + o_k1 + o_side);
    uint16_t *loc = (uint16_t *)(ws + o_k1 + o_loc);
    uint64_t *first = (uint64_t *)(ws + o_k1 + o_first);
    int32_t *before = (int32_t *)(ws + o_k1 + o_before), *tiles = (int32_t *)(ws + o_k1 + o_tiles);
    const int64_t nt = ((int64_t)n + RCB_TILE - 1) / RCB_TILE;
    // a list alternates between its two buffers
    int32_t *bx[2] = {(int32_t *)(ws + o_k0), x}, *by[2] = {(int32_t *)(ws + o_k0 + al256(4 * nn)), y};
    int ix = 0, iy = 0;
    ZeroRanges za;
    za.add(arrive, ARRIVE_WORDS);
    launch_zero(za, s);
    auto split = [&](bool of_y, int depth, bool mark) {
        const int32_t *in = of_y ? ly : lx;
        int32_t *out = of_y ? by[iy] : bx[ix];
        hipLaunchKernelGGL(rcb_first_k, dim3(grid_for(nt, 1, 4096)), dim3(RCB_THREADS), 0, s, in, n,
                           side, first, before, tiles);
        launch_scan(nt, TileF{tiles, nt}, TileW{tiles}, partials, arrive, nullptr, s);
        hipLaunchKernelGGL(rcb_split_k, grid, blk, 0, s, in, n, leaf, depth, first, before, tiles, out,
                           mark ? side : (uint8_t *)nullptr);
        if (of_y) {
            ly = out;
            iy ^= 1;
        } else {
            lx = out;
            ix ^= 1;
        }
    };
    hipLaunchKernelGGL(rcb_mark_k, grid, blk, 0, s, x0, n, leaf, 0, side);
    split(false, 0, false);
    split(true, 0, true);
    int depth = 1;
    int32_t most = n - (n >> 1);   // the largest box
    for (; most > RCB_BOX && most > leaf; most -= most >> 1, ++depth)
        split((depth & 1) == 0, depth, true);   // the list that is not the depth's own
    if (most > leaf)
        hipLaunchKernelGGL(rcb_block_k, dim3(1u << depth), dim3(RCB_THREADS), 0, s, x0, lx, ly, n,
                           leaf, depth, loc, order);
    else
        hipLaunchKernelGGL(rcb_out_k, grid, blk, 0, s, x0, lx, ly, n, leaf, order);
    HCHK(hipGetLastError());
    HCHK(hipStreamSynchronize(s));
    return KAPPA_OK;
}

// ws == nullptr: only *need is set.  hflag: pinned host words (flag, then at
// +2 the long rows' entries).  Synchronous.
kappa_status relabel_impl(const DevGraph &g, const int32_t *order, int64_t *nx, int32_t *nadj,
                          uint32_t *new_ew, uint32_t *nvw, hipStream_t s, char *ws,
                          size_t ws_bytes, size_t *need, uint32_t *hflag) {
    const size_t nn = (size_t)std::max(g.n, 1), ne = (size_t)std::max<int64_t>(g.nnz, 1);
    const size_t ts = exclusive_sum_ws_bytes((int64_t)nn + 1), t1 = radix_sort_ws_bytes((int64_t)ne, 4);
    const size_t o_inv = 0, o_flag = al256(4 * nn),
                 o_deg = al256(o_flag + 16), o_lx = al256(o_deg + 8 * (nn + 1)),
                 o_a = al256(o_lx + 8 * (nn + 1)),
                 o_w = al256(o_a + 4 * ne), o_row = al256(o_w + 4 * ne),
                 o_p0 = al256(o_row + 4 * ne), o_k1 = al256(o_p0 + 4 * ne),
                 o_p1 = al256(o_k1 + 4 * ne), o_r1 = al256(o_p1 + 4 * ne),
                 o_p2 = al256(o_r1 + 4 * ne), o_tmp = al256(o_p2 + 4 * ne),
                 total = al256(o_tmp + std::max(ts, t1));
    *need = total;
    if (!ws) return KAPPA_OK;
    if (ws_bytes < total) return KAPPA_E_NOMEM;
    int32_t *inv = (int32_t *)(ws + o_inv);
    uint32_t *flag = (uint32_t *)(ws + o_flag);
    uint64_t *longs = (uint64_t *)(flag + 2);
    int64_t *deg = (int64_t *)(ws + o_deg), *lx = (int64_t *)(ws + o_lx);
    int32_t *a0 = (int32_t *)(ws + o_a), *p0 = (int32_t *)(ws + o_p0);
    uint32_t *w0 = (uint32_t *)(ws + o_w), *row = (uint32_t *)(ws + o_row);
    uint32_t *k1 = (uint32_t *)(ws + o_k1), *r1 = (uint32_t *)(ws + o_r1);
    int32_t *p1 = (int32_t *)(ws + o_p1), *p2 = (int32_t *)(ws + o_p2);
    void *tmp = ws + o_tmp;
    ZeroRanges z;
    z.add(flag, 4);
    launch_zero(z, s);
    if (g.n > 0) {
        const dim3 grid(grid_for(g.n, BLOCK, 4096));
        hipLaunchKernelGGL(relabel_inverse_k, grid, dim3(BLOCK), 0, s, g, order, inv, longs);
        hipLaunchKernelGGL(relabel_check_k, grid, dim3(BLOCK), 0, s, order, g.n, inv, flag);
    }
    HCHK(hipMemcpyAsync(hflag, flag, 16, hipMemcpyDeviceToHost, s));
    HCHK(hipStreamSynchronize(s));
    if (*hflag) return KAPPA_E_ARG;   // not a permutation of 0 .. n-1
    const int64_t m = *(const int64_t *)(hflag + 2);
    const dim3 rows(grid_for((int64_t)g.n + 1, BLOCK, 4096));
    hipLaunchKernelGGL(relabel_rows_k, rows, dim3(BLOCK), 0, s, g, order, deg, nvw, 0);
    kappa_status st = exclusive_sum_i64(deg, nx, (int64_t)g.n + 1, (char *)tmp, s);
    if (st != KAPPA_OK) return st;
    if (g.n > 0 && g.nnz > 0)
        hipLaunchKernelGGL(relabel_short_k, dim3(grid_for(g.n, BLOCK / RL_GROUP, 16384)), dim3(BLOCK),
                           0, s, g, order, inv, nx, nadj, new_ew);
    if (m > 0) {
        if (m > g.nnz) return KAPPA_E_ARG;   // offsets that do not ascend
        hipLaunchKernelGGL(relabel_rows_k, rows, dim3(BLOCK), 0, s, g, order, deg, nvw, 1);
        st = exclusive_sum_i64(deg, lx, (int64_t)g.n + 1, (char *)tmp, s);
        if (st != KAPPA_OK) return st;
        hipLaunchKernelGGL(relabel_fill_k, dim3(grid_for(g.n, BLOCK / WAVE, 4096)), dim3(BLOCK), 0, s,
                           g, order, inv, lx, a0, w0, row, p0);
        // by new neighbour, then stably by row
        st = radix_sort_pairs<uint32_t>((const uint32_t *)a0, k1, (const uint32_t *)p0,
                                        (uint32_t *)p1, m, 0, bits_for(g.n), (char *)tmp, s);
        if (st != KAPPA_OK) return st;
        hipLaunchKernelGGL(gather_i32_k, dim3(grid_for(m, BLOCK, 4096)), dim3(BLOCK), 0, s,
                           (const int32_t *)row, p1, m, (int32_t *)k1);
        st = radix_sort_pairs<uint32_t>(k1, r1, (const uint32_t *)p1, (uint32_t *)p2, m, 0,
                                        bits_for(g.n), (char *)tmp, s);
        if (st != KAPPA_OK) return st;
        hipLaunchKernelGGL(relabel_gather_k, dim3(grid_for(m, BLOCK, 4096)), dim3(BLOCK), 0, s, a0,
                           w0, p2, r1, lx, nx, m, nadj, new_ew);
    }
    HCHK(hipGetLastError());
    HCHK(hipStreamSynchronize(s));
    return KAPPA_OK;
}

}  // namespace kappa
