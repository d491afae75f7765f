// Pairwise refinement of a k-way partition (Section 5).
//
//   quotient:  Q has an edge {a, b} (a < b) when an edge of G joins blocks a
//              and b; a k x k bitmap built with LDS-aggregated ORs.  The same
//              sweep marks the nodes with a neighbour in another block (ext)
//              and counts them per block.
//   colouring: Q's edges in ascending (a, b) order, each taking the smallest
//              colour free at both ends (the sequential greedy colouring that
//              Section 5.1 parallelises); one workgroup, since each choice
//              depends on all earlier ones.  Pairs of one colour share no
//              block, so their local searches touch disjoint node sets and
//              disjoint block weights and run side by side.
//   bucket:    the nodes listed by block, the marked ones of a block first,
//              once per global iteration.  A node that enters a block or gets
//              a neighbour in another block later in the iteration is a moved
//              node or a neighbour of one: an adoption appends those to a
//              second list, which every later pair reads too.  The lists may
//              name a node twice, or one that has left: a pair keeps what its
//              own test finds.
//   fm:        one launch per colour, one workgroup per pair.  A pair of at
//              most FM_AREA nodes is read once per launch, renumbered from 0,
//              and stays on chip (its rows too where they fit) for all its
//              local iterations.  A larger pair takes, per local iteration,
//              its boundary and the bounded BFS around it from memory, and
//              keeps the search area on chip.  Then the two local searches of
//              the local iteration (run seeds r = 0, 1) on one wave each, and
//              the adoption of the better one; the workgroup repeats local
//              iterations until one improves nothing (Section 5.2).
//
// Every choice is a maximum under a strict total order, so the result does
// not depend on the order of reductions or of the lists: it is bit-exact
// with the sequential definition.
#include <algorithm>
#include <type_traits>

#include "kappa_internal.h"

namespace kappa {

constexpr int RQ_THREADS = 256;
constexpr int RB_ITEMS = 16;           // nodes per thread in the bucket pass
constexpr int FM_THREADS = 512;
constexpr int FM_AREA = 4096;          // largest pair or search area kept in LDS
constexpr int FM_GROUPS = 32;          // groups of area nodes per side (one lane each)
constexpr int ROW_CHUNK = 8;
// Rows read from memory by a pair's workgroup: RG_LANES lanes a row, so that a
// wave's load touches few lines, and RG_U rows of a group in flight: one
// workgroup alone has to cover the latency of its loads.
constexpr int RG_LANES = 16, RG_U = 8;
constexpr int RG_GROUPS = FM_THREADS / RG_LANES, RG_ROWS = RG_GROUPS * RG_U;
constexpr int FM_TILE = 4096;          // listed nodes tested at a time (larger pairs)
constexpr int FM_ENT = 8;              // listed nodes or row entries of a thread in flight

// The lanes of the caller's group of RG_LANES for which x holds (all lanes of
// the wave call it).
__device__ __forceinline__ uint32_t group_ballot(bool x) {
    return (uint32_t)(__ballot(x) >> (lane_id() & ~(RG_LANES - 1))) & ((1u << RG_LANES) - 1u);
}
// Places for the lanes with x behind a counter in LDS: one atomic per wave
// (those of all lanes on one address would run one after the other).  All
// lanes of the wave call it.
__device__ __forceinline__ int32_t wave_places(bool x, int32_t *cnt) {
    const uint64_t m = __ballot(x);
    if (m == 0) return 0;
    int32_t base = 0;
    if (lane_id() == 0) base = atomicAdd(cnt, (int32_t)__popcll(m));
    return __builtin_amdgcn_readfirstlane(base) + (int32_t)__popcll(m & lanemask_lt());
}
__device__ __forceinline__ uint64_t run_seed_of(uint64_t seed, int32_t g, int32_t a, int32_t b,
                                                int32_t t, int32_t r) {
    uint64_t h = mix64(seed + (uint64_t)(uint32_t)g);
    h = mix64(h ^ (((uint64_t)(uint32_t)a << 32) | (uint32_t)b));
    return mix64(h + 2 * (uint64_t)(uint32_t)t + (uint64_t)(uint32_t)r);
}

__device__ __forceinline__ bool state_below(int64_t i1, int64_t c1, int64_t i2, int64_t c2) {
    return i1 < i2 || (i1 == i2 && c1 < c2);
}

__device__ __forceinline__ int64_t pair_imb(int64_t w0, int64_t w1, int64_t S, int64_t L) {
    const int64_t x = S * (w0 > w1 ? w0 : w1) - L;
    return x > 0 ? x : 0;
}

// Runs f(v, row start, row end, first, step) for every row of the wave's
// nodes: rows of at most ROW_LONG entries by the node's own lane (first 0,
// step 1), longer ones by the whole wave, one after the other (first = lane,
// step = WAVE).  Every lane calls it; v < 0: no node.
constexpr int ROW_LONG = 256;
template <class F>
__device__ __forceinline__ void wave_rows(int32_t v, int64_t x0, int64_t x1, F &&f) {
    const bool big = v >= 0 && x1 - x0 > ROW_LONG;
    if (v >= 0 && !big) f(v, x0, x1, 0, 1);
    uint64_t m = __ballot(big);
    while (m) {
        const int l = __builtin_ctzll(m);
        m &= m - 1;
        f(__shfl(v, l), __shfl(x0, l), __shfl(x1, l), lane_id(), WAVE);
    }
}

// block weights, node counts and degree sums, c(V), max c(v), the largest
// weighted degree and the sum of all; flags a block id outside [0, k).  Also clears the search
// scratch that starts empty.
__global__ void __launch_bounds__(RQ_THREADS)
    ref_weights_k(const int64_t *__restrict__ xadj, const uint32_t *__restrict__ ew,
                  const int32_t *__restrict__ part, const uint32_t *__restrict__ vw, int32_t n,
                  int32_t k, int64_t *bw, int32_t *bc, int64_t *bd, int32_t *loc, int32_t *xlist,
                  RefineCtl *ctl) {
    __shared__ unsigned long long s_w[REFINE_K_MAX], s_d[REFINE_K_MAX];
    __shared__ int32_t s_c[REFINE_K_MAX];
    __shared__ unsigned long long s_tot, s_max, s_wd, s_sum;
    __shared__ uint32_t s_bad;
    for (int i = threadIdx.x; i < k; i += blockDim.x) { s_w[i] = 0; s_d[i] = 0; s_c[i] = 0; }
    if (threadIdx.x == 0) { s_tot = 0; s_max = 0; s_wd = 0; s_sum = 0; s_bad = 0; }
    __syncthreads();
    unsigned long long tot = 0, mx = 0, wd = 0, all = 0;
    for (int64_t v0 = (int64_t)blockIdx.x * blockDim.x; v0 < n;
         v0 += (int64_t)gridDim.x * blockDim.x) {   // block-uniform
        const int64_t v = v0 + threadIdx.x;
        const bool live = v < n;
        int64_t x0 = 0, x1 = 0;
        if (live) {
            const int32_t p = part[v];
            const uint32_t c = vw[v];
            x0 = xadj[v];
            x1 = xadj[v + 1];
            loc[v] = -1;
            xlist[v] = 0;
            tot += c;
            mx = c > mx ? c : mx;
            if (p < 0 || p >= k) {
                s_bad = 1;
            } else {
                atomicAdd(&s_w[p], (unsigned long long)c);
                atomicAdd(&s_d[p], (unsigned long long)(x1 - x0));
                atomicAdd(&s_c[p], 1);
            }
        }
        wave_rows(live ? (int32_t)v : -1, x0, x1,
                  [&](int32_t, int64_t b, int64_t e, int first, int step) {
                      unsigned long long sum = 0;
                      for (int64_t j = b + first; j < e; j += (int64_t)step * ROW_CHUNK) {
                          uint32_t w[ROW_CHUNK];
#pragma unroll
                          for (int q = 0; q < ROW_CHUNK; ++q)
                              w[q] = j + (int64_t)q * step < e ? ew[j + (int64_t)q * step] : 0u;
#pragma unroll
                          for (int q = 0; q < ROW_CHUNK; ++q) sum += w[q];
                      }
                      all += sum;
                      if (step > 1) sum = wave_sum(sum);
                      wd = sum > wd ? sum : wd;
                  });
    }
    tot = wave_sum(tot);
    mx = wave_max(mx);
    wd = wave_max(wd);
    all = wave_sum(all);
    if (lane_id() == 0) {
        atomicAdd(&s_tot, tot);
        atomicMax(&s_max, mx);
        atomicMax(&s_wd, wd);
        atomicAdd(&s_sum, all);
    }
    __syncthreads();
    for (int i = threadIdx.x; i < k; i += blockDim.x) {
        if (s_c[i]) {
            atomicAdd((unsigned long long *)&bw[i], s_w[i]);
            atomicAdd((unsigned long long *)&bd[i], s_d[i]);
            atomicAdd(&bc[i], s_c[i]);
        }
    }
    if (threadIdx.x == 0) {
        atomicAdd(&ctl->total, s_tot);
        atomicMax(&ctl->max_node, s_max);
        atomicMax(&ctl->max_wd, s_wd);
        atomicAdd(&ctl->sum_wd, s_sum);
        if (s_bad) atomicOr(&ctl->flags, 1u);
    }
}

// Q as a bitmap (row a, bit b for a < b), the marked nodes (ext: a neighbour
// in another block) and their number per block
__global__ void __launch_bounds__(RQ_THREADS)
    ref_quotient_k(const int64_t *__restrict__ xadj, const int32_t *__restrict__ adj,
                   const int32_t *__restrict__ part, int32_t n, int32_t k,
                   unsigned long long *qbits, uint16_t *ext, int32_t *bcnt) {
    __shared__ unsigned long long s_q[REFINE_K_MAX * REFINE_QW];
    __shared__ int32_t s_n[REFINE_K_MAX];
    const int qw = (k + 63) / 64;
    for (int i = threadIdx.x; i < k * qw; i += blockDim.x) s_q[i] = 0;
    for (int i = threadIdx.x; i < k; i += blockDim.x) s_n[i] = 0;
    __syncthreads();
    for (int64_t v0 = (int64_t)blockIdx.x * blockDim.x; v0 < n;
         v0 += (int64_t)gridDim.x * blockDim.x) {   // block-uniform
        const int64_t v = v0 + threadIdx.x;
        int32_t mine = -1;
        int64_t x0 = 0, x1 = 0;
        if (v < n) {
            mine = part[v];
            x0 = xadj[v];
            x1 = xadj[v + 1];
        }
        const bool live = mine >= 0 && mine < k;   // others are reported by the weights pass
        bool out = false;
        wave_rows(live ? (int32_t)v : -1, x0, x1,
                  [&](int32_t r, int64_t b0, int64_t e0, int first, int step) {
                      const int32_t a = step > 1 ? part[r] : mine;
                      bool any = false;
                      for (int64_t j = b0 + first; j < e0; j += (int64_t)step * ROW_CHUNK) {
                          int32_t u[ROW_CHUNK], b[ROW_CHUNK];
#pragma unroll
                          for (int q = 0; q < ROW_CHUNK; ++q)
                              u[q] = j + (int64_t)q * step < e0 ? adj[j + (int64_t)q * step] : -1;
#pragma unroll
                          for (int q = 0; q < ROW_CHUNK; ++q) b[q] = u[q] >= 0 ? part[u[q]] : a;
#pragma unroll
                          for (int q = 0; q < ROW_CHUNK; ++q) {
                              any = any || b[q] != a;
                              if (a < b[q] && b[q] < k)
                                  atomicOr(&s_q[a * qw + (b[q] >> 6)], 1ull << (b[q] & 63));
                          }
                      }
                      if (step > 1) any = __ballot(any) != 0 && r == (int32_t)v;
                      out = out || any;
                  });
        if (live && out) atomicAdd(&s_n[mine], 1);
        if (v < n) ext[v] = out ? 1 : 0;
    }
    __syncthreads();
    for (int i = threadIdx.x; i < k * qw; i += blockDim.x)
        if (s_q[i]) atomicOr(&qbits[i], s_q[i]);
    for (int i = threadIdx.x; i < k; i += blockDim.x)
        if (s_n[i]) atomicAdd(&bcnt[i], s_n[i]);
}

// Greedy edge colouring of Q; pairs sorted by colour (ascending (a, b) inside
// a colour) into cpairs, colour c at [col_off[c], col_off[c + 1]).  Then the
// places of the blocks' nodes in their list (blo: k + 1 offsets, bme: where a
// block's marked nodes end; the counts of marked nodes become cursors) and
// an empty list of later boundary nodes.
// The colours are chosen one after the other by one wave with its values in
// scalar registers (one lane with its values in vector registers and LDS took
// 168 us a colouring over the levels of a 2^16-node graph at k = 64, this 118
// us).  A row's colours so far stay in a register and the next
// pair's column is read while the current colour is chosen (the pairs of a
// row have distinct columns), so the chain of a choice is a handful of scalar
// operations.  A colour holds at most one pair of a row, so a bit per (row,
// colour) and a table of columns order the pairs without ranking them.
__global__ void __launch_bounds__(RQ_THREADS)
    ref_colour_k(const unsigned long long *__restrict__ qbits, int32_t k, uint8_t *tab,
                 int32_t *cpairs, int32_t *col_off, const int32_t *bc, int32_t *bcnt, int32_t *blo,
                 int32_t *bme, RefineCtl *ctl) {
    __shared__ unsigned long long s_used[REFINE_K_MAX][REFINE_CW];   // colours at a block
    __shared__ unsigned long long s_low[REFINE_K_MAX][REFINE_CW];    // colours of a row's pairs
    __shared__ unsigned long long s_q[REFINE_K_MAX * REFINE_QW];
    __shared__ int32_t s_ncol;
    __shared__ int32_t sh[RQ_THREADS / WAVE + 1];
    const int qw = (k + 63) / 64;
    for (int i = threadIdx.x; i < k * REFINE_CW; i += blockDim.x) {
        s_used[i / REFINE_CW][i % REFINE_CW] = 0;
        s_low[i / REFINE_CW][i % REFINE_CW] = 0;
    }
    for (int i = threadIdx.x; i < k * qw; i += blockDim.x) s_q[i] = qbits[i];
    __syncthreads();
    if (threadIdx.x < WAVE) {
        auto uni = [](unsigned long long x) {
            return ((unsigned long long)(uint32_t)__builtin_amdgcn_readfirstlane((int32_t)(x >> 32)) << 32) |
                   (uint32_t)__builtin_amdgcn_readfirstlane((int32_t)x);
        };
        const bool w0 = threadIdx.x == 0;
        int32_t ncol = 0;
        for (int32_t a = 0; a < k; ++a) {
            unsigned long long ua = uni(s_used[a][0]);
            for (int w = 0; w < qw; ++w) {
                unsigned long long bits = uni(s_q[a * qw + w]);
                if (!bits) continue;
                int32_t b = w * 64 + __builtin_ctzll(bits);
                bits &= bits - 1;
                unsigned long long ub = s_used[b][0];
                for (;;) {
                    const int32_t bn = bits ? w * 64 + __builtin_ctzll(bits) : -1;
                    unsigned long long un = 0;
                    if (bn >= 0) un = s_used[bn][0];   // not changed by this pair
                    unsigned long long fr = ~(ua | uni(ub));
                    int x = 0;
                    while (!fr && x + 1 < REFINE_CW) {   // the first 64 colours are taken
                        ++x;
                        fr = ~(uni(s_used[a][x]) | uni(s_used[b][x]));
                    }
                    const int32_t cl = x * 64 + __builtin_ctzll(fr);
                    const unsigned long long bit = 1ull << (cl & 63);
                    if (x == 0) ua |= bit;
                    if (w0) {
                        s_used[a][x] |= bit;
                        s_used[b][x] |= bit;
                        s_low[a][x] |= bit;
                        tab[a * REFINE_COLOURS + cl] = (uint8_t)b;
                    }
                    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
                    ncol = cl + 1 > ncol ? cl + 1 : ncol;
                    if (bn < 0) break;
                    b = bn;
                    bits &= bits - 1;
                    ub = un;
                }
            }
        }
        if (w0) s_ncol = ncol;
    }
    __syncthreads();
    const int32_t ncol = s_ncol;
    int32_t base = 0;
    for (int32_t c0 = 0; c0 < ncol; c0 += RQ_THREADS) {   // block-uniform
        const int32_t c = c0 + threadIdx.x;
        const int x = c >> 6;
        const unsigned long long bit = 1ull << (c & 63);
        int32_t cnt = 0;
        if (c < ncol)
            for (int32_t a = 0; a < k; ++a) cnt += (s_low[a][x] & bit) ? 1 : 0;
        int32_t tot;
        int32_t at = base + block_excl_scan(cnt, sh, &tot);
        if (c < ncol) {
            col_off[c] = at;
            for (int32_t a = 0; a < k; ++a)
                if (s_low[a][x] & bit)
                    cpairs[at++] = a | ((int32_t)tab[a * REFINE_COLOURS + c] << 16);
        }
        base += tot;
    }
    const int32_t mine = (int)threadIdx.x < k ? bc[threadIdx.x] : 0;
    int32_t all;
    const int32_t lo = block_excl_scan(mine, sh, &all);
    if ((int)threadIdx.x < k) {
        blo[threadIdx.x] = lo;
        bme[threadIdx.x] = lo + bcnt[threadIdx.x];
        bcnt[threadIdx.x] = lo;
    }
    if (threadIdx.x == 0) {
        blo[k] = all;
        col_off[ncol] = base;
        ctl->ncol = ncol;
        ctl->npairs = base;
        ctl->xn = 0;
    }
}
static_assert(REFINE_K_MAX <= RQ_THREADS && REFINE_K_MAX <= 256, "one thread per block, 8-bit ids");

// The nodes by block, marked ones from the front of a block's places, the
// others from the back (the order decides nothing).  bcnt: front cursors;
// bcnt + k: back cursors, counting up from 0.
__global__ void __launch_bounds__(RQ_THREADS)
    ref_bucket_k(const int32_t *__restrict__ part, const uint16_t *__restrict__ ext, int32_t n,
                 int32_t k, const int32_t *__restrict__ blo, int32_t *bcnt, int32_t *blist) {
    __shared__ int32_t s_cnt[2 * REFINE_K_MAX], s_base[2 * REFINE_K_MAX];
    for (int i = threadIdx.x; i < 2 * k; i += blockDim.x) s_cnt[i] = 0;
    __syncthreads();
    const int64_t lo = (int64_t)blockIdx.x * RQ_THREADS * RB_ITEMS;
    int32_t p[RB_ITEMS], at[RB_ITEMS];
#pragma unroll
    for (int q = 0; q < RB_ITEMS; ++q) {
        const int64_t v = lo + q * RQ_THREADS + threadIdx.x;
        p[q] = -1;
        if (v < n) {
            const int32_t b = part[v];
            if (b >= 0 && b < k) p[q] = b + (ext[v] ? 0 : k);   // others: reported by the weights
        }
    }
#pragma unroll
    for (int q = 0; q < RB_ITEMS; ++q)
        if (p[q] >= 0) at[q] = atomicAdd(&s_cnt[p[q]], 1);
    __syncthreads();
    for (int i = threadIdx.x; i < 2 * k; i += blockDim.x)
        s_base[i] = s_cnt[i] ? atomicAdd(&bcnt[i], s_cnt[i]) : 0;
    __syncthreads();
#pragma unroll
    for (int q = 0; q < RB_ITEMS; ++q) {
        if (p[q] < 0) continue;
        const int32_t at_q = s_base[p[q]] + at[q];
        const int32_t to = p[q] < k ? at_q : blo[p[q] - k + 1] - 1 - at_q;
        if ((uint32_t)to < (uint32_t)n) blist[to] = (int32_t)(lo + q * RQ_THREADS + threadIdx.x);
    }
}

struct FmArgs {
    const int64_t *xadj;
    const int32_t *adj;
    const uint32_t *ew;
    const uint32_t *vw;
    int32_t *part;
    int32_t n, k;
    uint32_t eps_num, eps_den;
    uint64_t seed;
    uint32_t alpha_num, alpha_den;
    int32_t depth, max_local;
    const int32_t *cpairs;
    int64_t *bw, *bd;
    const int32_t *bc_in;   // node counts before this colour
    int32_t *bc_out;        //   and after it
    const int32_t *blo, *bme, *blist;
    int32_t *xlist;
    uint16_t *ext;          // [n] 0: on no list; 1: marked; else listed later, by the launch
    int32_t stamp;          //   of this stamp (unique in the global iteration, above 1)
    // per pair, from the sum of the counts of the pairs before it on: the
    // nodes of the pair or of the search area (bit 31: in block b); where the
    // area is too large for LDS also row lengths, and per run keys
    int32_t *alist, *ldeg;
    uint64_t *key;          // [2][n]
    int32_t *mlog;          // [2][n] moved nodes, local ids
    int32_t *loc;           // [n] -1, or a pair's or area's node: its place in alist (over all
                            //   pairs of the launch, so that places of two pairs differ)
    int2 *lrow;             // [nnz] rows at the nodes' CSR offsets: {local id, weight}; null:
                            //   no memory for them (everything else is in memory then too)
    int32_t acap;           // pairs and areas of at most acap nodes live in LDS (<= FM_AREA)
    int32_t gain_bits;      // 32-bit keys: bits of gain + bias
    RefineCtl *ctl;
};

// weights of blocks and cuts in a search
template <bool WIDE>
using SumOf = std::conditional_t<WIDE, uint64_t, uint32_t>;

// a finished search, published for the adoption
struct RunState {
    int64_t best_imb, best_cut, best_w[2];
    int32_t best_cnt[2], m, kept;
};

// A node's key: its gain (biased, so that it is positive), the high bits of
// its tie hash, its side (bit 2: block b) and its state (bits 0-1: idle,
// queued, or moved; nodes outside the search area count as moved).  Queued
// keys of one side order by gain, then hash; none is 0.  Gains lie within
// the largest weighted degree, so 32 bits take them with at least 12 hash
// bits on most graphs (the caller's choice); 64 bits do where the edge
// weights sum to less than 2^32: gains stay below that in magnitude, which
// leaves 28 hash bits.  WIDE, for sums of 2^32 and more: 64 bits take gains
// below 2^60 and the hash bits that those leave, at the last none.
constexpr int ST_QUEUED = 1, ST_MOVED = 2, ST_SIDE = 4, ST_MASK = 7;
constexpr int KEY32_GAIN_MAX_BITS = 17, KEY64_GAIN_MAX_BITS = 61;
template <class KT, bool WIDE>
struct KeyForm;
template <>
struct KeyForm<uint32_t, false> {
    int shift;        // of the gain
    int64_t bias;
    __device__ explicit KeyForm(int gain_bits) : shift(32 - gain_bits), bias((int64_t)1 << (gain_bits - 1)) {}
    __device__ uint32_t make(int64_t gain, uint64_t h, uint32_t st) const {
        const int hb = shift - 3;
        return ((uint32_t)(gain + bias) << shift) | ((uint32_t)(h >> (64 - hb)) << 3) | st;
    }
    __device__ int64_t gain(uint32_t k) const { return (int64_t)(k >> shift) - bias; }
    __device__ uint32_t step(uint32_t k, int64_t d) const { return k + ((uint32_t)d << shift); }
};
template <>
struct KeyForm<uint64_t, true> {
    int shift;
    int64_t bias;
    __device__ explicit KeyForm(int gain_bits) : shift(64 - gain_bits), bias((int64_t)1 << (gain_bits - 1)) {}
    __device__ uint64_t make(int64_t gain, uint64_t h, uint32_t st) const {
        const int hb = shift - 3;
        return ((uint64_t)(gain + bias) << shift) | (hb > 0 ? h >> (64 - hb) << 3 : 0) | st;
    }
    __device__ int64_t gain(uint64_t k) const { return (int64_t)(k >> shift) - bias; }
    __device__ uint64_t step(uint64_t k, int64_t d) const { return k + ((uint64_t)d << shift); }
};
template <>
struct KeyForm<uint64_t, false> {
    static constexpr int shift = 31;
    static constexpr int64_t bias = (int64_t)1 << 32;
    __device__ explicit KeyForm(int) {}
    __device__ uint64_t make(int64_t gain, uint64_t h, uint32_t st) const {
        return ((uint64_t)(gain + bias) << shift) | (h >> 36 << 3) | st;
    }
    __device__ int64_t gain(uint64_t k) const { return (int64_t)(k >> shift) - bias; }
    __device__ uint64_t step(uint64_t k, int64_t d) const { return k + ((uint64_t)d << shift); }
};

// Row entries on chip: with 32-bit keys a weight is below 2^16 (it is at most
// its node's weighted degree) and a local id below FM_AREA = 2^12, one word;
// otherwise {local id, weight}.
template <class KT>
struct RowForm;
template <>
struct RowForm<uint32_t> {
    using E = uint32_t;
    static __device__ E make(int32_t u, uint32_t w) { return (uint32_t)u | (w << 12); }
    static __device__ int32_t id(E e) { return (int32_t)(e & (FM_AREA - 1)); }
    static __device__ uint32_t w(E e) { return e >> 12; }
};
template <>
struct RowForm<uint64_t> {
    using E = int2;
    static __device__ E make(int32_t u, uint32_t w) { return make_int2(u, (int32_t)w); }
    static __device__ int32_t id(E e) { return e.x; }
    static __device__ uint32_t w(E e) { return (uint32_t)e.y; }
};
static_assert(FM_AREA == 1 << 12, "local ids of a packed row entry");

// LDS of a pair or area of at most `cap` nodes, carved from one block; what
// the nodes leave takes rows.  Keys have FM_PAD empty places behind them, so
// that whole waves read groups without a bound.
constexpr int FM_PAD = WAVE;
constexpr int FM_LDS = 38 * FM_AREA + 16 * FM_PAD + 16;
template <class KT>
struct FmLds {
    uint4 *info;             // row start (in lrow, or in row), row length, c(v), degree in G
    KT *key0, *key1;         // per run
    uint32_t *gid;           // node, bit 31: in block b
    uint16_t *level;         // hops from the boundary inside the block (LV_NONE: not reached),
                             //   bit 15: in block b
    typename RowForm<KT>::E *row;
    int32_t row_cap;         // entries
};
constexpr uint32_t LV_SIDE = 0x8000u, LV_NONE = 0x7fffu;
template <class KT>
__device__ __forceinline__ FmLds<KT> fm_carve(char *p, int32_t cap) {
    FmLds<KT> f;
    f.info = (uint4 *)p;
    f.key0 = (KT *)(f.info + cap);
    f.key1 = f.key0 + cap + FM_PAD;
    f.gid = (uint32_t *)(f.key1 + cap + FM_PAD);
    f.level = (uint16_t *)(f.gid + cap);
    const int32_t used =
        ((22 + 2 * (int)sizeof(KT)) * cap + 2 * (int)sizeof(KT) * FM_PAD + 7) & ~7;
    f.row = (typename RowForm<KT>::E *)(p + used);
    f.row_cap = (FM_LDS - used) / (int)sizeof(typename RowForm<KT>::E);
    return f;
}

// DPP lane moves: after the four row shifts and the broadcast of lane 15 to
// the next row, lanes 31 and 63 hold the maxima of their half-waves.
template <int CTRL, int ROWS>
__device__ __forceinline__ uint32_t dpp_max(uint32_t x) {
    const uint32_t o = (uint32_t)__builtin_amdgcn_update_dpp(0, (int32_t)x, CTRL, ROWS, 0xF, true);
    return o > x ? o : x;
}
__device__ __forceinline__ uint32_t half_max(uint32_t x) {
    x = dpp_max<0x111, 0xF>(x);
    x = dpp_max<0x112, 0xF>(x);
    x = dpp_max<0x114, 0xF>(x);
    x = dpp_max<0x118, 0xF>(x);
    return dpp_max<0x142, 0xA>(x);
}
__device__ __forceinline__ uint32_t lane_u32(uint32_t x, int l) {
    return (uint32_t)__builtin_amdgcn_readlane((int32_t)x, l);
}
// the maxima of the two half-waves (uniform); 64 bits: high words first
__device__ __forceinline__ void half_max2(uint32_t x, uint32_t &m0, uint32_t &m1) {
    const uint32_t m = half_max(x);
    m0 = lane_u32(m, 31);
    m1 = lane_u32(m, 63);
}
__device__ __forceinline__ void half_max2(uint64_t x, uint64_t &m0, uint64_t &m1) {
    const uint32_t hi = (uint32_t)(x >> 32);
    uint32_t h0, h1, l0, l1;
    half_max2(hi, h0, h1);
    half_max2(hi == (lane_id() < 32 ? h0 : h1) ? (uint32_t)x : 0u, l0, l1);
    m0 = ((uint64_t)h0 << 32) | l0;
    m1 = ((uint64_t)h1 << 32) | l1;
}
// the half-wave's maximum in its last lane (31, 63)
__device__ __forceinline__ uint32_t half_top(uint32_t x) { return half_max(x); }
__device__ __forceinline__ uint64_t half_top(uint64_t x) {
    uint64_t m0, m1;
    half_max2(x, m0, m1);
    return lane_id() < 32 ? m0 : m1;
}
__device__ __forceinline__ void lds_max(uint32_t *p, uint32_t v) { atomicMax(p, v); }
__device__ __forceinline__ void lds_max(uint64_t *p, uint64_t v) {
    atomicMax((unsigned long long *)p, (unsigned long long)v);
}

// One local search, on one wave.  A search is a chain of dependent moves, and
// a lone wave issues a dependent instruction every 8 cycles or so: what counts
// is how many instructions a move takes, then the reads on its chain (LDS 64
// cycles, a memory read 300 and more).  The nodes form up to FM_GROUPS groups
// of 2^gsh consecutive local ids; gb holds the best queued key of every side
// and group: a key that grows, or that enters the queue, raises it by an LDS
// maximum, and a group is scanned again only when its best key shrank or was
// moved (two such groups at a time, a half-wave each).  A move then is one
// maximum over the 64 group bests (both sides at once, a half-wave each), the
// search for the winner in its group, and one read of its row, the neighbours'
// state being in LDS: no barrier, and at most one memory access on the chain.
// Equal keys are told apart by the whole hash and the id in a rare second
// pass.  Weights of blocks and cuts fit 32 bits where the sums of all weights do
// (WIDE: 64), and (imbalance, cut) orders as (the heavier block's weight if above L_max
// else 0, cut).  What only the end needs (weights and counts of the best
// state, degrees) is taken from the log of moves afterwards.
// MODE 0: everything in memory; 1: state on chip, rows in memory; 2: rows on
// chip too.  On chip the keys are padded with zeros.
template <class KT, bool WIDE, int MODE>
__device__ __forceinline__ void fm_search(const FmArgs &A, const FmLds<KT> &f, KT *gb, RunState &R,
                                          int r, int32_t off, int32_t N, int32_t qn, int gsh,
                                          uint64_t rseed, int64_t S, int64_t L, SumOf<WIDE> w0,
                                          SumOf<WIDE> w1, int32_t c0, int32_t c1, SumOf<WIDE> cut,
                                          unsigned long long &bytes) {
    constexpr bool CHIP = MODE > 0;
    using Row = RowForm<KT>;
    using W = SumOf<WIDE>;
    const KeyForm<KT, WIDE> kf(A.gain_bits);
    const int lane = lane_id();
    KT *const gkey = (KT *)(A.key + (size_t)r * A.n + off);
    KT *const skey = r ? f.key1 : f.key0;
    int32_t *const mlog = A.mlog + (size_t)r * A.n + off;
    const int32_t *const alist = A.alist + off;
    auto ld_key = [&](int32_t i) { return CHIP ? skey[i] : gkey[i]; };
    // the first node of key M under (hash, id)
    auto first_of = [&](KT M, uint64_t &h, int32_t &v) {
        int32_t at = -1;
        h = 0;
        v = -1;
        for (int32_t i = lane; i < N; i += WAVE) {
            if (ld_key(i) != M) continue;
            const int32_t x = (int32_t)((CHIP ? f.gid[i] : (uint32_t)alist[i]) & 0x7fffffffu);
            const uint64_t hx = mix64(rseed ^ (uint64_t)(uint32_t)x);
            if (at < 0 || hx > h || (hx == h && x < v)) { at = i; h = hx; v = x; }
        }
        for (int o = 1; o < WAVE; o <<= 1) {
            const int32_t at2 = __shfl_xor(at, o), v2 = __shfl_xor(v, o);
            const uint64_t h2 = __shfl_xor(h, o);
            if (at2 >= 0 && (at < 0 || h2 > h || (h2 == h && v2 < v))) { at = at2; h = h2; v = v2; }
        }
        return __builtin_amdgcn_readfirstlane(at);
    };
    const W sw0 = w0, sw1 = w1;
    // since * alpha_den > alpha_num * smaller, S * w > L
    const int32_t patience = (int32_t)min<int64_t>(
        (int64_t)A.alpha_num * min(c0, c1) / (int64_t)A.alpha_den, INT32_MAX);
    const W wmax = (W)min<int64_t>(L / S, WIDE ? INT64_MAX : (int64_t)UINT32_MAX);
    W mx = max(w0, w1), over = mx > wmax ? mx : (W)0;
    W best_over = over, best_cut = cut;
    int32_t m = 0, kept = 0, since = 0;
    uint64_t sum_q = 0;
    for (;;) {
        wave_order();
        const KT K = gb[lane];
        KT M0, M1;
        half_max2(K, M0, M1);
        if ((M0 | M1) == 0) break;
        int from = (M1 >> 3) > (M0 >> 3) ? 1 : 0;     // TopGain (also: one queue is empty)
        int32_t node = -1;
        if (over | ((M0 >> 3) == (M1 >> 3) ? 1u : 0u)) {
            if (over && w0 != w1) {                   // a block is overloaded: MaxLoad
                from = w0 > w1 ? 0 : 1;
                if ((from ? M1 : M0) == 0) from = 1 - from;
            } else if ((M0 >> 3) == (M1 >> 3)) {
                uint64_t ha, hb;
                int32_t va, vb;
                const int32_t na = first_of(M0, ha, va), nb = first_of(M1, hb, vb);
                from = __builtin_amdgcn_readfirstlane(hb > ha || (hb == ha && vb < va) ? 1 : 0);
                node = from ? nb : na;
            }
        }
        const KT M = from ? M1 : M0;
        // the node of key M, in the group whose best it is
        if (node < 0) {
            const uint64_t gm = __ballot(K == M);
            const int32_t i0 = (int32_t)(__builtin_ctzll(gm) & (FM_GROUPS - 1)) << gsh;
            uint64_t many = gm & (gm - 1);
            if (CHIP && gsh <= 6) {
                const uint64_t b = __ballot(ld_key(i0 + lane) == M);
                many |= b & (b - 1);
                node = i0 + (int32_t)__builtin_ctzll(b);
            } else {
                const int32_t i1 = min(N, i0 + (1 << gsh));
                for (int32_t i = i0; i < i1; i += WAVE) {
                    const uint64_t b = __ballot(i + lane < i1 && ld_key(i + lane) == M);
                    if (b == 0) continue;
                    many |= (b & (b - 1)) | (node >= 0 ? 1ull : 0ull);
                    node = i + (int32_t)__builtin_ctzll(b);
                }
            }
            if (many) {   // equal keys
                uint64_t h;
                int32_t v;
                node = first_of(M, h, v);
            }
        }
        int64_t x0;
        int32_t deg;
        uint32_t cv;
        if (CHIP) {
            const uint4 q = f.info[node];
            x0 = (int64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int32_t)q.x);
            deg = __builtin_amdgcn_readfirstlane((int32_t)q.y);
            cv = (uint32_t)__builtin_amdgcn_readfirstlane((int32_t)q.z);
        } else {
            const int32_t v = (int32_t)((uint32_t)alist[node] & 0x7fffffffu);
            x0 = A.xadj[v];
            deg = __builtin_amdgcn_readfirstlane(A.ldeg[off + node]);
            cv = (uint32_t)__builtin_amdgcn_readfirstlane((int32_t)A.vw[v]);
        }
        const typename Row::E *const prow =
            MODE == 2 ? f.row + x0 : (const typename Row::E *)(A.lrow + x0);
        typename Row::E e{};
        int2 e2 = make_int2(0, 0);
        // an entry in memory; without the pair's rows, from the graph's own: a
        // neighbour outside the area becomes {the node itself, 0}
        auto entry = [&](int64_t x) {
            if (A.lrow) return A.lrow[x];
            const int32_t lu = A.loc[A.adj[x]] - off;
            return (uint32_t)lu < (uint32_t)N ? make_int2(lu, (int32_t)A.ew[x]) : make_int2(node, 0);
        };
        if (lane < deg) {   // in flight while the move is booked
            if (CHIP) e = prow[lane];
            else e2 = entry(x0 + lane);
        }
        {   // every lane writes the same
            const KT k = (M & ~(KT)3) | (KT)ST_MOVED;
            if (CHIP) skey[node] = k;
            else gkey[node] = k;
        }
        mlog[m] = node;
        sum_q += (uint32_t)qn;
        ++m;
        const W dw = from ? (W)cv : (W)0 - cv;   // to block a
        w0 += dw;
        w1 -= dw;
        cut -= (W)kf.gain(M);
        mx = max(w0, w1);
        over = mx > wmax ? mx : (W)0;
        ++since;
        if (over < best_over || (over == best_over && cut < best_cut)) {
            best_over = over;
            best_cut = cut;
            kept = m;
            since = 0;
        }
        if (since > patience) break;
        // the neighbours: those on the side left gain 2 w, the others lose it
        int slot_a = from * FM_GROUPS + (node >> gsh);   // the group the moved node left
        --qn;
        for (int32_t t0 = 0;; t0 += WAVE) {
            bool queue = false, dirty = false;
            int slot = 0;
            if (t0 + lane < deg) {
                if (t0 > 0) {
                    if (CHIP) e = prow[t0 + lane];
                    else e2 = entry(x0 + t0 + lane);
                }
                const int32_t u = CHIP ? Row::id(e) : e2.x;
                const KT ku = ld_key(u);
                const int side = (int)(ku >> 2) & 1;
                slot = side * FM_GROUPS + (u >> gsh);
                const KT top = gb[slot];
                const int64_t d = 2 * (int64_t)(CHIP ? Row::w(e) : (uint32_t)e2.y);
                const bool up = side == from, live = !(ku & ST_MOVED);
                const KT k2 = kf.step(ku, up ? d : -d) | (KT)ST_QUEUED;
                queue = live && !(ku & ST_QUEUED);
                const bool rise = live && (queue || up);
                dirty = live && !rise && top == ku;
                if (live) {
                    if (CHIP) skey[u] = k2;
                    else gkey[u] = k2;
                }
                if (rise) lds_max(&gb[slot], k2);
            }
            qn += (int32_t)__popcll(__ballot(queue));
            wave_order();
            // groups to scan again, two at a time
            uint64_t dm = __ballot(dirty);
            for (;;) {
                int sa = slot_a, sb = -1;
                if (sa < 0) {
                    if (dm == 0) break;
                    sa = (int)lane_u32((uint32_t)slot, __builtin_ctzll(dm));
                }
                slot_a = -1;
                if (dm) {
                    dm &= ~__ballot(slot == sa);
                    if (dm) {
                        sb = (int)lane_u32((uint32_t)slot, __builtin_ctzll(dm));
                        dm &= ~__ballot(slot == sb);
                    }
                }
                const int sl = lane < 32 ? sa : (sb < 0 ? sa : sb);
                const uint32_t want = (uint32_t)(ST_QUEUED | (sl >= FM_GROUPS ? ST_SIDE : 0));
                const int32_t i0 = (sl & (FM_GROUPS - 1)) << gsh;
                KT top = 0;
                auto offer = [&](KT x) {
                    if (((uint32_t)x & ST_MASK) == want && x > top) top = x;
                };
                if (CHIP && gsh <= 6) {
                    offer(ld_key(i0 + (lane & 31)));
                    if (gsh == 6) offer(ld_key(i0 + 32 + (lane & 31)));
                } else {
                    const int32_t i1 = min(N, i0 + (1 << gsh));
                    for (int32_t i = i0 + (lane & 31); i < i1; i += 32) offer(ld_key(i));
                }
                top = half_top(top);
                if ((lane & 31) == 31) gb[sl] = top;
            }
            if (t0 + WAVE >= deg) break;
            wave_order();
        }
    }
    // the best state's weights and counts, and the degrees moved, from the log
    // (a moved node's key keeps the side it left)
    uint64_t sum_d = 0;
    W out_w = 0, in_w = 0;   // weights kept moves took out of blocks a and b
    int32_t out_n = 0, in_n = 0;
    for (int32_t t = lane; t < m; t += WAVE) {
        const int32_t i = mlog[t];
        const bool side = (ld_key(i) & ST_SIDE) != 0;
        uint32_t cv, fd;
        if (CHIP) {
            const uint4 q = f.info[i];
            cv = q.z;
            fd = q.w;
        } else {
            const int32_t v = (int32_t)((uint32_t)alist[i] & 0x7fffffffu);
            cv = A.vw[v];
            fd = (uint32_t)(A.xadj[v + 1] - A.xadj[v]);
        }
        sum_d += fd;
        if (t >= kept) continue;
        if (side) { in_w += cv; ++in_n; }
        else { out_w += cv; ++out_n; }
    }
    sum_d = wave_sum(sum_d);
    out_w = wave_sum(out_w);
    in_w = wave_sum(in_w);
    out_n = wave_sum(out_n);
    in_n = wave_sum(in_n);
    bytes = 17 * sum_q + 25 * sum_d;
    if (lane == 0) {
        R.best_w[0] = (int64_t)(W)(sw0 - out_w + in_w);
        R.best_w[1] = (int64_t)(W)(sw1 + out_w - in_w);
        R.best_imb = pair_imb(R.best_w[0], R.best_w[1], S, L);
        R.best_cut = (int64_t)best_cut;
        R.best_cnt[0] = c0 - out_n + in_n;
        R.best_cnt[1] = c1 + out_n - in_n;
        R.kept = kept;
        R.m = m;
    }
}

// The pairs of one colour, a workgroup each.  A launch lasts as long as its
// slowest pair, a pair as long as its chain of moves, so the chip is mostly
// idle and nothing here is bound by bandwidth.  Measured (MI355X, preset fast):
// random geometric graph of 2^18 + 1 nodes, k = 16: 504 -> 82 ms, a step of
// both searches' moves 6.0 -> 1.0 us (before: queue entries of 24-byte keys
// reduced by eight waves with three block barriers per move, the neighbours'
// state gathered from memory); way back up of one of 2^16 nodes, k = 64: 311 ->
// 113 ms, preparation of a pair's searches 41 -> 25 us.  512 threads: with 1024
// the search spills (1.26 us per step).
template <class KT, bool WIDE>
__global__ void __launch_bounds__(FM_THREADS)
    ref_fm_k(FmArgs A, int32_t gi, int32_t p0, int32_t np) {
    using Row = RowForm<KT>;
    __shared__ __align__(16) char s_mem[FM_LDS];
    __shared__ KT s_gb[2][2 * FM_GROUPS];   // best queued key per (side, group); 0: none
    __shared__ int32_t s_grew[2];
    __shared__ RunState rs[2];
    __shared__ int32_t s_off, s_cnt, s_rows, s_stop, s_pick, s_bc[2];
    __shared__ int64_t s_bw[2], s_bd[2];
    __shared__ unsigned long long s_cut, s_bytes;
    // entries of the later list: other pairs of the launch append to it, so
    // that one thread reads the count and the block takes its value (the loops
    // over the list hold barriers).  Entries of those pairs are none of this
    // one's, its own are counted by the next local iteration.
    __shared__ unsigned long long s_xn;
    __shared__ uint8_t s_in[REFINE_K_MAX];
    const KeyForm<KT, WIDE> kf(A.gain_bits);
    const int32_t j = blockIdx.x;
    const int32_t ab = A.cpairs[p0 + j], a = ab & 0xffff, b = ab >> 16;
    const int tid = threadIdx.x, wv = tid / WAVE, gl = tid % RG_LANES, grp = tid / RG_LANES;
    const int32_t la = A.blo[a], lb = A.blo[b];
    auto later_count = [&]() {
        return __hip_atomic_load(&A.ctl->xn, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    };
    if (tid == 0) {
        s_xn = later_count();
        s_bytes = 0;
        s_off = 0;
        s_rows = 0;
        s_cnt = 0;
        s_bc[0] = A.bc_in[a];
        s_bc[1] = A.bc_in[b];
        s_bw[0] = A.bw[a];
        s_bw[1] = A.bw[b];
        s_bd[0] = A.bd[a];
        s_bd[1] = A.bd[b];
    }
    for (int i = tid; i < A.k; i += FM_THREADS) s_in[i] = 0;
    __syncthreads();
    // the pair's arrays start after those of the pairs before it; the counts
    // of blocks in no pair of this colour carry over
    for (int i = tid; i < np; i += FM_THREADS) {
        const int32_t q = A.cpairs[p0 + i], pa = q & 0xffff, pb = q >> 16;
        if (i < j) atomicAdd(&s_off, A.bc_in[pa] + A.bc_in[pb]);
        s_in[pa] = 1;
        s_in[pb] = 1;
    }
    __syncthreads();
    if (j == 0)
        for (int i = tid; i < A.k; i += FM_THREADS)
            if (!s_in[i]) A.bc_out[i] = A.bc_in[i];
    const int32_t off = s_off, len = s_bc[0] + s_bc[1];
    if ((int64_t)off + len > A.n) {   // the counts are not those of part
        if (tid == 0) atomicOr(&A.ctl->flags, 2u);
        return;
    }
    const int64_t S = (int64_t)A.k * A.eps_den;
    const int64_t L = ((int64_t)A.eps_den + A.eps_num) * (int64_t)A.ctl->total +
                      S * (int64_t)A.ctl->max_node;
    int32_t *const alist = A.alist + off;
    // a small pair is read once and stays on chip; the lists name all its
    // nodes.  Of a larger pair only the marked nodes are read.
    const bool whole = len <= A.acap;
    const int32_t na = (whole ? A.blo[a + 1] : A.bme[a]) - la,
                  nb = (whole ? A.blo[b + 1] : A.bme[b]) - lb;
    const FmLds<KT> f = fm_carve<KT>(s_mem, whole ? len : FM_AREA);
    const bool chip_rows = whole && s_bd[0] + s_bd[1] <= f.row_cap;
    // a row in memory starts at its node's CSR offset in 8-byte slots, whatever
    // the entries' size: pairs of one launch may differ in it
    auto mrow = [&](int64_t x) { return (typename Row::E *)(A.lrow + x); };
    unsigned long long ticks_init = 0, ticks_moves = 0, t0 = 0;
    if (tid == 0) t0 = wall_clock64();
    if (whole) {
        // the pair's nodes: those of the blocks' lists that are still in the
        // pair (a node is on one of them once), then those of the later list
        // not found yet (a moved node may be there several times).  A node's
        // place is kept with the pair's offset, so that places of different
        // pairs differ and a place says whether a node is in this pair.
        auto put = [&](bool in, int32_t v, int32_t pv, int64_t x0, int64_t x1, uint32_t c) {
            const int32_t pos = wave_places(in, &s_cnt);
            if (!in || pos >= len) return;   // valid lists never exceed len
            const uint32_t id = (uint32_t)v | (pv == b ? 0x80000000u : 0u);
            alist[pos] = (int32_t)id;
            A.loc[v] = off + pos;
            f.gid[pos] = id;
            f.info[pos] = make_uint4((uint32_t)x0, 0u, c, (uint32_t)(x1 - x0));
        };
        const unsigned long long xn = s_xn;
        const bool every = xn > (unsigned long long)A.n;   // the later list overflowed
        for (int32_t b0 = 0; b0 < na + nb; b0 += FM_THREADS * FM_ENT) {   // block-uniform
            int32_t v[FM_ENT], pv[FM_ENT];
            int64_t x0[FM_ENT], x1[FM_ENT];
            uint32_t c[FM_ENT];
#pragma unroll
            for (int z = 0; z < FM_ENT; ++z) {
                const int32_t i = b0 + z * FM_THREADS + tid;
                v[z] = i < na + nb ? A.blist[i < na ? la + i : lb + (i - na)] : -1;
            }
#pragma unroll
            for (int z = 0; z < FM_ENT; ++z) {
                const bool in = v[z] >= 0;
                pv[z] = in ? A.part[v[z]] : -1;
                x0[z] = in ? A.xadj[v[z]] : 0;
                x1[z] = in ? A.xadj[v[z] + 1] : 0;
                c[z] = in ? A.vw[v[z]] : 0u;
            }
#pragma unroll
            for (int z = 0; z < FM_ENT; ++z)
                put(pv[z] >= 0 && (pv[z] == a || pv[z] == b), v[z], pv[z], x0[z], x1[z], c[z]);
        }
        __syncthreads();
        const int64_t more = s_cnt == len ? 0 : (every ? A.n : (int64_t)xn);
        __syncthreads();   // every thread has read the count before it grows
        for (int64_t b0 = 0; b0 < more; b0 += FM_THREADS) {   // block-uniform
            const int64_t i = b0 + tid;
            const int32_t v = i < more ? (every ? (int32_t)i : A.xlist[i]) : -1;
            const int32_t pv = v >= 0 ? A.part[v] : -1;
            const bool in = v >= 0 && (pv == a || pv == b) && A.loc[v] == -1 &&
                            atomicCAS(&A.loc[v], -1, -2) == -1;
            put(in, v, pv, in ? A.xadj[v] : 0, in ? A.xadj[v + 1] : 0, in ? A.vw[v] : 0u);
        }
        __syncthreads();
        if (s_cnt != len) {   // the lists are not those of part
            if (tid == 0) atomicOr(&A.ctl->flags, 2u);
            return;
        }
        // Rows: an entry inside the pair becomes {local id, weight}, another one
        // {the node itself, 0}, which changes nothing in a search (the node has
        // moved by then) and is on the node's own side for the others.  On chip:
        // places are taken per node and filled with the node's local id, then
        // every entry is replaced by a thread of its own.
        if (chip_rows) {
            for (int32_t b0 = 0; b0 < len; b0 += FM_THREADS) {   // block-uniform
                const int32_t i = b0 + tid;
                const uint4 q = i < len ? f.info[i] : make_uint4(0u, 0u, 0u, 0u);
                uint32_t inc = wave_incl_scan(q.w);
                int32_t base = 0;
                if (lane_id() == WAVE - 1) base = atomicAdd(&s_rows, (int32_t)inc);
                const uint32_t at = (uint32_t)__shfl(base, WAVE - 1) + inc - q.w;
                for (uint32_t e = 0; e < q.w; ++e) f.row[at + e] = Row::make(i, 0u);
                if (i < len) {
                    f.info[i].y = at;   // x: the row's CSR offset, until the entries are in
                    f.info[i].x = q.x;
                }
            }
            __syncthreads();
            const int32_t ne = s_rows;
            for (int32_t b0 = 0; b0 < ne; b0 += FM_THREADS * FM_ENT) {   // block-uniform
                int32_t own[FM_ENT], u[FM_ENT], lu[FM_ENT];
                uint32_t w[FM_ENT];
#pragma unroll
                for (int z = 0; z < FM_ENT; ++z) {
                    const int32_t e = b0 + z * FM_THREADS + tid;
                    own[z] = e < ne ? Row::id(f.row[e]) : -1;
                }
#pragma unroll
                for (int z = 0; z < FM_ENT; ++z) {
                    u[z] = -1;
                    w[z] = 0;
                    if (own[z] < 0) continue;
                    const uint4 q = f.info[own[z]];
                    const size_t at = (size_t)q.x + (uint32_t)(b0 + z * FM_THREADS + tid) - q.y;
                    u[z] = A.adj[at];
                    w[z] = A.ew[at];
                }
#pragma unroll
                for (int z = 0; z < FM_ENT; ++z) lu[z] = u[z] >= 0 ? A.loc[u[z]] - off : -1;
#pragma unroll
                for (int z = 0; z < FM_ENT; ++z)
                    if ((uint32_t)lu[z] < (uint32_t)len)
                        f.row[b0 + z * FM_THREADS + tid] = Row::make(lu[z], w[z]);
            }
            __syncthreads();
            for (int32_t i = tid; i < len; i += FM_THREADS) {
                const uint4 q = f.info[i];
                f.info[i] = make_uint4(q.y, q.w, q.z, q.w);
            }
        } else {
            for (int32_t b0 = 0; b0 < len; b0 += RG_ROWS) {   // block-uniform
                uint32_t x0[RG_U], dg[RG_U];
#pragma unroll
                for (int z = 0; z < RG_U; ++z) {
                    const int32_t i = b0 + z * RG_GROUPS + grp;
                    x0[z] = dg[z] = 0;
                    if (i < len) {
                        x0[z] = f.info[i].x;
                        dg[z] = f.info[i].w;
                    }
                }
                for (uint32_t j0 = 0;; j0 += RG_LANES) {
                    bool more_rows = false;
#pragma unroll
                    for (int z = 0; z < RG_U; ++z) more_rows = more_rows || j0 < dg[z];
                    if (!__any(more_rows)) break;   // wave-uniform
                    int32_t u[RG_U], lu[RG_U];
                    uint32_t w[RG_U];
#pragma unroll
                    for (int z = 0; z < RG_U; ++z) {
                        const bool in = j0 + gl < dg[z];
                        u[z] = in ? A.adj[(size_t)x0[z] + j0 + gl] : -1;
                        w[z] = in ? A.ew[(size_t)x0[z] + j0 + gl] : 0u;
                    }
#pragma unroll
                    for (int z = 0; z < RG_U; ++z) lu[z] = u[z] >= 0 ? A.loc[u[z]] - off : -1;
#pragma unroll
                    for (int z = 0; z < RG_U; ++z)
                        if (j0 + gl < dg[z])
                            mrow(x0[z])[j0 + gl] =
                                (uint32_t)lu[z] < (uint32_t)len
                                    ? Row::make(lu[z], w[z])
                                    : Row::make(b0 + z * RG_GROUPS + grp, 0u);
                }
#pragma unroll
                for (int z = 0; z < RG_U; ++z) {
                    const int32_t i = b0 + z * RG_GROUPS + grp;
                    if (i < len && gl == 0) f.info[i].y = dg[z];
                }
            }
        }
        __syncthreads();
    }
    int gsh = 5;
    for (int32_t t = 0; t < A.max_local; ++t) {
        if (tid == 0) {
            s_cut = 0;
            s_cnt = 0;
            s_xn = later_count();
            if (t > 0) t0 = wall_clock64();
            s_bytes += 40ull * (unsigned)len + 12ull * (unsigned long long)(s_bd[0] + s_bd[1]);
        }
        for (int i = tid; i < 2 * 2 * FM_GROUPS; i += FM_THREADS) s_gb[i >> 6][i & 63] = 0;
        if (tid < 2) s_grew[tid] = 0;
        __syncthreads();
        const uint64_t rs0 = run_seed_of(A.seed, gi, a, b, t, 0);
        const uint64_t rs1 = run_seed_of(A.seed, gi, a, b, t, 1);
        unsigned long long cut = 0;
        int32_t N, n0;
        bool chip;
        gsh = 5;
        if (whole) {
            N = len;
            chip = true;
            while ((FM_GROUPS << gsh) < N) ++gsh;
            // gains, keys, the boundary and the first group bests
            for (int32_t i = N + tid; i < N + FM_PAD; i += FM_THREADS) f.key0[i] = f.key1[i] = 0;
            int32_t n_bnd = 0;
            for (int32_t i = tid; i < N; i += FM_THREADS) {
                const uint32_t id = f.gid[i];
                const uint32_t side = id >> 31;
                const uint4 inf = f.info[i];
                int64_t gain = 0;
                bool bnd = false;
                for (uint32_t e0 = 0; e0 < inf.y; e0 += ROW_CHUNK) {
                    typename Row::E e[ROW_CHUNK];
                    uint32_t g[ROW_CHUNK];
#pragma unroll
                    for (int q = 0; q < ROW_CHUNK; ++q)
                        e[q] = e0 + q < inf.y ? (chip_rows ? f.row[inf.x + e0 + q] : mrow(inf.x)[e0 + q])
                                              : Row::make(i, 0u);
#pragma unroll
                    for (int q = 0; q < ROW_CHUNK; ++q) g[q] = f.gid[Row::id(e[q])] >> 31;
#pragma unroll
                    for (int q = 0; q < ROW_CHUNK; ++q) {
                        const uint32_t w = Row::w(e[q]);
                        const bool other = g[q] != side;
                        bnd = bnd || other;
                        gain += other ? (int64_t)w : -(int64_t)w;
                        if (other && side == 0) cut += w;
                    }
                }
                const uint64_t v = id & 0x7fffffffu;
                const uint32_t st = (bnd ? ST_QUEUED : ST_MOVED) | (side ? ST_SIDE : 0);
                const KT k0 = kf.make(gain, mix64(rs0 ^ v), st), k1 = kf.make(gain, mix64(rs1 ^ v), st);
                f.key0[i] = k0;
                f.key1[i] = k1;
                f.level[i] = (uint16_t)((bnd ? 0u : LV_NONE) | (side ? LV_SIDE : 0u));
                if (bnd) {
                    ++n_bnd;
                    const int slot = (int)side * FM_GROUPS + (i >> gsh);
                    lds_max(&s_gb[0][slot], k0);
                    lds_max(&s_gb[1][slot], k1);
                }
            }
            n_bnd = wave_sum(n_bnd);
            if (lane_id() == 0 && n_bnd) atomicAdd(&s_cnt, n_bnd);
            __syncthreads();
            n0 = s_cnt;
            // bounded BFS inside each block: nodes within `depth` hops enter the
            // area, the others keep the state of a moved node.  Every node not
            // reached yet looks at its neighbours' levels: a few instructions per
            // entry, where pushing a frontier takes dozens (marks, places, lists).
            for (int32_t d = 1; d <= A.depth; ++d) {
                bool grew = false;
                for (int32_t i = tid; i < N; i += FM_THREADS) {
                    const uint32_t lv = f.level[i];
                    if ((lv & LV_NONE) != LV_NONE) continue;
                    const uint4 inf = f.info[i];
                    const uint32_t sb = lv & LV_SIDE;
                    uint32_t low = 0xffffu;   // levels of the other side lie above
                    for (uint32_t e0 = 0; e0 < inf.y; e0 += ROW_CHUNK) {
                        int32_t u[ROW_CHUNK];
#pragma unroll
                        for (int q = 0; q < ROW_CHUNK; ++q)
                            u[q] = e0 + q < inf.y ? Row::id(chip_rows ? f.row[inf.x + e0 + q]
                                                                      : mrow(inf.x)[e0 + q])
                                                  : i;
#pragma unroll
                        for (int q = 0; q < ROW_CHUNK; ++q)
                            low = min(low, (uint32_t)f.level[u[q]] ^ sb);
                    }
                    if (low < (uint32_t)d) {   // a neighbour on its side, d - 1 hops away
                        f.level[i] = (uint16_t)((uint32_t)d | sb);
                        f.key0[i] &= ~(KT)ST_MOVED;   // idle
                        f.key1[i] &= ~(KT)ST_MOVED;
                        grew = true;
                    }
                }
                if (__any(grew) && lane_id() == 0) s_grew[d & 1] = 1;
                __syncthreads();
                const bool go = s_grew[d & 1] != 0;
                if (tid == 0) s_grew[(d + 1) & 1] = 0;
                __syncthreads();
                if (!go) break;
            }
        } else {
            // the boundary, from the marked nodes and the later list, each once.
            // Area nodes below FM_AREA keep {id, degree, row start} on chip (where
            // their final record goes) for the next step.
            uint4 *const rec = (uint4 *)s_mem, *const cand = rec + FM_AREA;
            static_assert((FM_AREA + FM_TILE) * 16 <= FM_LDS, "records and tile fit the block");
            auto record = [&](int32_t i, uint32_t &id, int64_t &x0, uint32_t &dg) {
                if (i < FM_AREA) {
                    const uint4 q = rec[i];
                    id = q.x;
                    dg = q.y;
                    x0 = (int64_t)(((uint64_t)q.w << 32) | q.z);
                } else {
                    id = (uint32_t)alist[i];
                    const int32_t v = (int32_t)(id & 0x7fffffffu);
                    x0 = A.xadj[v];
                    dg = (uint32_t)(A.xadj[v + 1] - x0);
                }
            };
            auto enter = [&](bool in, uint32_t id, int64_t x0, uint32_t dg) {
                const int32_t pos = wave_places(in, &s_cnt);
                if (!in || pos >= len) return;   // too many: flagged below
                alist[pos] = (int32_t)id;
                if (pos < FM_AREA)
                    rec[pos] = make_uint4(id, dg, (uint32_t)x0, (uint32_t)((uint64_t)x0 >> 32));
            };
            const unsigned long long xn = s_xn;
            const bool every = xn > (unsigned long long)A.n;   // the later list overflowed
            const int64_t total = every ? A.n : (int64_t)na + nb + (int64_t)xn;
            for (int64_t t1 = 0; t1 < total; t1 += FM_TILE) {   // block-uniform
                if (tid == 0) s_rows = 0;
                __syncthreads();
                static_assert(FM_TILE == FM_THREADS * FM_ENT, "one pass per tile");
                int32_t v[FM_ENT], pv[FM_ENT];
                int64_t x0[FM_ENT], x1[FM_ENT];
#pragma unroll
                for (int z = 0; z < FM_ENT; ++z) {
                    const int64_t i = t1 + z * FM_THREADS + tid;
                    v[z] = i >= total ? -1
                         : every ? (int32_t)i
                         : i < na ? A.blist[la + i]
                         : i < (int64_t)na + nb ? A.blist[lb + (i - na)] : A.xlist[i - na - nb];
                }
#pragma unroll
                for (int z = 0; z < FM_ENT; ++z) pv[z] = v[z] >= 0 ? A.part[v[z]] : -1;
#pragma unroll
                for (int z = 0; z < FM_ENT; ++z) {
                    const bool in = v[z] >= 0 && (pv[z] == a || pv[z] == b);
                    x0[z] = in ? A.xadj[v[z]] : 0;
                    x1[z] = in ? A.xadj[v[z] + 1] : 0;
                }
#pragma unroll
                for (int z = 0; z < FM_ENT; ++z) {
                    const bool in = x1[z] > x0[z];
                    const int32_t at = wave_places(in, &s_rows);
                    if (in)
                        cand[at] = make_uint4((uint32_t)v[z] | (pv[z] == b ? 0x80000000u : 0u),
                                              (uint32_t)(x1[z] - x0[z]), (uint32_t)x0[z],
                                              (uint32_t)((uint64_t)x0[z] >> 32));
                }
                __syncthreads();
                const int32_t nc = s_rows;
                for (int32_t b0 = 0; b0 < nc; b0 += RG_ROWS) {   // block-uniform
                    uint4 q[RG_U];
                    uint32_t bnd[RG_U], dg[RG_U];
#pragma unroll
                    for (int z = 0; z < RG_U; ++z) {
                        const int32_t i = b0 + z * RG_GROUPS + grp;
                        q[z] = i < nc ? cand[i] : make_uint4(0u, 0u, 0u, 0u);
                        dg[z] = q[z].y;
                        bnd[z] = 0;
                    }
                    for (uint32_t j0 = 0;; j0 += RG_LANES) {
                        bool more_rows = false;
#pragma unroll
                        for (int z = 0; z < RG_U; ++z) more_rows = more_rows || j0 < dg[z];
                        if (!__any(more_rows)) break;   // wave-uniform
                        int32_t u[RG_U], pu[RG_U];
#pragma unroll
                        for (int z = 0; z < RG_U; ++z) {
                            const int64_t r0 = (int64_t)(((uint64_t)q[z].w << 32) | q[z].z);
                            u[z] = j0 + gl < dg[z] ? A.adj[r0 + j0 + gl] : -1;
                        }
#pragma unroll
                        for (int z = 0; z < RG_U; ++z) pu[z] = u[z] >= 0 ? A.part[u[z]] : -1;
#pragma unroll
                        for (int z = 0; z < RG_U; ++z) {
                            bnd[z] |= group_ballot(pu[z] == ((q[z].x >> 31) ? a : b));
                            if (bnd[z]) dg[z] = 0;
                        }
                    }
                    bool in[RG_U];
#pragma unroll
                    for (int z = 0; z < RG_U; ++z)
                        in[z] = bnd[z] && gl == 0 &&
                                atomicCAS(&A.loc[q[z].x & 0x7fffffffu], -1, -2) == -1;
#pragma unroll
                    for (int z = 0; z < RG_U; ++z)
                        enter(in[z], q[z].x, (int64_t)(((uint64_t)q[z].w << 32) | q[z].z), q[z].y);
                }
                __syncthreads();
            }
            __syncthreads();
            n0 = s_cnt;
            // bounded BFS inside each block, one frontier per distance
            int32_t f0 = 0, f1 = n0;
            __syncthreads();   // every thread has read the count before it grows
            for (int32_t d = 1; d <= A.depth && f0 < f1 && f1 <= len; ++d) {
                for (int32_t b0 = f0; b0 < f1; b0 += RG_ROWS) {   // block-uniform
                    uint32_t id[RG_U], dg[RG_U];
                    int64_t x0[RG_U];
#pragma unroll
                    for (int z = 0; z < RG_U; ++z) {
                        const int32_t i = b0 + z * RG_GROUPS + grp;
                        id[z] = dg[z] = 0;
                        x0[z] = 0;
                        if (i < f1) record(i, id[z], x0[z], dg[z]);
                    }
                    for (uint32_t j0 = 0;; j0 += RG_LANES) {
                        bool more_rows = false;
#pragma unroll
                        for (int z = 0; z < RG_U; ++z) more_rows = more_rows || j0 < dg[z];
                        if (!__any(more_rows)) break;   // wave-uniform
                        int32_t u[RG_U], pu[RG_U], lu[RG_U];
                        int64_t y0[RG_U], y1[RG_U];
#pragma unroll
                        for (int z = 0; z < RG_U; ++z)
                            u[z] = j0 + gl < dg[z] ? A.adj[x0[z] + j0 + gl] : -1;
#pragma unroll
                        for (int z = 0; z < RG_U; ++z) {
                            const bool in = u[z] >= 0;
                            pu[z] = in ? A.part[u[z]] : -1;
                            lu[z] = in ? A.loc[u[z]] : 0;
                            y0[z] = in ? A.xadj[u[z]] : 0;
                            y1[z] = in ? A.xadj[u[z] + 1] : 0;
                        }
#pragma unroll
                        for (int z = 0; z < RG_U; ++z) {
                            const int32_t pv = (id[z] >> 31) ? b : a;
                            lu[z] = pu[z] == pv && lu[z] == -1 ? atomicCAS(&A.loc[u[z]], -1, -2) : 0;
                        }
#pragma unroll
                        for (int z = 0; z < RG_U; ++z)
                            enter(lu[z] == -1, (uint32_t)u[z] | (id[z] & 0x80000000u), y0[z],
                                  (uint32_t)(y1[z] - y0[z]));
                    }
                }
                __syncthreads();
                f0 = f1;
                f1 = s_cnt;
                __syncthreads();   // every thread has read the count before it grows
            }
            N = f1;
            if (N > len) {   // more area nodes than the blocks hold: broken state
                if (tid == 0) atomicOr(&A.ctl->flags, 2u);
                return;
            }
            for (int32_t i = tid; i < N; i += FM_THREADS)
                A.loc[(uint32_t)alist[i] & 0x7fffffffu] = off + i;
            __syncthreads();
            // rows inside the area, gains, keys and the first group bests; the
            // queues start with the boundary
            chip = N <= A.acap;
            while (((int64_t)FM_GROUPS << gsh) < N) ++gsh;
            if (chip)
                for (int32_t i = N + tid; i < N + FM_PAD; i += FM_THREADS) f.key0[i] = f.key1[i] = 0;
            for (int32_t b0 = 0; b0 < N; b0 += RG_ROWS) {   // block-uniform
                uint32_t id[RG_U], cv[RG_U], deg[RG_U], dg[RG_U];
                int64_t x0[RG_U], gain[RG_U];
#pragma unroll
                for (int z = 0; z < RG_U; ++z) {
                    const int32_t i = b0 + z * RG_GROUPS + grp;
                    id[z] = dg[z] = deg[z] = 0;
                    x0[z] = gain[z] = 0;
                    if (i < N) record(i, id[z], x0[z], dg[z]);
                }
#pragma unroll
                for (int z = 0; z < RG_U; ++z)
                    cv[z] = b0 + z * RG_GROUPS + grp < N ? A.vw[id[z] & 0x7fffffffu] : 0u;
                for (uint32_t j0 = 0;; j0 += RG_LANES) {
                    bool more_rows = false;
#pragma unroll
                    for (int z = 0; z < RG_U; ++z) more_rows = more_rows || j0 < dg[z];
                    if (!__any(more_rows)) break;   // wave-uniform
                    int32_t u[RG_U], pu[RG_U], lu[RG_U];
                    uint32_t w[RG_U];
#pragma unroll
                    for (int z = 0; z < RG_U; ++z) {
                        const bool in = j0 + gl < dg[z];
                        u[z] = in ? A.adj[x0[z] + j0 + gl] : -1;
                        w[z] = in ? A.ew[x0[z] + j0 + gl] : 0u;
                    }
#pragma unroll
                    for (int z = 0; z < RG_U; ++z) {
                        pu[z] = u[z] >= 0 ? A.part[u[z]] : -1;
                        lu[z] = u[z] >= 0 ? A.loc[u[z]] - off : -1;
                    }
#pragma unroll
                    for (int z = 0; z < RG_U; ++z) {
                        const bool in_b = (id[z] >> 31) != 0;
                        const bool own = pu[z] == (in_b ? b : a), oth = pu[z] == (in_b ? a : b);
                        gain[z] += oth ? (int64_t)w[z] : (own ? -(int64_t)w[z] : 0);
                        if (oth && !in_b) cut += w[z];
                        const bool in = (own || oth) && (uint32_t)lu[z] < (uint32_t)N;   // in the area
                        const uint32_t m = group_ballot(in);
                        if (in) {
                            const uint32_t to = deg[z] + __popc(m & ((1u << gl) - 1u));
                            if (chip) mrow(x0[z])[to] = Row::make(lu[z], w[z]);
                            else if (A.lrow) A.lrow[x0[z] + to] = make_int2(lu[z], (int32_t)w[z]);
                        }
                        deg[z] += __popc(m);
                    }
                }
#pragma unroll
                for (int z = 0; z < RG_U; ++z) {
                    for (int o = RG_LANES / 2; o > 0; o >>= 1)
                        gain[z] += __shfl_xor(gain[z], o, RG_LANES);
                    const int32_t i = b0 + z * RG_GROUPS + grp;
                    if (i >= N || gl != 0) continue;
                    const uint64_t v = id[z] & 0x7fffffffu;
                    const int side = (int)(id[z] >> 31);
                    const uint32_t st = (i < n0 ? ST_QUEUED : 0) | (side ? ST_SIDE : 0);
                    const KT k0 = kf.make(gain[z], mix64(rs0 ^ v), st);
                    const KT k1 = kf.make(gain[z], mix64(rs1 ^ v), st);
                    if (chip) {   // info[i] takes the place of rec[i]
                        f.gid[i] = id[z];
                        f.info[i] = make_uint4((uint32_t)x0[z], deg[z], cv[z], dg[z]);
                        f.key0[i] = k0;
                        f.key1[i] = k1;
                    } else {
                        A.ldeg[off + i] = (int32_t)(A.lrow ? deg[z] : dg[z]);
                        ((KT *)(A.key + off))[i] = k0;
                        ((KT *)(A.key + (size_t)A.n + off))[i] = k1;
                    }
                    if (i < n0) {
                        const int slot = side * FM_GROUPS + (i >> gsh);
                        lds_max(&s_gb[0][slot], k0);
                        lds_max(&s_gb[1][slot], k1);
                    }
                }
            }
        }
        cut = wave_sum(cut);
        if (lane_id() == 0 && cut) atomicAdd(&s_cut, cut);
        __syncthreads();
        const int64_t start_cut = (int64_t)s_cut;
        const int64_t start_imb = pair_imb(s_bw[0], s_bw[1], S, L);
        if (tid == 0) {
            const unsigned long long t1 = wall_clock64();
            ticks_init += t1 - t0;
            t0 = t1;
        }
        if (wv < 2) {
            unsigned long long bytes = 0;
            const uint64_t seed = wv ? rs1 : rs0;
            using W = SumOf<WIDE>;
            const W w0 = (W)s_bw[0], w1 = (W)s_bw[1], c = (W)start_cut;
            if (chip_rows)
                fm_search<KT, WIDE, 2>(A, f, s_gb[wv], rs[wv], wv, off, N, n0, gsh, seed, S, L, w0,
                                       w1, s_bc[0], s_bc[1], c, bytes);
            else if (chip)
                fm_search<KT, WIDE, 1>(A, f, s_gb[wv], rs[wv], wv, off, N, n0, gsh, seed, S, L, w0,
                                       w1, s_bc[0], s_bc[1], c, bytes);
            else
                fm_search<KT, WIDE, 0>(A, f, s_gb[wv], rs[wv], wv, off, N, n0, gsh, seed, S, L, w0,
                                       w1, s_bc[0], s_bc[1], c, bytes);
            if (lane_id() == 0) atomicAdd(&s_bytes, bytes);
        }
        __syncthreads();
        if (!whole)
            for (int32_t i = tid; i < N; i += FM_THREADS)
                A.loc[(uint32_t)alist[i] & 0x7fffffffu] = -1;
        // adopt the better run if it improves on the start
        if (tid == 0) {
            ticks_moves += wall_clock64() - t0;
            const int rb = state_below(rs[1].best_imb, rs[1].best_cut, rs[0].best_imb, rs[0].best_cut) ? 1 : 0;
            const bool imp = state_below(rs[rb].best_imb, rs[rb].best_cut, start_imb, start_cut);
            atomicAdd(&A.ctl->stats[1], 2ull);
            atomicAdd(&A.ctl->stats[2], (unsigned long long)rs[0].m + (unsigned long long)rs[1].m);
            if (imp) {
                s_bytes += 12ull * (unsigned long long)rs[rb].kept;
                atomicAdd(&A.ctl->stats[3], (unsigned long long)rs[rb].kept);
                atomicAdd(&A.ctl->stats[4], 1ull);
                s_bw[0] = rs[rb].best_w[0];
                s_bw[1] = rs[rb].best_w[1];
                s_bc[0] = rs[rb].best_cnt[0];
                s_bc[1] = rs[rb].best_cnt[1];
            }
            s_stop = imp ? 0 : 1;
            s_pick = rb;
        }
        __syncthreads();
        if (s_stop) break;
        {
            // the kept moves: blocks flipped, degree sums moved, and the moved
            // nodes and their neighbours on the later list
            const int32_t *mb = A.mlog + (size_t)s_pick * A.n + off;
            const int32_t kk = rs[s_pick].kept;
            for (int32_t i = tid; i < kk; i += FM_THREADS) {
                const int32_t li = mb[i];
                const uint32_t id = whole ? f.gid[li] : (uint32_t)alist[li];
                const int32_t v = (int32_t)(id & 0x7fffffffu);
                const bool in_a = (id >> 31) == 0;
                const int64_t x0 = A.xadj[v], x1 = A.xadj[v + 1];
                A.part[v] = in_a ? b : a;
                if (whole) f.gid[li] = id ^ 0x80000000u;
                const unsigned long long d = (unsigned long long)(x1 - x0);
                atomicAdd((unsigned long long *)&s_bd[in_a ? 1 : 0], d);
                atomicAdd((unsigned long long *)&s_bd[in_a ? 0 : 1], 0ull - d);
                // The list takes the node, and those neighbours that are on no
                // list from before this launch, while it has room; beyond n
                // entries it stands for every node.  It may name a node several
                // times: for a pair of this launch whose entry may not be written
                // yet, and for this one again.  Telling the two apart, by stamps of
                // the pair's own, cost as much as the entries do (13 calls within
                // 3 % each way; with an exchange per neighbour up to 6 % more).
                if (later_count() > (unsigned long long)A.n) continue;
                unsigned long long at = atomicAdd(&A.ctl->xn, 1ull);
                if (at < (unsigned long long)A.n) A.xlist[at] = v;
                for (int64_t e = x0; e < x1; ++e) {
                    const int32_t u = A.adj[e];
                    const uint16_t was = A.ext[u];
                    if (was != 0 && was != (uint16_t)A.stamp) continue;
                    A.ext[u] = (uint16_t)A.stamp;
                    at = atomicAdd(&A.ctl->xn, 1ull);
                    if (at < (unsigned long long)A.n) A.xlist[at] = u;
                }
            }
        }
        __syncthreads();
    }
    if (whole)
        for (int32_t i = tid; i < len; i += FM_THREADS)
            A.loc[(uint32_t)alist[i] & 0x7fffffffu] = -1;
    if (tid == 0) {
        A.bw[a] = s_bw[0];
        A.bw[b] = s_bw[1];
        A.bd[a] = s_bd[0];
        A.bd[b] = s_bd[1];
        A.bc_out[a] = s_bc[0];
        A.bc_out[b] = s_bc[1];
        atomicAdd(&A.ctl->stats[5], s_bytes);
        atomicAdd(&A.ctl->stats[6], ticks_init);
        atomicAdd(&A.ctl->stats[7], ticks_moves);
    }
}

void launch_refine_weights(const RefineLaunch &R, hipStream_t s) {
    KAPPA_PROF("refine_weights", s);
    hipLaunchKernelGGL(ref_weights_k, dim3(grid_for(R.n, RQ_THREADS * 8, 1024)), dim3(RQ_THREADS),
                       0, s, R.xadj, R.ew, R.part, R.vw, R.n, R.k, R.bw, R.bc, R.bd, R.loc,
                       R.xlist, R.ctl);
}

void launch_refine_colouring(const RefineLaunch &R, int parity, hipStream_t s) {
    {
        KAPPA_PROF("refine_quotient", s);
        hipLaunchKernelGGL(ref_quotient_k, dim3(grid_for(R.n, RQ_THREADS * 2, 2048)),
                           dim3(RQ_THREADS), 0, s, R.xadj, R.adj, R.part, R.n, R.k, R.qbits, R.ext,
                           R.bcnt);
    }
    {
        KAPPA_PROF("refine_colour", s);
        hipLaunchKernelGGL(ref_colour_k, dim3(1), dim3(RQ_THREADS), 0, s, R.qbits, R.k, R.tab,
                           R.cpairs, R.col_off, R.bc + (parity ? R.k : 0), R.bcnt, R.blo, R.bme,
                           R.ctl);
    }
    KAPPA_PROF("refine_bucket", s);
    hipLaunchKernelGGL(ref_bucket_k, dim3(grid_for(R.n, RQ_THREADS * RB_ITEMS, 1u << 30)),
                       dim3(RQ_THREADS), 0, s, R.part, R.ext, R.n, R.k, R.blo, R.bcnt,
                       R.blist);
}

// bits of gain + 2^(bits - 1), |gain| at most the largest weighted degree
static int refine_gain_bits(uint64_t max_wd) {
    int bits = 2;
    while (bits < 64 && max_wd >= (1ull << (bits - 1))) ++bits;
    return bits;
}
bool refine_gains_fit(uint64_t max_wd) { return refine_gain_bits(max_wd) <= KEY64_GAIN_MAX_BITS; }

void launch_refine_colour(const RefineLaunch &R, int32_t gi, int32_t c, int32_t p0, int32_t npairs,
                          int parity, hipStream_t s) {
    FmArgs A;
    A.xadj = R.xadj; A.adj = R.adj; A.ew = R.ew; A.vw = R.vw; A.part = R.part;
    A.n = R.n; A.k = R.k; A.eps_num = R.eps_num; A.eps_den = R.eps_den; A.seed = R.seed;
    A.alpha_num = R.alpha_num; A.alpha_den = R.alpha_den; A.depth = R.depth;
    A.max_local = R.max_local; A.cpairs = R.cpairs;
    A.bw = R.bw; A.bd = R.bd;
    A.bc_in = R.bc + (parity ? R.k : 0);
    A.bc_out = R.bc + (parity ? 0 : R.k);
    A.blo = R.blo; A.bme = R.bme; A.blist = R.blist; A.xlist = R.xlist; A.ext = R.ext;
    A.stamp = c + 2;
    A.alist = R.alist; A.ldeg = R.ldeg; A.key = R.key; A.mlog = R.mlog;
    A.loc = R.loc; A.lrow = R.lrow; A.ctl = R.ctl;
    A.acap = R.acap < 0 || R.acap > FM_AREA ? FM_AREA : R.acap;
    A.gain_bits = refine_gain_bits(R.max_wd);
    KAPPA_PROF("refine_fm", s);
    const auto k = R.wide                              ? ref_fm_k<uint64_t, true>
                   : A.gain_bits <= KEY32_GAIN_MAX_BITS ? ref_fm_k<uint32_t, false>
                                                        : ref_fm_k<uint64_t, false>;
    hipLaunchKernelGGL(k, dim3(npairs), dim3(FM_THREADS), 0, s, A, gi, p0, npairs);
}

}  // namespace kappa
