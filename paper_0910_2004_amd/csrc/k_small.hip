// k_small.hip -- small levels, whole, in one workgroup's LDS.
//
// A level of a few thousand nodes as grid launches is 11 kernels and two or
// three rounds of two more, each a chain of dependent loads of a few
// microseconds, and a finisher that walks global memory: 77 us a level on a
// 64 x 64 grid and its coarser levels, whatever the size.  Here one launch takes
// every level from the first that fits to the end of the loop.  The level's node
// state (attribute, choice, mate, pending lists) is in LDS during the matching,
// the entries to merge are in LDS during the contraction; the graph itself is
// read from global memory (it stays in the XCD's L2 from level to level), so a
// phase is one chain of loads for all nodes together, between barriers.
// 64 x 64 grid down to 100 nodes, 6 levels: 330 us in one launch, 111 for the
// level of 4096 nodes, 23 for that of 186; the whole call 0.67 -> 0.40 ms.
// Levels of 3000 to 4000 nodes that lose few of them take 110 to 210 us here and
// 75 to 150 on the grid: a loop that ends on two to four such levels can lose 5 %
// (hubs and leaves, 3500 nodes: 410 and 430 us), one that goes on gains (twelve
// levels: 3.7 and 1.8 ms).
//
// What bounds it is one compute unit's issue rate on the largest levels (four
// waves a SIMD: a merge costs some hundred instructions per entry) and the
// phases' latency on small ones, hence the limits: SMALL_N nodes and SMALL_E
// entries fill the LDS, and rows of up to SMALL_DEG entries merge by ranks
// (compares grow with the square of a row).
#include "kappa_internal.h"

namespace kappa {

constexpr int SL_THREADS = 1024;
constexpr int SL_G = 4;        // lanes per row of the matching
constexpr int SL_SHORT = 32;   // longer rows: a wave each
// lanes per merged row and entries per lane, of at most 16 entries, 64 and above
constexpr int SL_MG = 8, SL_MU = 2;
constexpr int SL_MG2 = 16, SL_MU2 = 4;
constexpr int SL_MU3 = 8;
constexpr uint16_t SL_NONE = 0xffff;

struct SmallLds {
    union {
        struct {
            uint32_t attr[SMALL_N];
            uint16_t best[SMALL_N], pend[2][SMALL_N], longs[SMALL_N];
        } m;
        struct {
            uint32_t w[SMALL_E];
            uint16_t k[SMALL_E];   // rows start at even positions; SL_NONE: no entry
        } e;
    } u;
    uint16_t xadj[SMALL_N + 2];   // the level's offsets; merged degrees; the next level's offsets
    uint16_t mate[SMALL_N];
    uint16_t cmap[SMALL_N];       // after the staging: lists of the longer merged rows
    uint16_t soff[SMALL_N + 2];   // staged rows
    int64_t sh[SL_THREADS / WAVE + 1];
    // the loop's control block, read once and written back at the end, and the
    // level's and the next one's arrays: a level that fetched them from global
    // memory spent 11 us of 20 on those chains
    Control ctl;
    const int32_t *adj;
    const uint32_t *ew, *vw;
    int32_t *gmate, *gcmap;
    int64_t *nxadj;
    int32_t *nadj, *ngmate, *ngcmap;
    uint32_t *new_, *nvw;
    int32_t n, nnz, go, npend[2], nmid, nlong, pairs, point;
    int32_t degs, sdeg;
};
static_assert(sizeof(SmallLds) <= 160 * 1024, "one workgroup's LDS");
static_assert(SMALL_N <= 4 * SL_THREADS && SMALL_E < (1 << 16), "16-bit offsets");
static_assert(2 * SMALL_DEG + 2 <= SL_MU3 * WAVE, "a wave holds a merged row");

// Best edge from v to a free neighbour, over the lanes of a group of G.
template <int R, int G, bool FIRST>
__device__ __forceinline__ Cand small_scan(const SmallLds &s, int v, int sub, uint64_t seed) {
    constexpr int T = 4;   // entries of a lane in flight
    const int b = s.xadj[v], e = s.xadj[v + 1];
    const uint32_t av = R == KAPPA_WEIGHT ? 0u : s.u.m.attr[v];
    Cand best = cand_none();
    for (int j0 = b + sub; j0 < e; j0 += G * T) {
        int32_t u[T];
        uint32_t w[T];
#pragma unroll
        for (int t = 0; t < T; ++t) {
            const int j = j0 + t * G;
            u[t] = j < e ? s.adj[j] : -1;
            w[t] = j < e ? s.ew[j] : 0u;
        }
#pragma unroll
        for (int t = 0; t < T; ++t) {
            if ((uint32_t)u[t] >= (uint32_t)s.n || (!FIRST && s.mate[u[t]] != SL_NONE)) continue;
            const uint32_t au = R == KAPPA_WEIGHT ? 0u : s.u.m.attr[u[t]];
            Cand cd;
            rate<R>(w[t], au, av, au, av, cd.num, cd.den);
            cd.h = mix64(seed ^ edge_id_local(v, u[t], 0));
            cd.u = u[t];
            if (cand_better(cd, best, v)) best = cd;
        }
    }
    return group_reduce<G>(best, v);
}

// The choices of the `count` nodes of list (null: 0 .. count-1) that have none
// among the free nodes; the long rows after a barrier, a wave each.
template <int R, bool FIRST>
__device__ __forceinline__ void small_pick(SmallLds &s, const uint16_t *list, int count,
                                           uint64_t seed) {
    const int sub = threadIdx.x % SL_G;
    for (int i = threadIdx.x / SL_G; i < count; i += SL_THREADS / SL_G) {
        const int v = FIRST ? i : list[i];
        if (!FIRST) {
            const int b = s.u.m.best[v];
            if (s.mate[b] == SL_NONE) continue;   // still free: still the maximum
        }
        if (s.xadj[v + 1] - s.xadj[v] > SL_SHORT) {
            if (sub == 0) s.u.m.longs[atomicAdd(&s.nlong, 1)] = (uint16_t)v;
            continue;
        }
        const Cand cd = small_scan<R, SL_G, FIRST>(s, v, sub, seed);
        if (sub == 0) s.u.m.best[v] = (uint16_t)cd.u;   // -1: SL_NONE
    }
    __syncthreads();
    if (s.nlong == 0) return;
    for (int i = threadIdx.x / WAVE; i < s.nlong; i += SL_THREADS / WAVE) {   // wave-uniform
        const int v = s.u.m.longs[i];
        const Cand cd = small_scan<R, WAVE, FIRST>(s, v, lane_id(), seed);
        if (lane_id() == 0) s.u.m.best[v] = (uint16_t)cd.u;
    }
    __syncthreads();
    if (threadIdx.x == 0) s.nlong = 0;
}

// Mutual check over the round's nodes; the rest that points goes on.
template <bool FIRST>
__device__ __forceinline__ void small_mate(SmallLds &s, const uint16_t *list, int count,
                                           uint16_t *out, int32_t *nout) {
    int point = 0, degs = 0, pairs = 0, sdeg = 0;
    for (int i0 = 0; i0 < count; i0 += SL_THREADS) {   // block-uniform
        const int i = i0 + threadIdx.x;
        bool on = false;
        int v = 0;
        if (i < count) {
            v = FIRST ? i : list[i];
            const int b = s.u.m.best[v], deg = s.xadj[v + 1] - s.xadj[v];
            sdeg += deg;
            if (b != SL_NONE) {
                ++point;
                degs += deg;
                if (s.u.m.best[b] == v) {
                    s.mate[v] = (uint16_t)b;
                    pairs += v < b;
                } else {
                    on = true;
                }
            }
        }
        const uint64_t m = __ballot(on);
        if (m == 0) continue;
        int base = 0;
        if (lane_id() == 0) base = atomicAdd(nout, (int)__popcll(m));
        base = __shfl(base, 0, WAVE);
        if (on) out[base + (int)__popcll(m & lanemask_lt())] = (uint16_t)v;
    }
    point = wave_sum(point);
    if (point == 0 && !__ballot(sdeg > 0)) return;
    degs = wave_sum(degs);
    pairs = wave_sum(pairs);
    sdeg = wave_sum(sdeg);
    if (lane_id() == 0) {
        atomicAdd(&s.point, point);
        atomicAdd(&s.degs, degs);
        atomicAdd(&s.pairs, pairs);
        atomicAdd(&s.sdeg, sdeg);
    }
}

// Row [a, a + len) of the staged entries (len even, at most G * MU) merged in
// place by G lanes.  An entry's place in the sorted row is the number of
// smaller keys and of equal ones before it, counted two 16-bit keys an
// instruction; the first of a run of equal keys (up to four: two nodes, two
// neighbours) adds up the run.  Returns the distinct keys.
typedef uint16_t u16x2 __attribute__((ext_vector_type(2)));
template <int G, int MU>
__device__ __forceinline__ int small_merge(SmallLds &s, int a, int len, int sub) {
    uint16_t *const k = s.u.e.k + a;
    uint32_t *const w = s.u.e.w + a;
    const u16x2 *const kk = (const u16x2 *)k;
    const u16x2 one = {1, 1};
    uint16_t key[MU];
    uint32_t wt[MU];
    u16x2 below[MU];
#pragma unroll
    for (int q = 0; q < MU; ++q) {
        const int t = sub + q * G;
        key[q] = t < len ? k[t] : SL_NONE;
        wt[q] = t < len ? w[t] : 0u;
        below[q] = u16x2{0, 0};
    }
    for (int p0 = 0; p0 < len; p0 += 8) {
        u16x2 x[4];
#pragma unroll
        for (int h = 0; h < 4; ++h)
            x[h] = p0 + 2 * h < len ? kk[p0 / 2 + h] : u16x2{SL_NONE, SL_NONE};
#pragma unroll
        for (int h = 0; h < 4; ++h) {
            const uint16_t p = (uint16_t)(p0 + 2 * h);
            const u16x2 at = {p, (uint16_t)(p + 1)};
#pragma unroll
            for (int q = 0; q < MU; ++q) {
                if (MU > 2 && q * G >= len) continue;
                const uint16_t t = (uint16_t)(sub + q * G);
                const u16x2 t2 = {t, t}, k2 = {key[q], key[q]};
                // x below key, or equal and before t: x < key + (p < t)
                const u16x2 lim = k2 + __builtin_elementwise_min(__builtin_elementwise_sub_sat(t2, at), one);
                below[q] += __builtin_elementwise_min(__builtin_elementwise_sub_sat(lim, x[h]), one);
            }
        }
    }
    wave_sync_lds();
#pragma unroll
    for (int q = 0; q < MU; ++q) {
        if (sub + q * G >= len) continue;
        // entries without a key go behind the others, in their order
        const int r = key[q] != SL_NONE ? below[q].x + below[q].y : -1;
        if (r < 0) continue;
        k[r] = key[q];
        w[r] = wt[q];
    }
    // the sorted keys end where those without one begin
    int n = 0;
#pragma unroll
    for (int q = 0; q < MU; ++q) n += key[q] != SL_NONE;
    for (int o = G / 2; o > 0; o >>= 1) n += __shfl_xor(n, o, G);
    wave_sync_lds();
    int done = 0;   // distinct keys of the slots before
    const uint64_t group = G == WAVE ? ~0ull : (((1ull << (G % WAVE)) - 1) << (lane_id() / G * G));
    int to[MU];
#pragma unroll
    for (int q = 0; q < MU; ++q) {
        const int t = sub + q * G;
        to[q] = -1;
        bool lead = false;
        if (t < n) {
            key[q] = k[t];
            wt[q] = w[t];
            lead = t == 0 || k[t - 1] != key[q];
            if (lead)
                for (int z = t + 1; z < n && k[z] == key[q]; ++z) wt[q] += w[z];
        }
        const uint64_t m = __ballot(lead) & group;
        if (lead) to[q] = done + (int)__popcll(m & lanemask_lt());
        done += (int)__popcll(m);
    }
    wave_sync_lds();
#pragma unroll
    for (int q = 0; q < MU; ++q) {
        if (to[q] < 0) continue;
        k[to[q]] = key[q];
        w[to[q]] = wt[q];
    }
    return done;
}

template <int R>
__global__ void __launch_bounds__(SL_THREADS) small_levels_k(Ctx c, int l0) {
    __shared__ SmallLds s;
    const int tid = threadIdx.x;
    Control &ctl = s.ctl;   // thread 0's
    if (tid == 0) {
        LevelDesc *const L = c.lv + l0;
        ctl = *c.ctrl;
        s.go = !ctl.done && ctl.nlevels == l0 + 1 && L->phase == PH_IDLE && L->mate && L->cmap;
        const int64_t nnz = L->nnz;
        s.n = L->n;
        if (s.n > SMALL_N || nnz + s.n > SMALL_E) {
            // a level that does not fit may still be the one to stop at (left to
            // the grid, that took a read-back and the launches of a batch of
            // levels, 110 us)
            const int stop = s.n <= ctl.stop_n ? KAPPA_STOP_SIZE
                                               : (l0 >= ctl.max_levels ? KAPPA_STOP_MAXLEVEL : KAPPA_STOP_NONE);
            if (s.go && stop != KAPPA_STOP_NONE) {
                L->stop = stop;
                L->phase = PH_STOPPED;
                c.ctrl->done = 1;
            }
            s.go = 0;
        }
        s.nnz = (int32_t)nnz;
        s.adj = L->adj;
        s.ew = L->ew;
        s.vw = L->vw;
        s.gmate = L->mate;
        s.gcmap = L->cmap;
    }
    __syncthreads();
    if (!s.go) return;
    for (int l = l0;; ++l) {
        // every level from here on is no larger; go: it starts
        LevelDesc *const L = c.lv + l, *const N = L + 1;
        if (tid == 0)
            s.npend[0] = s.npend[1] = s.nmid = s.nlong = s.pairs = s.point = s.degs = s.sdeg = 0;
        const int n = s.n;
        if (l == l0) {   // (later levels: the offsets are there)
            const int64_t *x = L->xadj;
            for (int v = tid; v <= n; v += SL_THREADS) s.xadj[v] = (uint16_t)x[v];
            __syncthreads();
        }
        // a row too long, or (unchecked input) offsets that are none: the staged
        // entries have to fit
        bool deep = tid == 0 && (s.xadj[0] != 0 || s.xadj[n] != s.nnz);
        for (int v = tid; v < n; v += SL_THREADS) {
            const int d = s.xadj[v + 1] - s.xadj[v];
            deep = deep || d < 0 || d > SMALL_DEG;
            s.mate[v] = SL_NONE;
            if (R != KAPPA_WEIGHT && (R != KAPPA_INNER_OUTER || l > 0))
                s.u.m.attr[v] = R == KAPPA_INNER_OUTER ? c.ms.out[v] : s.vw[v];
        }
        if (__syncthreads_or(deep)) break;
        if (tid == 0) {   // level_gate's rules
            const int stop = s.n <= ctl.stop_n ? KAPPA_STOP_SIZE
                                               : (l >= ctl.max_levels ? KAPPA_STOP_MAXLEVEL : KAPPA_STOP_NONE);
            s.go = stop == KAPPA_STOP_NONE;
            if (!s.go) {
                L->stop = stop;
                L->phase = PH_STOPPED;
                ctl.done = 1;
            }
        }
        if (R == KAPPA_INNER_OUTER && l == 0) {   // Out(v)
            for (int v = tid / SL_G; v < n; v += SL_THREADS / SL_G) {
                uint32_t o = 0;
                for (int j = s.xadj[v] + tid % SL_G; j < s.xadj[v + 1]; j += SL_G) o += s.ew[j];
                o += __shfl_xor(o, 1, SL_G);
                o += __shfl_xor(o, 2, SL_G);
                if (tid % SL_G == 0) s.u.m.attr[v] = o;
            }
        }
        __syncthreads();
        if (!s.go) break;

        // --- matching ---------------------------------------------------------
        const uint64_t seed = level_seed(c, l);
        int r = 0, used = 0;
        do {
            ++r;
            uint16_t *const in = s.u.m.pend[(r - 1) & 1], *const out = s.u.m.pend[r & 1];
            const int count = r == 1 ? n : s.npend[(r - 1) & 1];
            if (r == 1) small_pick<R, true>(s, in, count, seed);
            else small_pick<R, false>(s, in, count, seed);
            if (r == 1) small_mate<true>(s, in, count, out, &s.npend[r & 1]);
            else small_mate<false>(s, in, count, out, &s.npend[r & 1]);
            __syncthreads();
            if (tid == 0) {
                if (s.point) {
                    used = r;
                    // (the last slot keeps the sums of all further rounds)
                    int64_t *const st = L->stat[min(r, STAT_ROUNDS) - 1];
                    const bool first = r <= STAT_ROUNDS, rescan = r > 1 && c.rescan_stats;
                    st[0] = (first ? 0 : st[0]) + s.point;
                    st[1] = (first ? 0 : st[1]) + s.degs;
                    st[2] = (first ? 0 : st[2]) + (rescan ? count : 0);
                    st[3] = (first ? 0 : st[3]) + (rescan ? s.sdeg : 0);
                }
                s.point = s.degs = s.sdeg = 0;
                s.npend[(r - 1) & 1] = 0;
            }
            __syncthreads();
            // (a round that points matches a pair, so the cap is for broken input)
        } while (s.npend[r & 1] > 0 && r < n + 2);
        const bool capped = s.npend[r & 1] > 0;
        for (int v = tid; v < n; v += SL_THREADS)
            s.gmate[v] = s.mate[v] == SL_NONE ? -1 : (int32_t)s.mate[v];
        if (tid == 0) {
            L->matched = s.pairs;
            L->rounds = used;
            L->grid_rounds = used;
            if (capped) ctl.flags |= CF_ROUNDS;
            if (s.pairs == 0 || capped) {
                L->stop = KAPPA_STOP_EMPTY;
                L->phase = PH_STOPPED;
                ctl.done = 1;
            }
        }
        if (s.pairs == 0 || capped) break;   // block-uniform: both are settled

        // --- contraction ------------------------------------------------------
        // coarse ids and staged rows, four consecutive nodes a thread
        int64_t mine = 0, all;
        int tot[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int v = 4 * tid + q;
            tot[q] = -1;   // no representative
            if (v >= n) continue;
            const int m = s.mate[v];
            if (m != SL_NONE && m < v) continue;
            tot[q] = s.xadj[v + 1] - s.xadj[v];
            if (m != SL_NONE) tot[q] += s.xadj[m + 1] - s.xadj[m];
            mine += ((int64_t)1 << 32) + ((tot[q] + 1) & ~1);
        }
        const int64_t pre = block_excl_scan(mine, s.sh, &all);
        const int nc = (int)(all >> 32);
        int x = (int)(pre >> 32), at = (int)(pre & 0xffffffff);
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            if (tot[q] < 0) continue;
            const int v = 4 * tid + q, m = s.mate[v];
            s.cmap[v] = (uint16_t)x;
            if (m != SL_NONE) s.cmap[m] = (uint16_t)x;
            s.soff[x] = (uint16_t)at;
            ++x;
            at += (tot[q] + 1) & ~1;
        }
        if (tid == 0) {
            s.soff[nc] = (uint16_t)(all & 0xffffffff);
            const uint64_t b4 = (uint64_t)nc * 4, bytes[4] = {b4, (uint64_t)(nc + 1) * 8, b4, b4};
            void *a[4];
            s.go = arena_alloc_k<4>(&ctl, bytes, a);
            s.nvw = (uint32_t *)a[0];
            s.nxadj = (int64_t *)a[1];
            s.ngmate = (int32_t *)a[2];
            s.ngcmap = (int32_t *)a[3];
        }
        __syncthreads();
        if (!s.go) {
            if (tid == 0) {
                L->phase = PH_STOPPED;
                ctl.done = 1;
            }
            break;
        }
        // entries, renamed, to their coarse rows
        for (int v = tid / SL_G; v < n; v += SL_THREADS / SL_G) {
            const int sub = tid % SL_G, m = s.mate[v], b = s.xadj[v], deg = s.xadj[v + 1] - b;
            const int y = s.cmap[v];
            const bool second = m != SL_NONE && m < v;
            int d = s.soff[y];
            if (second) d += s.xadj[m + 1] - s.xadj[m];
            if (sub == 0) {
                s.gcmap[v] = y;
                if (!second) s.nvw[y] = s.vw[v] + (m != SL_NONE ? s.vw[m] : 0u);
                // the odd row's last slot, by its second node (or only one)
                if ((second || m == SL_NONE) && d + deg < s.soff[y + 1]) s.u.e.k[d + deg] = SL_NONE;
            }
            for (int j0 = sub; j0 < deg; j0 += SL_G * 4) {
                int32_t u[4];
                uint32_t w[4];
#pragma unroll
                for (int t = 0; t < 4; ++t) {
                    const int j = j0 + t * SL_G;
                    u[t] = j < deg ? s.adj[b + j] : -1;
                    w[t] = j < deg ? s.ew[b + j] : 0u;
                }
#pragma unroll
                for (int t = 0; t < 4; ++t) {
                    const int j = j0 + t * SL_G;
                    if (j >= deg) continue;
                    s.u.e.k[d + j] = (uint32_t)u[t] >= (uint32_t)n || u[t] == m ? SL_NONE : s.cmap[u[t]];
                    s.u.e.w[d + j] = w[t];
                }
            }
        }
        __syncthreads();
        // merged rows: degrees to xadj.  Rows of more than 16 entries wait in cmap,
        // those of up to 64 from its front (a quarter of a wave each), longer ones
        // from its back (a wave each): merged where they stand, each made the
        // other seven rows of its wave take the steps of a long one (levels of
        // 3000 nodes by weight on a 700 x 700 grid: 165 us, a 64 x 64 grid's 32)
        {
            const int sub = tid % SL_MG;
            for (int i0 = 0; i0 < nc; i0 += SL_THREADS / SL_MG) {   // block-uniform
                const int y = i0 + tid / SL_MG;
                int a = 0, len = 0;
                if (y < nc) {
                    a = s.soff[y];
                    len = s.soff[y + 1] - a;
                }
                if (len > SL_MG * SL_MU) {
                    if (sub == 0)
                        s.cmap[len <= SL_MG2 * SL_MU2 ? atomicAdd(&s.nmid, 1)
                                                      : SMALL_N - 1 - atomicAdd(&s.nlong, 1)] = (uint16_t)y;
                    len = 0;
                }
                const int k = small_merge<SL_MG, SL_MU>(s, a, len, sub);
                if (y < nc && sub == 0) s.xadj[y] = (uint16_t)k;
            }
            __syncthreads();
            constexpr int PER = WAVE / SL_MG2;
            for (int i0 = tid / WAVE * PER; i0 < s.nmid; i0 += SL_THREADS / SL_MG2) {   // wave-uniform
                const int i = i0 + lane_id() / SL_MG2;
                int y = 0, a = 0, len = 0;
                if (i < s.nmid) {
                    y = s.cmap[i];
                    a = s.soff[y];
                    len = s.soff[y + 1] - a;
                }
                const int k = small_merge<SL_MG2, SL_MU2>(s, a, len, tid % SL_MG2);
                if (i < s.nmid && tid % SL_MG2 == 0) s.xadj[y] = (uint16_t)k;
            }
            for (int i = tid / WAVE; i < s.nlong; i += SL_THREADS / WAVE) {   // wave-uniform
                const int y = s.cmap[SMALL_N - 1 - i], a = s.soff[y];
                const int k = small_merge<WAVE, SL_MU3>(s, a, s.soff[y + 1] - a, lane_id());
                if (lane_id() == 0) s.xadj[y] = (uint16_t)k;
            }
            __syncthreads();
        }
        // offsets
        int deg[4];
        mine = 0;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int y = 4 * tid + q;
            deg[q] = y < nc ? s.xadj[y] : 0;
            mine += deg[q];
        }
        int64_t run = block_excl_scan(mine, s.sh, &all);   // (reads of xadj are done)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int y = 4 * tid + q;
            if (y >= nc) continue;
            s.xadj[y] = (uint16_t)run;
            s.nxadj[y] = run;
            run += deg[q];
        }
        if (tid == 0) {
            s.xadj[nc] = (uint16_t)all;
            s.nxadj[nc] = all;
            const uint64_t b4 = (uint64_t)all * 4, bytes[2] = {b4, b4};
            void *a[2];
            s.go = arena_alloc_k<2>(&ctl, bytes, a);
            s.nadj = (int32_t *)a[0];
            s.new_ = (uint32_t *)a[1];
        }
        __syncthreads();
        if (!s.go) {
            if (tid == 0) {
                L->phase = PH_STOPPED;
                ctl.done = 1;
            }
            break;
        }
        for (int y = tid / SL_MG; y < nc; y += SL_THREADS / SL_MG) {
            const int sub = tid % SL_MG, a = s.soff[y], d = s.xadj[y], len = s.xadj[y + 1] - d;
            uint32_t sum = 0;
            for (int t = sub; t < len; t += SL_MG) {
                const uint32_t w = s.u.e.w[a + t];
                s.nadj[d + t] = s.u.e.k[a + t];
                s.new_[d + t] = w;
                sum += w;
            }
            if (R == KAPPA_INNER_OUTER) {
                for (int o = SL_MG / 2; o > 0; o >>= 1) sum += __shfl_xor(sum, o, SL_MG);
                if (sub == 0) c.ms.out[y] = sum;
            }
        }
        __syncthreads();
        if (tid == 0) {   // the next level; the stall rule
            const bool stall = ctl.stall_num > 0 && (uint64_t)(n - nc) * ctl.stall_den <
                                                        (uint64_t)ctl.stall_num * (uint64_t)n;
            L->phase = PH_DONE;
            N->n = nc;
            N->nnz = all;
            N->maxdeg = 0;   // not tracked below level 0
            N->xadj = s.nxadj;
            N->adj = s.nadj;
            N->ew = s.new_;
            N->vw = s.nvw;
            N->mate = s.ngmate;
            N->cmap = s.ngcmap;
            N->gid = nullptr;
            N->noff = nullptr;
            N->stop = stall ? KAPPA_STOP_STALL : KAPPA_STOP_NONE;
            N->phase = stall ? PH_STOPPED : PH_IDLE;
            ctl.nlevels = l + 2;
            ctl.last_n = nc;
            ctl.last_nnz = all;
            if (stall) ctl.done = 1;
            s.go = !stall;
            s.n = nc;
            s.nnz = (int32_t)all;
            s.adj = s.nadj;
            s.ew = s.new_;
            s.vw = s.nvw;
            s.gmate = s.ngmate;
            s.gcmap = s.ngcmap;
        }
        __syncthreads();
        if (!s.go) break;
    }
    if (tid == 0) *c.ctrl = ctl;
}

void launch_small_levels(const Ctx &c, int l, hipStream_t s) {
    KAPPA_PROF("small_levels", s);
    const dim3 g(1), b(SL_THREADS);
    switch (c.rating) {
    case KAPPA_INNER_OUTER: hipLaunchKernelGGL(small_levels_k<KAPPA_INNER_OUTER>, g, b, 0, s, c, l); break;
    case KAPPA_WEIGHT: hipLaunchKernelGGL(small_levels_k<KAPPA_WEIGHT>, g, b, 0, s, c, l); break;
    case KAPPA_EXPANSION: hipLaunchKernelGGL(small_levels_k<KAPPA_EXPANSION>, g, b, 0, s, c, l); break;
    case KAPPA_EXPANSION_STAR: hipLaunchKernelGGL(small_levels_k<KAPPA_EXPANSION_STAR>, g, b, 0, s, c, l); break;
    default: hipLaunchKernelGGL(small_levels_k<KAPPA_EXPANSION_STAR2>, g, b, 0, s, c, l); break;
    }
}

}  // namespace kappa
