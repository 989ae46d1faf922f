// build.hip -- octree construction on gfx950.
//
// Steps (Barnes-Hut tree of Section 2.4 of Arnold, Baumgardt & Wang 2021):
//   bbox     per-cluster bounding box and NaN/Inf check (per-block partial boxes,
//            reduced again by every workgroup of the keys)
//   keys     cluster id above D-bit-per-axis Morton codes (x, y, z interleaved)
//   sort     stable sort (sort.hip) -> sorted keys and permutation
//   topology a node is a run of sorted particles sharing a key prefix whose
//            parent holds more than n_leaf particles; each particle knows the
//            levels of the nodes it starts, so a count per tile and level, one
//            scan of those counts and ballots within a tile give every node its
//            place in breadth-first order, in which children are contiguous
//   moments  bottom-up inside tiles of particles, then the nodes that straddle
//            tiles: M, centre of mass, traceless quadrupole about it
//            (parallel-axis sums over children), tight box
//   groups   tree-bounded runs of <= n_crit sorted particles (rule at k_group_pass)
//
// A build is 11 launches up to 1024 particles, 12 up to 8192, 18 up to 2^17 and 19
// up to 2^22 (there were 43 to 53; beyond, the radix sort alone has 32 or more):
// with kernels of a few microseconds the launches, and the scans between them, were
// most of its time.
//
// FP64 arithmetic that decides the tree (keys, moments) is evaluated without
// fused multiply-add so it rounds exactly as written.
#include "pbh_internal.hpp"
#include "wave.hpp"

namespace pbh {

namespace {

constexpr int BB_T = 256;

// ------------------------------------------------------------------ bbox
__device__ inline double wave_min_f64(double v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v = fmin(v, __shfl_xor(v, o, 64));
    return v;
}

// box[6] (lo, -hi) of the workgroup's threads, in thread 0 .. all (min is exact,
// so the order does not matter); s has 6 entries per wave
__device__ inline void block_box(double (&v)[6], double (*s)[6]) {
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    for (int k = 0; k < 6; ++k) v[k] = wave_min_f64(v[k]);
    if (lane == 0)
        for (int k = 0; k < 6; ++k) s[w][k] = v[k];
    __syncthreads();
    for (int k = 0; k < 6; ++k) {
        double m = s[0][k];
        for (int q = 1; q < BB_T / 64; ++q) m = fmin(m, s[q][k]);
        v[k] = m;
    }
}

// Partial boxes of the blocks of the cluster table, and the zeroing of the counters
// but for those that outlive a build.
__global__ __launch_bounds__(BB_T) void k_bbox_part(const double* __restrict__ pos,
                                                    const double* __restrict__ mass,
                                                    const int64_t* __restrict__ range,
                                                    double* __restrict__ part, int32_t* __restrict__ bad,
                                                    unsigned long long* __restrict__ cnt) {
    __shared__ double s_v[BB_T / 64][6];
    const int t = threadIdx.x;
    for (int i = blockIdx.x * BB_T + t; i < kNumCounters + kQueueWords; i += gridDim.x * BB_T)
        if (i < kCntKept || i >= kNumCounters) cnt[i] = 0ull;
    const int64_t b0 = range[2 * blockIdx.x], b1 = range[2 * blockIdx.x + 1];
    double v[6] = {INFINITY, INFINITY, INFINITY, INFINITY, INFINITY, INFINITY};
    int nf = 0;
#pragma unroll 8
    for (int64_t i = b0 + t; i < b1; i += BB_T) {
        const double x = pos[3 * i], y = pos[3 * i + 1], z = pos[3 * i + 2], mm = mass[i];
        nf |= !(isfinite(x) && isfinite(y) && isfinite(z) && isfinite(mm));
        v[0] = fmin(v[0], x); v[1] = fmin(v[1], y); v[2] = fmin(v[2], z);
        v[3] = fmin(v[3], -x); v[4] = fmin(v[4], -y); v[5] = fmin(v[5], -z);
    }
    const int any = __syncthreads_or(nf);
    block_box(v, s_v);
    if (t < 6) part[6 * blockIdx.x + t] = t == 0 ? v[0] : t == 1 ? v[1] : t == 2 ? v[2] : t == 3 ? v[3] : t == 4 ? v[4] : v[5];
    if (t == 0) bad[blockIdx.x] = any;
}

// ------------------------------------------------------------------ keys
__device__ inline uint64_t spread_bits3(uint64_t v) {
    // spread the low 21 bits of v to every third bit
    v &= 0x1fffffull;
    v = (v | (v << 32)) & 0x1f00000000ffffull;
    v = (v | (v << 16)) & 0x1f0000ff0000ffull;
    v = (v | (v << 8)) & 0x100f00f00f00f00full;
    v = (v | (v << 4)) & 0x10c30c30c30c30c3ull;
    v = (v | (v << 2)) & 0x1249249249249249ull;
    return v;
}

// The cluster's box from its blocks' partial boxes (cluster c: blocks
// [cblk[c], cblk[c+1])), then the keys of the block's particles.
__global__ __launch_bounds__(BB_T) void k_keys(const double* __restrict__ pos,
                                               const int64_t* __restrict__ range,
                                               const int32_t* __restrict__ blk_cluster,
                                               const int32_t* __restrict__ cblk,
                                               const double* __restrict__ part, const int32_t* __restrict__ bad,
                                               int D, uint64_t* __restrict__ keys,
                                               unsigned long long* __restrict__ cnt) {
#pragma clang fp contract(off)
    __shared__ double s_v[BB_T / 64][6];
    const int c = blk_cluster[blockIdx.x];
    const int p0 = cblk[c], p1 = cblk[c + 1];
    double v[6] = {INFINITY, INFINITY, INFINITY, INFINITY, INFINITY, INFINITY};
    int nf = 0;
    for (int b = p0 + threadIdx.x; b < p1; b += BB_T) {
        for (int k = 0; k < 6; ++k) v[k] = fmin(v[k], part[6 * (int64_t)b + k]);
        nf |= bad[b];
    }
    const int any = __syncthreads_or(nf);
    if (any && threadIdx.x == 0 && (int)blockIdx.x == p0) atomicOr(&cnt[kErr], kErrNonFinite);
    block_box(v, s_v);
    const int64_t b0 = range[2 * blockIdx.x], b1 = range[2 * blockIdx.x + 1];
    double L = 0.0;
    for (int k = 0; k < 3; ++k) {
        const double e = -v[3 + k] - v[k];
        if (e > L) L = e;
    }
    if (L == 0.0) L = 1.0;
    const double scale = ldexp(1.0, D) / L;
    const int64_t maxc = ((int64_t)1 << D) - 1;
    const uint64_t cid = (uint64_t)c << (3 * D);
#pragma unroll 4
    for (int64_t i = b0 + threadIdx.x; i < b1; i += BB_T) {
        const double x[3] = {pos[3 * i], pos[3 * i + 1], pos[3 * i + 2]};
        uint64_t key = 0;
        for (int k = 0; k < 3; ++k) {
            int64_t q = (int64_t)floor((x[k] - v[k]) * scale);
            q = q > maxc ? maxc : (q < 0 ? 0 : q);
            key |= spread_bits3((uint64_t)q) << (2 - k);
        }
        keys[i] = cid | key;
    }
}

// -------------------------------------------------------------- topology
// Key layout: [cluster id | D levels of 3 bits]. Level l >= 1 prefix = key >> 3(D-l).
__device__ inline uint64_t prefix(uint64_t key, int l, int D) { return key >> (3 * (D - l)); }

__device__ inline int cluster_of(uint64_t key, int D) { return (int)(key >> (3 * D)); }

// Topology runs over tiles of kTopoT particles. A particle i carries the first
// level at which its key differs from that of i - 1 (0 at the start of a
// cluster, D + 1 for equal keys): level-l runs start exactly at the particles
// whose first level is at most l. It starts nodes at the levels first .. last
// (last < first: none).
constexpr int kTopoT = 256;
constexpr int kTopoW = kTopoT / 64;

__device__ inline int lv_first(int lv) { return lv & 255; }
__device__ inline int lv_last(int lv) { return (lv >> 8) - 1; }

// Levels of every particle's nodes, and the nodes per tile and level:
// table[l][tile]. Sorts the particles into place on the way (x, y, z, m) and
// clears the group flags and histograms.
__global__ __launch_bounds__(kTopoT) void k_topo_count(const uint64_t* __restrict__ keys,
                                                       const int64_t* __restrict__ cl_off, int64_t n, int D,
                                                       int n_leaf, int32_t* __restrict__ lv_out, int64_t ntile,
                                                       int32_t* __restrict__ table, const double* __restrict__ pos,
                                                       const double* __restrict__ mass,
                                                       const int32_t* __restrict__ perm, double* __restrict__ x,
                                                       double* __restrict__ y, double* __restrict__ z,
                                                       double* __restrict__ m, int32_t* __restrict__ g_flag,
                                                       unsigned* __restrict__ hist, int64_t hist_len) {
    __shared__ int s_c[kTopoW][64];
    const int t = threadIdx.x, lane = t & 63, w = t >> 6;
    for (int64_t k = (int64_t)blockIdx.x * kTopoT + t; k < hist_len; k += (int64_t)gridDim.x * kTopoT) hist[k] = 0u;
    const int64_t i = (int64_t)blockIdx.x * kTopoT + t;
    int first = D + 1, last = D;   // (beyond n: no nodes)
    if (i < n) {
        const int64_t src = perm[i];
        const double px = pos[3 * src], py = pos[3 * src + 1], pz = pos[3 * src + 2], pm = mass[src];
        const uint64_t key = keys[i];
        const int c = cluster_of(key, D);
        const int64_t cs = cl_off[c], ce = cl_off[c + 1];
        bool starts = true;
        if (i == cs) {
            first = 0;
        } else {
            const uint64_t q = key ^ keys[i - 1];
            if (q == 0) {
                starts = false;
            } else {
                first = D - (63 - __clzll(q)) / 3;
                // the parent run (level first - 1) contains i - 1 and i: it must hold more than n_leaf
                const uint64_t pp = prefix(key, first - 1, D);
                int64_t a = i - 1, b = i + 1;
                while (a > cs && b - a <= n_leaf && prefix(keys[a - 1], first - 1, D) == pp) --a;
                while (b < ce && b - a <= n_leaf && prefix(keys[b], first - 1, D) == pp) ++b;
                starts = b - a > n_leaf;
            }
        }
        last = first - 1;
        if (starts) {
            // levels first + 1 .. exist while the run of level l - 1 starting at i holds > n_leaf:
            // while particle i + n_leaf is in it
            last = first;
            const int64_t j = i + n_leaf;
            if (j < ce) {
                const uint64_t q = key ^ keys[j];
                const int same = q == 0 ? D : D - 1 - (63 - __clzll(q)) / 3;   // deepest common level
                if (same + 1 > last) last = same + 1 < D ? same + 1 : D;
            }
        }
        lv_out[i] = first | (last + 1) << 8;
        x[i] = px;
        y[i] = py;
        z[i] = pz;
        m[i] = pm;
        g_flag[i] = 0;
    }
    int cnt = 0;
    for (int l = 0; l <= D; ++l) {
        const int c = __popcll(__ballot(first <= l && l <= last));
        cnt = lane == l ? c : cnt;
    }
    s_c[w][lane] = cnt;
    __syncthreads();
    if (t <= D) {
        int c = 0;
        for (int q = 0; q < kTopoW; ++q) c += s_c[q][t];
        table[(int64_t)t * (ntile + 1) + blockIdx.x] = c;
    }
}

// Exclusive scan of a level's counts over the tiles, its total behind them (one
// workgroup a level).
__global__ __launch_bounds__(1024) void k_topo_scan(int64_t ntile, int32_t* __restrict__ table) {
    __shared__ int s_w[16];
    int32_t* row = table + (int64_t)blockIdx.x * (ntile + 1);
    const int t = threadIdx.x, lane = t & 63, w = t >> 6;
    int carry = 0;
    for (int64_t c0 = 0; c0 < ntile; c0 += 4096) {
        int v[4], sum = 0;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int64_t k = c0 + 4 * t + u;
            v[u] = k < ntile ? row[k] : 0;
            sum += v[u];
        }
        const int inc = wave_incl_scan(sum, lane);
        __syncthreads();
        if (lane == 63) s_w[w] = inc;
        __syncthreads();
        int run = carry + inc - sum;
        for (int q = 0; q < 16; ++q) {
            if (q < w) run += s_w[q];
            carry += s_w[q];
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int64_t k = c0 + 4 * t + u;
            if (k < ntile) row[k] = run;
            run += v[u];
        }
    }
    if (t == 0) row[ntile] = carry;
}

// First node of every level, s_off[0 .. D + 1] (the levels' totals stand at
// table[l][ntile]); more nodes than the capacity: all zero. Threads 0 .. 63.
__device__ inline void level_offsets(const int32_t* __restrict__ table, int64_t ntile, int D, int64_t cap,
                                     int* s_off) {
    const int l = threadIdx.x;
    const int v = l <= D ? table[(int64_t)l * (ntile + 1) + ntile] : 0;
    const int inc = wave_incl_scan(v, l);
    const bool over = (int64_t)last_lane(inc) > cap;   // (node capacities stay below 2^31)
    if (l <= D + 1) s_off[l] = over ? 0 : inc - v;
}

// End (exclusive) of the level-l run that contains particle a, by the 8 lanes of
// an aligned lane group that share (a, l): each step probes 8 places, first at
// growing distances, then evenly between the last particle known inside and the
// first known outside. Every lane of the wave takes part; groups with on = false
// return a at once.
__device__ inline int64_t run_end8(const uint64_t* __restrict__ keys, bool on, int64_t a, int64_t ce, int l, int D) {
    const int lane = threadIdx.x & 63, g = lane & 7, sh = lane & 56;
    const uint64_t p = on ? prefix(keys[a], l, D) : 0;
    int64_t lo = a, hi = on ? ce : a + 1;
    bool grow = true;
    while (__ballot(hi - lo > 1)) {
        int64_t q;
        if (grow) q = a + ((int64_t)1 << (3 * g));
        else if (hi - lo <= 9) q = lo + 1 + g;
        else q = lo + (hi - lo) * (g + 1) / 9;
        const bool in = hi - lo > 1 && q < hi && prefix(keys[q], l, D) == p;
        const int c = __popc((unsigned)((__ballot(in) >> sh) & 255u));   // probes inside (they come first)
        const int64_t q0 = __shfl(q, sh + (c > 0 ? c - 1 : 0), 64), q1 = __shfl(q, sh + (c < 8 ? c : 7), 64);
        if (hi - lo > 1) {
            if (c > 0) lo = q0;
            if (c < 8 && q1 < hi) hi = q1;
        }
        grow = false;
    }
    return on ? hi : a;
}

// The nodes of a tile's particles, at their places in breadth-first order: the
// level's offset, its count in the tiles before, then the nodes of the level
// before this particle in the tile. A run ends before the next particle whose
// first level is no deeper, found in the tile's masks, or by a search beyond
// the tile. The first child of a node that holds more than n_leaf particles is
// the node of the next level that the same particle starts; the number of
// children is a difference of places when the node ends in the tile, and left
// to the moments (-1) when it does not.
__global__ __launch_bounds__(kTopoT) void k_topo_emit(const uint64_t* __restrict__ keys,
                                                      const int64_t* __restrict__ cl_off, int64_t n, int D,
                                                      int n_leaf, const int32_t* __restrict__ lv_in, int64_t ntile,
                                                      const int32_t* __restrict__ table, int64_t cap,
                                                      NodePlanes node, int32_t* __restrict__ lvl_off,
                                                      unsigned long long* __restrict__ cnt) {
    __shared__ int s_off[64];
    __shared__ uint64_t s_run[kMaxLevels + 1][kTopoW];  // particles that start a run of level l
    __shared__ uint64_t s_node[kMaxLevels + 1][kTopoW]; // ... a node
    __shared__ int s_pre[kMaxLevels + 1][kTopoW + 1];   // place of a wave's first node of a level
    __shared__ int64_t s_end[kMaxLevels + 1];           // end of the run that reaches out of the tile
    __shared__ int s_leaves;
    const int t = threadIdx.x, lane = t & 63, w = t >> 6;
    if (t < 64) level_offsets(table, ntile, D, cap, s_off);
    if (t == 0) s_leaves = 0;
    const int64_t t0 = (int64_t)blockIdx.x * kTopoT, i = t0 + t;
    const int lv = i < n ? lv_in[i] : (D + 1) | (D + 1) << 8;
    const int first = lv_first(lv), last = lv_last(lv);
    for (int l = 0; l <= D; ++l) {
        const uint64_t r = __ballot(first <= l), q = __ballot(first <= l && l <= last);
        if (lane == 0) {
            s_run[l][w] = r;
            s_node[l][w] = q;
        }
    }
    __syncthreads();
    if (t <= D) {
        int c = s_off[t] + table[(int64_t)t * (ntile + 1) + blockIdx.x];
        for (int q = 0; q < kTopoW; ++q) {
            s_pre[t][q] = c;
            c += __popcll(s_node[t][q]);
        }
        s_pre[t][kTopoW] = c;
    }
    // Where the last run of a level that starts in the tile is a node and reaches
    // beyond the tile, its end is searched here, 8 lanes a level.
    static_assert(8 * (kMaxLevels + 1) <= kTopoT, "8 threads a level");
    {
        const int l = t >> 3;
        bool on = false;
        const int64_t last_p = t0 + kTopoT - 1;
        if (l <= D && t0 + kTopoT < n) {
            for (int q = kTopoW - 1; q >= 0; --q)
                if (s_run[l][q]) {
                    on = (s_node[l][q] >> (63 - __clzll(s_run[l][q]))) & 1ull;
                    break;
                }
        }
        const int64_t pe = on ? cl_off[cluster_of(keys[last_p], D) + 1] : 0;
        const int64_t e = run_end8(keys, on, last_p, pe, l <= D ? l : D, D);
        if (on && (t & 7) == 0) s_end[l] = e;
    }
    if (blockIdx.x == 0) {
        if (t <= kMaxLevels) lvl_off[t] = s_off[t <= D + 1 ? t : D + 1];
        if (t == 0) {
            int64_t total = 0;
            int deepest = 0;
            for (int l = 0; l <= D; ++l) {
                const int v = table[(int64_t)l * (ntile + 1) + ntile];
                total += v;
                if (v) deepest = l;
            }
            if (total > cap) atomicOr(&cnt[kErr], kErrNodeCap);
            cnt[kCntNodes] = total > cap ? 0ull : (unsigned long long)total;
            cnt[kCntMaxLevel] = (unsigned long long)deepest;
        }
    }
    if (s_off[D + 1] == 0) return;   // beyond the capacity (workgroup-uniform: a build has a root)
    __syncthreads();
    // place of the first node of level l that starts at or behind particle p of the tile
    auto before = [&](int l, int p) {
        const int pw = p >> 6;
        return s_pre[l][pw] + ((p & 63) ? __popcll(s_node[l][pw] & (~0ull >> (64 - (p & 63)))) : 0);
    };
    int leaves = 0;
    int place = first <= last ? before(first, t) : 0;
    for (int l = first; l <= last; ++l) {
        // the next start of a level-l run in the tile
        int e = -1;
        const uint64_t m = lane < 63 ? s_run[l][w] >> (lane + 1) : 0ull;
        if (m) e = t + 1 + (__ffsll((unsigned long long)m) - 1);
        for (int q = w + 1; e < 0 && q < kTopoW; ++q)
            if (s_run[l][q]) e = 64 * q + __ffsll((unsigned long long)s_run[l][q]) - 1;
        int64_t end;
        if (e >= 0) {
            end = t0 + e;
        } else if (t0 + kTopoT >= n) {
            end = n;   // the run reaches the end of the last cluster
        } else {
            end = s_end[l];
        }
        const int count = (int)(end - i);
        const bool inner = count > n_leaf && l < D;
        int child = -1, nch = 0;
        if (inner) {
            child = before(l + 1, t);
            nch = e >= 0 ? before(l + 1, e) - child : (end == t0 + kTopoT ? before(l + 1, kTopoT) - child : -1);
        }
        node.set_range(place, make_int4((int)i, count, child, nch));
        leaves += inner ? 0 : 1;
        place = child;
    }
    for (int o = 32; o > 0; o >>= 1) leaves += __shfl_xor(leaves, o, 64);
    if (lane == 0 && leaves) atomicAdd(&s_leaves, leaves);
    __syncthreads();
    // one atomic per workgroup: a single counter serialises same-address atomics
    if (t == 0 && s_leaves) atomicAdd(&cnt[kCntLeaves], (unsigned long long)s_leaves);
}

// ----------------------------------------------------------------- moments
// Leaves sum their particles, inner nodes their (contiguous) children, in order:
// M, the mass-weighted centre, the tight box, then the traceless quadrupole about
// the new centre (children's own quadrupoles shifted by the parallel-axis terms).
//
// Eight lanes a node: lane k loads part k (siblings are neighbours in memory) and
// forms its products, which pass through LDS to the lane that sums a component
// over the parts in order, so every sum rounds as one thread's loop would. A
// thread for a whole node waited for three dependent loads and a chain of eight
// parts' sums on every level: 3.8 us a level against 1.9.
struct MomLds {
    double v[10][66];     // component, 8 * node of the wave + part (padded: a component a lane, other banks)
    double r[17][8];      // component, node: M, sums or centre (3), box lo (3), hi (3), quadrupole (6), 0
};

__device__ inline void lds_order() {
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// Moments of the node b (range rg) of this lane group; `on`: the group has one.
// kids_end: end of the next level's nodes. A node whose children were not counted
// (-1 of them) holds those that start inside it. All lanes of the wave take part.
__device__ inline void moments_group(MomLds& L, bool on, int b, int4 rg, int kids_end,
                                     const double* __restrict__ x, const double* __restrict__ y,
                                     const double* __restrict__ z, const double* __restrict__ m, NodePlanes node,
                                     Mom64Planes q64, Mom32Planes q32) {
#pragma clang fp contract(off)
    const int lane = threadIdx.x & 63, g = lane & 7, nd = lane >> 3;
    const bool leaf = rg.z < 0;
    int nsub = leaf ? rg.y : rg.w;
    double M = 0.0, c[3] = {0.0, 0.0, 0.0}, lo[3] = {0.0, 0.0, 0.0}, hi[3] = {0.0, 0.0, 0.0};
    Mom64 mq = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
    const int kid = rg.z + g < kids_end ? rg.z + g : kids_end - 1;   // (inner nodes: the level has nodes)
    if (on && leaf) {
        if (g < nsub) {
            const int j = rg.x + g;
            M = m[j];
            c[0] = x[j]; c[1] = y[j]; c[2] = z[j];
            for (int d = 0; d < 3; ++d) { lo[d] = c[d]; hi[d] = c[d]; }
        }
    } else if (on) {
        mq = q64.load(kid);
        M = mq.M;
        node.com(kid, c);
        node.box(kid, lo, hi);
    }
    const bool uncounted = on && !leaf && rg.w < 0;
    if (__ballot(uncounted)) {
        const bool in = uncounted && rg.z + g < kids_end && node.range(kid).x < rg.x + rg.y;
        const uint64_t k = __ballot(in);
        if (uncounted) {
            nsub = __popc((unsigned)((k >> (lane & 56)) & 255u));   // the children come first
            if (g == 0) node.set_range(b, make_int4(rg.x, rg.y, rg.z, nsub));
        }
    }
    // parts beyond 8 (leaves of more than 8 particles) are summed by every lane in turn below
    const int n8 = nsub < 8 ? nsub : 8;
    L.v[0][lane] = M;
    for (int d = 0; d < 3; ++d) {
        L.v[1 + d][lane] = M * c[d];
        L.v[4 + d][lane] = lo[d];
        L.v[7 + d][lane] = hi[d];
    }
    lds_order();
    {
        // lanes 0 .. 3 sum M and M c, every lane but those of M takes a box side: lanes
        // 1 .. 3 lo, 4 .. 6 hi (min of the negatives: exact)
        const int ks = g < 4 ? g : 3, kb = g >= 1 && g < 7 ? 3 + g : 4;
        const double flip = kb < 7 ? 1.0 : -1.0;
        double a = 0.0, e = INFINITY, u[8], v[8];
#pragma unroll
        for (int p = 0; p < 8; ++p) {
            u[p] = L.v[ks][8 * nd + p];
            v[p] = L.v[kb][8 * nd + p];
        }
#pragma unroll
        for (int p = 0; p < 8; ++p) {
            a = p < n8 ? a + u[p] : a;
            e = p < n8 ? fmin(e, v[p] * flip) : e;
        }
        if (on && leaf) {
            // leaves of more than 8 particles: the loads of four at a time, in flight together
            // (build of 131072 particles in leaves of up to 32 in 319 -> 270 us, of 1048576
            // 567 -> 504; eight at a time, in more registers, 311 and 554)
            const double* ps = (g == 1 ? x : (g == 2 ? y : z)) + rg.x;
            const double* pb = (kb % 3 == 1 ? x : (kb % 3 == 2 ? y : z)) + rg.x;
#pragma unroll 4
            for (int p = 8; p < nsub; ++p) {
                const double mj = m[rg.x + p], xs = ps[p];
                a = a + (g == 0 ? mj : mj * xs);
                e = fmin(e, pb[p] * flip);
            }
        }
        if (g < 4) L.r[g][nd] = a;
        if (g >= 1 && g < 7) L.r[kb][nd] = e * flip;
        if (g == 7) L.r[16][nd] = 0.0;
    }
    lds_order();
    const double Ms = L.r[0][nd];
    if (g >= 1 && g < 4) {
        const double s = L.r[g][nd];
        L.r[g][nd] = Ms > 0.0 ? s / Ms : (L.r[3 + g][nd] + L.r[6 + g][nd]) * 0.5;
    }
    lds_order();
    const double com[3] = {L.r[1][nd], L.r[2][nd], L.r[3][nd]};
    {
        const double dx = c[0] - com[0], dy = c[1] - com[1], dz = c[2] - com[2];
        const double r2 = dx * dx + dy * dy + dz * dz;
        L.v[0][lane] = mq.qxx + M * (3.0 * dx * dx - r2);
        L.v[1][lane] = mq.qyy + M * (3.0 * dy * dy - r2);
        L.v[2][lane] = mq.qzz + M * (3.0 * dz * dz - r2);
        L.v[3][lane] = mq.qxy + M * (3.0 * dx * dy);
        L.v[4][lane] = mq.qxz + M * (3.0 * dx * dz);
        L.v[5][lane] = mq.qyz + M * (3.0 * dy * dz);
    }
    lds_order();
    if (g < 6) {
        double a = 0.0;
        double u[8];
#pragma unroll
        for (int p = 0; p < 8; ++p) u[p] = L.v[g][8 * nd + p];
#pragma unroll
        for (int p = 0; p < 8; ++p)
            if (p < n8) a = a + u[p];
        if (on && leaf) {
#pragma unroll 4
            for (int p = 8; p < nsub; ++p) {
                const int j = rg.x + p;
                const double dx = x[j] - com[0], dy = y[j] - com[1], dz = z[j] - com[2];
                const double r2 = dx * dx + dy * dy + dz * dz, mj = m[j];
                const double e = g == 0 ? 3.0 * dx * dx - r2 : g == 1 ? 3.0 * dy * dy - r2 : g == 2 ? 3.0 * dz * dz - r2
                                 : g == 3 ? 3.0 * dx * dy : g == 4 ? 3.0 * dx * dz : 3.0 * dy * dz;
                a = a + (0.0 + mj * e);
            }
        }
        L.r[10 + g][nd] = a;
    }
    lds_order();
    if (on) {
        // the results in pieces of two: lane 0 .. 3 the node's first four planes, lane 4
        // .. 7 the four of the FP64 moments; then the rest of the centre and the FP32
        // moments
        const int i0 = (int)((0xfdb01864u >> (4 * g)) & 15u);   // 4 6 8 1 | 0 11 13 15
        int i1 = (int)((0x0eca2975u >> (4 * g)) & 15u);         // 5 7 9 2 | 10 12 14 -
        if (g == 7) i1 = 16;
        double2* dst = g < 4 ? node.p + (int64_t)g * node.cap + b : q64.p + (int64_t)(g - 4) * q64.cap + b;
        *dst = make_double2(L.r[i0][nd], L.r[i1][nd]);
        if (g == 0) reinterpret_cast<double*>(node.plane(4) + b)[0] = L.r[3][nd];
        if (g == 1 || g == 2) {
            const double f = L.r[g == 1 ? 0 : 13][nd];
            const int k1 = g == 1 ? 10 : 14;
            q32.p[(int64_t)(g - 1) * q32.cap + b] =
                make_float4((float)f, (float)L.r[k1][nd], (float)L.r[k1 + 1][nd], (float)L.r[g == 1 ? 12 : 16][nd]);
        }
    }
    lds_order();
}

// A node's children start inside it, so the nodes that lie inside one tile of
// kMomTiles topology tiles (1024 particles) depend on no other tile: a workgroup
// takes them level by level, with barriers for launches.
constexpr int kMomTiles = 4;
constexpr int kMomT = 512;
__global__ __launch_bounds__(kMomT) void k_moments_tile(int64_t n, int D, int64_t ntile, int64_t cap,
                                                        const int32_t* __restrict__ table,
                                                        const double* __restrict__ x, const double* __restrict__ y,
                                                        const double* __restrict__ z, const double* __restrict__ m,
                                                        NodePlanes node, Mom64Planes q64, Mom32Planes q32) {
    __shared__ MomLds s_m[kMomT / 64];
    __shared__ int s_off[64];
    __shared__ int s_b[kMaxLevels + 1][2];
    const int t = threadIdx.x;
    if (t < 64) level_offsets(table, ntile, D, cap, s_off);
    __syncthreads();
    if (s_off[D + 1] == 0) return;
    const int64_t a = (int64_t)blockIdx.x * kMomTiles, e = a + kMomTiles < ntile ? a + kMomTiles : ntile;
    if (t <= D) {
        s_b[t][0] = s_off[t] + table[(int64_t)t * (ntile + 1) + a];
        s_b[t][1] = s_off[t] + table[(int64_t)t * (ntile + 1) + e];
    }
    __syncthreads();
    const int64_t pend = e * kTopoT < n ? e * kTopoT : n;
    for (int l = D; l >= 0; --l) {
        const int b0 = s_b[l][0], b1 = s_b[l][1];
        if (b0 == b1) continue;   // workgroup-uniform
        const int kids_end = s_off[l + 2 <= D + 1 ? l + 2 : D + 1];
        for (int w0 = b0 + (t >> 6) * 8; w0 < b1; w0 += kMomT / 8) {   // 8 nodes a wave
            const int b = w0 + ((t & 63) >> 3);
            const int4 rg = node.range(b < b1 ? b : b1 - 1);
            const bool on = b < b1 && (int64_t)rg.x + rg.y <= pend;
            moments_group(s_m[t >> 6], on, b, rg, kids_end, x, y, z, m, node, q64, q32);
        }
        __syncthreads();
    }
}

// The nodes that reach beyond a unit of `inner` topology tiles but not beyond
// one of `outer`: of a level, only the last node that starts in a unit can reach
// beyond it. One workgroup per outer unit, eight lanes per inner unit, level by
// level; levels without such nodes are skipped.
// kStradU of them at a time: 64, or 128 where that saves a second launch (65537 to
// 131072 particles: 100003 build in 202 us with two, 187 with one of 1024 threads;
// with more units than that the larger workgroups cost 6 us at 524288).
template <int kStradU>
__global__ __launch_bounds__(8 * kStradU) void k_moments_straddle(int64_t n, int D, int64_t ntile, int64_t cap,
                                                              int64_t inner, int64_t outer,
                                                              const int32_t* __restrict__ table,
                                                              const double* __restrict__ x,
                                                              const double* __restrict__ y,
                                                              const double* __restrict__ z,
                                                              const double* __restrict__ m, NodePlanes node,
                                                              Mom64Planes q64, Mom32Planes q32) {
    __shared__ MomLds s_m[kStradU / 8];
    __shared__ int s_off[64];
    __shared__ unsigned s_levels;   // levels at which some unit has such a node
    __shared__ int s_cand[kMaxLevels][kStradU];   // of the first kStradU units: the node and its range
    __shared__ int4 s_rg[kMaxLevels][kStradU];
    const int t = threadIdx.x, g = t & 7;
    if (t < 64) level_offsets(table, ntile, D, cap, s_off);
    if (t == 0) s_levels = 0u;
    __syncthreads();
    if (s_off[D + 1] == 0) return;
    const int64_t o0 = (int64_t)blockIdx.x * outer, o1 = o0 + outer < ntile ? o0 + outer : ntile;
    const int64_t oend = o1 * kTopoT < n ? o1 * kTopoT : n;
    const int64_t units = (o1 - o0 + inner - 1) / inner;
    // the last node of level l that starts in unit u and its range; -1 unless it
    // reaches out of the unit and not out of the outer one
    auto candidate = [&](int64_t u, int l, int4& rg) -> int {
        const int64_t a = o0 + u * inner, e = a + inner < o1 ? a + inner : o1;
        const int c0 = table[(int64_t)l * (ntile + 1) + a], c1 = table[(int64_t)l * (ntile + 1) + e];
        if (c1 == c0) return -1;
        const int b = s_off[l] + c1 - 1;
        rg = node.range(b);
        const int64_t end = (int64_t)rg.x + rg.y;
        return end > e * kTopoT && end <= oend ? b : -1;
    };
    for (int64_t u = t >> 3; u < units; u += kStradU) {   // a lane group's levels, 8 at a time
        unsigned mask = 0;
        int4 rg = make_int4(0, 0, -1, 0);
        for (int l = g; l <= D; l += 8) {
            const int b = candidate(u, l, rg);
            mask |= b >= 0 ? 1u << l : 0u;
            if (u < kStradU) {
                s_cand[l][u] = b;
                s_rg[l][u] = rg;
            }
        }
        if (mask) atomicOr(&s_levels, mask);
    }
    __syncthreads();
    unsigned levels = s_levels;
    while (levels) {
        const int l = 31 - __clz(levels);
        levels &= ~(1u << l);
        const int kids_end = s_off[l + 2 <= D + 1 ? l + 2 : D + 1];
        for (int64_t u0 = (t >> 6) * 8; u0 < units; u0 += kStradU) {
            const int64_t u = u0 + ((t & 63) >> 3);
            int4 rg = make_int4(0, 0, -1, 0);
            int b = -1;
            if (u < units) {
                if (u < kStradU) {
                    b = s_cand[l][u];
                    rg = s_rg[l][u];
                } else {
                    b = candidate(u, l, rg);
                }
            }
            if (b < 0) rg = make_int4(0, 0, -1, 0);
            if (__ballot(b >= 0))
                moments_group(s_m[t >> 6], b >= 0, b, rg, kids_end, x, y, z, m, node, q64, q32);
        }
        __syncthreads();
    }
}

// ------------------------------------------------------------------ groups
// A node is "big" if it holds more than n_crit particles or its tight box is
// larger (largest side) than the cluster's size limit S. Every big node splits
// into walk groups: a big leaf into runs of n_crit particles, or into single
// particles if its box exceeds S; an inner node packs its consecutive
// children that are not big, greedily in order, into groups of at most
// n_crit particles whose joint box stays within S (a big child interrupts the
// run). A root that is not big is one group. S = 2^5 x 2^e for the octave e
// (2^e <= x < 2^(e+1)) holding the median box size of the groups formed with
// S = infinity (first pass, histogram only). The first particle of each group
// is flagged; a scan of the flags numbers the groups in particle order.
constexpr int kGroupLimitLog2 = 5;

__device__ inline double box_extent(const double* lo, const double* hi) {
    double e = 0.0;
    for (int k = 0; k < 3; ++k)
        if (hi[k] - lo[k] > e) e = hi[k] - lo[k];
    return e;
}

__device__ inline int octave_index(double x) {
    if (!(x > 0.0)) return 0;
    int e = ilogb(x);   // 2^e <= x < 2^(e+1)
    e = e < -64 ? -64 : (e > 63 ? 63 : e);
    return e + 64;
}

// emit one group: first pass -> octave histogram of its box size; second
// pass -> flag its first particle and store its length
template <bool HIST>
__device__ inline void emit_group(int begin, int count, const double* lo, const double* hi, unsigned* hist,
                                  int32_t* flag, int32_t* len, double* box) {
    if (HIST) {
        atomicAdd(&hist[octave_index(box_extent(lo, hi))], 1u);
    } else {
        flag[begin] = 1;
        len[begin] = count;
        for (int k = 0; k < 3; ++k) {
            box[6 * (int64_t)begin + k] = lo[k];
            box[6 * (int64_t)begin + 3 + k] = hi[k];
        }
    }
}

// The runs of the wave's big leaves (run: their length, 0 for lanes without one; slot:
// their histogram), a lane a run: leaf of 20000 particles in one cell of the finest
// level 2809 -> 40 us, and 2623 -> 35 for the pass that writes the groups (a lane a leaf
// waited for every particle in turn).
template <bool HIST>
__device__ inline void big_leaf_runs(int lane, int begin, int count, int run, int64_t slot,
                                     const double* __restrict__ x, const double* __restrict__ y,
                                     const double* __restrict__ z, unsigned* __restrict__ hist,
                                     int32_t* __restrict__ flag, int32_t* __restrict__ len,
                                     double* __restrict__ box) {
    const int runs = run ? (count + run - 1) / run : 0;
    const int incl = wave_incl_scan(runs, lane);   // (at most n + 64)
    const int total = last_lane(incl);
    for (int q0 = 0; q0 < total; q0 += 64) {
        const int q = q0 + lane;
        int src = 0;   // the first lane with q < incl
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) src += __shfl(incl, src + o - 1, 64) <= q ? o : 0;
        const int rl = __shfl(run, src, 64), first = __shfl(incl - runs, src, 64);
        const int lb = __shfl(begin, src, 64), le = lb + __shfl(count, src, 64);
        const int64_t sl = __shfl((long long)slot, src, 64);
        if (q >= total) continue;   // (past the last run)
        const int s0 = lb + (q - first) * rl, e0 = min(s0 + rl, le);
        double lo[3] = {x[s0], y[s0], z[s0]}, hi[3] = {lo[0], lo[1], lo[2]};
#pragma unroll 4
        for (int j = s0 + 1; j < e0; ++j) {
            const double v[3] = {x[j], y[j], z[j]};
            for (int k = 0; k < 3; ++k) {
                if (v[k] < lo[k]) lo[k] = v[k];
                if (v[k] > hi[k]) hi[k] = v[k];
            }
        }
        emit_group<HIST>(s0, e0 - s0, lo, hi, hist + sl * kOctaves, flag, len, box);
    }
}

template <bool HIST>
__global__ __launch_bounds__(256) void k_group_pass(NodePlanes node,
                             const unsigned long long* __restrict__ n_dev,
                             const uint64_t* __restrict__ keys, int D, int n_crit,
                             const double* __restrict__ x, const double* __restrict__ y,
                             const double* __restrict__ z, const double* __restrict__ cl_S,
                             unsigned* __restrict__ hist, int nc, int reps, int32_t* __restrict__ flag,
                             int32_t* __restrict__ len, double* __restrict__ box) {
    const int64_t nn = (int64_t)*n_dev;
    const int lane = threadIdx.x & 63;
    // (the loop is wave-uniform: all lanes take part in big_leaf_runs)
    for (int64_t b0 = (int64_t)blockIdx.x * blockDim.x + (threadIdx.x - lane); b0 < nn;
         b0 += (int64_t)gridDim.x * blockDim.x) {
        const int64_t b = b0 + lane;
        const bool on = b < nn;
        WNode w;
        w.begin = w.count = w.nchild = 0;
        int64_t slot = 0;
        double S = INFINITY, ext = 0.0;
        bool big = false;
        if (on) {
            node.box(b, w.lo, w.hi);
            const int4 rg = node.range(b);
            w.begin = rg.x; w.count = rg.y; w.first_child = rg.z; w.nchild = rg.w;
            const int c = cluster_of(keys[w.begin], D);
            if (!HIST) S = cl_S[c];
            slot = (int64_t)(b % reps) * nc + c;
            ext = box_extent(w.lo, w.hi);
            big = w.count > n_crit || ext > S;
        }
        unsigned* h = hist + slot * kOctaves;
        if (on && b < nc && !big) emit_group<HIST>(w.begin, w.count, w.lo, w.hi, h, flag, len, box);
        const int run = !big || w.nchild != 0 ? 0 : (ext > S ? 1 : n_crit);   // of a big leaf
        if (__ballot(run != 0)) big_leaf_runs<HIST>(lane, w.begin, w.count, run, slot, x, y, z, hist, flag, len, box);
        if (!big || run != 0) continue;
        int run_begin = 0, run_count = 0;
        double rlo[3] = {0, 0, 0}, rhi[3] = {0, 0, 0};
        // the children's boxes and counts are loaded together (one memory
        // latency per node, not one per child); the loops are unrolled so the
        // arrays stay in registers
        const int nch = w.nchild;
        double alo[8][3], ahi[8][3];
        int acnt[8], abeg[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            if (u < nch) {
                node.box(w.first_child + u, alo[u], ahi[u]);
                const int4 cr = node.range(w.first_child + u);
                acnt[u] = cr.y;
                abeg[u] = cr.x;
            }
        }
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            if (u >= nch) break;
            const double clo[3] = {alo[u][0], alo[u][1], alo[u][2]};
            const double chi[3] = {ahi[u][0], ahi[u][1], ahi[u][2]};
            const int cc = acnt[u];
            if (cc > n_crit || box_extent(clo, chi) > S) {
                if (run_count > 0) emit_group<HIST>(run_begin, run_count, rlo, rhi, h, flag, len, box);
                run_count = 0;
                continue;
            }
            double ulo[3], uhi[3];
            for (int k = 0; k < 3; ++k) {
                ulo[k] = (run_count > 0 && rlo[k] < clo[k]) ? rlo[k] : clo[k];
                uhi[k] = (run_count > 0 && rhi[k] > chi[k]) ? rhi[k] : chi[k];
            }
            if (run_count > 0 && (run_count + cc > n_crit || box_extent(ulo, uhi) > S)) {
                emit_group<HIST>(run_begin, run_count, rlo, rhi, h, flag, len, box);
                run_count = 0;
                for (int k = 0; k < 3; ++k) { ulo[k] = clo[k]; uhi[k] = chi[k]; }
            }
            if (run_count == 0) run_begin = abeg[u];
            run_count += cc;
            for (int k = 0; k < 3; ++k) { rlo[k] = ulo[k]; rhi[k] = uhi[k]; }
        }
        if (run_count > 0) emit_group<HIST>(run_begin, run_count, rlo, rhi, h, flag, len, box);
    }
}

// one block per cluster: 8 threads per octave sum the histogram copies (one
// batch of loads each), then the size limit from the median octave of the
// first pass (the first octave whose running count reaches half the groups,
// found by a scan over the octaves)
constexpr int kLimitT = 8 * kOctaves;
__global__ __launch_bounds__(kLimitT) void k_group_limit(const unsigned* __restrict__ hist, int nc,
                                                         int reps, double* __restrict__ cl_S) {
    static_assert(kOctaves == 128, "two waves scan the octaves");
    __shared__ int64_t s_part[8][kOctaves];
    __shared__ int64_t s_w[2];
    const int c = blockIdx.x, t = threadIdx.x, oct = t & (kOctaves - 1), part = t / kOctaves;
    int64_t v = 0;
#pragma unroll 8
    for (int r = part; r < reps; r += 8) v += hist[((int64_t)r * nc + c) * kOctaves + oct];
    s_part[part][oct] = v;
    __syncthreads();
    // the first two waves scan the octaves; every wave reaches both barriers
    const int i = t, lane = i & 63, w = i >> 6;
    int64_t inc = 0;
    v = 0;
    if (i < kOctaves) {
        for (int k = 0; k < 8; ++k) v += s_part[k][i];
        inc = v;   // inclusive running count over octaves 0..i
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const int64_t u = __shfl_up(inc, o, 64);
            if (lane >= o) inc += u;
        }
        if (lane == 63) s_w[w] = inc;
    }
    __syncthreads();
    if (i >= kOctaves) return;
    if (w == 1) inc += s_w[0];
    const int64_t total = s_w[0] + s_w[1];
    const int64_t need = (total + 1) / 2;
    // the first octave whose running count reaches need (octave 0 when empty)
    if (inc >= need && inc - v < need) cl_S[c] = ldexp(1.0, i - 64 + kGroupLimitLog2);
    else if (i == 0 && need == 0) cl_S[c] = ldexp(1.0, -64 + kGroupLimitLog2);
}

// Groups in particle order: the flags of a tile of kGrpT * kGrpI particles are
// counted, then (second launch) ranked, behind the counts of the tiles before,
// and every group found is copied to its place. Level-0 nodes are the clusters'
// roots in cluster order. Block 0 hands the build's error
// bits to the host.
constexpr int kGrpT = 256;
constexpr int kGrpI = 4;
constexpr int kGrpTile = kGrpT * kGrpI;
constexpr int kGrpFew = 8;

__global__ __launch_bounds__(kGrpT) void k_group_count(const int32_t* __restrict__ flag, int64_t n,
                                                       int32_t* __restrict__ tmp) {
    __shared__ int s_w[kGrpT / 64];
    const int64_t base = (int64_t)blockIdx.x * kGrpTile;
    int c = 0;
#pragma unroll
    for (int k = 0; k < kGrpI; ++k) {
        const int64_t i = base + k * kGrpT + threadIdx.x;
        c += __popcll(__ballot(i < n && flag[i] != 0));
    }
    if ((threadIdx.x & 63) == 0) s_w[threadIdx.x >> 6] = c;
    __syncthreads();
    if (threadIdx.x == 0) {
        int v = 0;
        for (int q = 0; q < kGrpT / 64; ++q) v += s_w[q];
        tmp[blockIdx.x] = v;
    }
}

__global__ __launch_bounds__(kGrpT) void k_group_fill(const int32_t* __restrict__ flag,
                                                      const int32_t* __restrict__ len, int64_t n,
                                                      const int32_t* __restrict__ tmp, int64_t nb,
                                                      const uint64_t* __restrict__ keys, int D,
                                                      const double* __restrict__ box, GroupArrays g,
                                                      unsigned long long* __restrict__ cnt,
                                                      unsigned long long* __restrict__ host_err) {
    __shared__ int s_w[kGrpT / 64];
    __shared__ int s_first[kGrpTile];   // the tile's groups: first particle in the tile
    const int t = threadIdx.x, lane = t & 63, w = t >> 6;
    const int64_t base = (int64_t)blockIdx.x * kGrpTile;
    int part = 0;
    if (tmp) {
        for (int64_t k = t; k < (int64_t)blockIdx.x; k += kGrpT) part += tmp[k];
    } else {   // few tiles: counted here
#pragma unroll 8
        for (int64_t k = t; k < base; k += kGrpT) part += flag[k] != 0 ? 1 : 0;
    }
    for (int o = 32; o > 0; o >>= 1) part += __shfl_xor(part, o, 64);
    if (lane == 0) s_w[w] = part;
    __syncthreads();
    int off = 0;
    for (int q = 0; q < kGrpT / 64; ++q) off += s_w[q];
    __syncthreads();
    // a wave holds kGrpI * 64 consecutive particles
    const int p0 = w * (kGrpI * 64) + lane;
    uint64_t ball[kGrpI];
    int c = 0;
#pragma unroll
    for (int k = 0; k < kGrpI; ++k) {
        const int64_t i = base + p0 + 64 * k;
        ball[k] = __ballot(i < n && flag[i] != 0);
        c += __popcll(ball[k]);
    }
    if (lane == 0) s_w[w] = c;
    __syncthreads();
    int at = 0, total = 0;
    for (int q = 0; q < kGrpT / 64; ++q) {
        at += q < w ? s_w[q] : 0;
        total += s_w[q];
    }
#pragma unroll
    for (int k = 0; k < kGrpI; ++k) {
        if ((ball[k] >> lane) & 1ull) s_first[at + popc_below(ball[k])] = p0 + 64 * k;
        at += __popcll(ball[k]);
    }
    __syncthreads();
    if ((int64_t)blockIdx.x == nb - 1 && t == 0) cnt[kCntGroups] = (unsigned long long)(off + total);
    if (blockIdx.x == 0 && t == 0) *host_err = cnt[kErr];   // (every kernel that sets a bit is done)
    for (int q = t; q < total; q += kGrpT) {
        const int64_t b = base + s_first[q];
        const int64_t gi = (int64_t)off + q;
        const int c = cluster_of(keys[b], D);
        for (int k = 0; k < 3; ++k) {
            g.lo[3 * gi + k] = box[6 * b + k];
            g.hi[3 * gi + k] = box[6 * b + 3 + k];
        }
        g.begin[gi] = (int32_t)b;
        g.count[gi] = len[b];
        g.cluster[gi] = c;
        g.root[gi] = c;
    }
}

inline int grid_for(int64_t n, int threads, int maxb = 4096) {
    int64_t b = (n + threads - 1) / threads;
    if (b < 1) b = 1;
    if (b > maxb) b = maxb;
    return (int)b;
}

}  // namespace

void launch_bbox(Dev& d, const BuildCfg& c, const double* pos, const double* mass, int nblk,
                 hipStream_t s) {
    (void)c;
    hipLaunchKernelGGL(k_bbox_part, dim3(nblk), dim3(BB_T), 0, s, pos, mass,
                       (const int64_t*)d.blk_range, d.blk_part, d.blk_bad, d.cnt);
}

void launch_keys(Dev& d, const BuildCfg& c, const double* pos, int nblk, hipStream_t s) {
    // d.blk_cluster is followed by the per-cluster block offsets (see host setup)
    hipLaunchKernelGGL(k_keys, dim3(nblk), dim3(BB_T), 0, s, pos, (const int64_t*)d.blk_range,
                       (const int32_t*)d.blk_cluster, (const int32_t*)(d.blk_cluster + nblk),
                       (const double*)d.blk_part, (const int32_t*)d.blk_bad, c.D,
                       sort_iota_in_alt(c.n) ? d.keys_alt : d.keys, d.cnt);
}

void launch_key_sort(Dev& d, const BuildCfg& c, hipStream_t s) {
    sort_iota(d.keys, d.perm, d.keys_alt, d.vals_alt, c.n, 3 * c.D + c.cbits, d.rs_hist, d.scan_tmp, d.sort_tmp, s);
}

int64_t topo_table_need(int64_t n) { return (kMaxLevels + 1) * ((n + kTopoT - 1) / kTopoT + 1); }

void launch_topology(Dev& d, const BuildCfg& c, const double* pos, const double* mass, hipStream_t s) {
    const int64_t ntile = (c.n + kTopoT - 1) / kTopoT;
    const int64_t hist_len = (int64_t)group_hist_reps(c.n_clusters) * c.n_clusters * kOctaves;
    hipLaunchKernelGGL(k_topo_count, dim3((unsigned)ntile), dim3(kTopoT), 0, s, (const uint64_t*)d.keys,
                       (const int64_t*)d.cl_off, c.n, c.D, c.n_leaf, d.p_lv, ntile, d.topo_table, pos, mass,
                       (const int32_t*)d.perm, d.x, d.y, d.z, d.m, d.g_flag, d.g_hist, hist_len);
    hipLaunchKernelGGL(k_topo_scan, dim3(c.D + 1), dim3(1024), 0, s, ntile, d.topo_table);
    hipLaunchKernelGGL(k_topo_emit, dim3((unsigned)ntile), dim3(kTopoT), 0, s, (const uint64_t*)d.keys,
                       (const int64_t*)d.cl_off, c.n, c.D, c.n_leaf, (const int32_t*)d.p_lv, ntile,
                       (const int32_t*)d.topo_table, c.node_cap, d.node, d.lvl_off, d.cnt);
}

void launch_moments(Dev& d, const BuildCfg& c, hipStream_t s) {
    const int64_t ntile = (c.n + kTopoT - 1) / kTopoT;
    hipLaunchKernelGGL(k_moments_tile, dim3((unsigned)((ntile + kMomTiles - 1) / kMomTiles)), dim3(kMomT), 0, s,
                       c.n, c.D, ntile, c.node_cap, (const int32_t*)d.topo_table, (const double*)d.x,
                       (const double*)d.y, (const double*)d.z, (const double*)d.m, d.node, d.q64, d.q32);
    // units of 1024 particles, then of 64 times that; the last launch takes all
    auto straddle = [&](auto kernel, int64_t u, int64_t inner, int64_t outer) {
        const int64_t blocks = (ntile + outer - 1) / outer;
        hipLaunchKernelGGL(kernel, dim3((unsigned)blocks), dim3((unsigned)(8 * u)), 0, s, c.n, c.D, ntile, c.node_cap,
                           inner, outer, (const int32_t*)d.topo_table, (const double*)d.x, (const double*)d.y,
                           (const double*)d.z, (const double*)d.m, d.node, d.q64, d.q32);
    };
    constexpr int64_t kU = 64;
    if (ntile > kMomTiles * kU && ntile <= 2 * kMomTiles * kU) {
        straddle(k_moments_straddle<2 * kU>, 2 * kU, kMomTiles, ntile);
    } else if (ntile > kMomTiles) {
        const bool one = ntile <= kMomTiles * kU;
        straddle(k_moments_straddle<kU>, kU, kMomTiles, one ? ntile : kMomTiles * kU);
        if (!one) straddle(k_moments_straddle<kU>, kU, kMomTiles * kU, ntile);
    }
}

int64_t group_tmp_need(int64_t n) { return (n + kGrpTile - 1) / kGrpTile; }

void launch_groups(Dev& d, const BuildCfg& c, hipStream_t s) {
    const int64_t n = c.n;
    const unsigned long long* n_nodes = d.cnt + kCntNodes;
    const int gb = grid_for(n, 256, 2048);   // about half as many nodes as particles
    const int reps = group_hist_reps(c.n_clusters);
    hipLaunchKernelGGL(k_group_pass<true>, dim3(gb), dim3(256), 0, s, d.node, n_nodes,
                       (const uint64_t*)d.keys, c.D, c.n_crit, (const double*)d.x, (const double*)d.y,
                       (const double*)d.z, (const double*)d.cl_S, d.g_hist, c.n_clusters, reps, d.g_flag, d.g_len,
                       d.g_box);
    hipLaunchKernelGGL(k_group_limit, dim3(c.n_clusters), dim3(kLimitT), 0, s,
                       (const unsigned*)d.g_hist, c.n_clusters, reps, d.cl_S);
    hipLaunchKernelGGL(k_group_pass<false>, dim3(gb), dim3(256), 0, s, d.node, n_nodes,
                       (const uint64_t*)d.keys, c.D, c.n_crit, (const double*)d.x, (const double*)d.y,
                       (const double*)d.z, (const double*)d.cl_S, d.g_hist, c.n_clusters, reps, d.g_flag, d.g_len,
                       d.g_box);
    const int64_t nb = group_tmp_need(n);
    // up to kGrpFew tiles the fill counts the tiles before its own itself: cheaper than
    // a launch (build of 700 particles 93 -> 91 us, 4096 133.5 -> 132.8)
    const bool few = nb <= kGrpFew;
    if (!few)
        hipLaunchKernelGGL(k_group_count, dim3((unsigned)nb), dim3(kGrpT), 0, s, (const int32_t*)d.g_flag, n,
                           d.g_tmp);
    hipLaunchKernelGGL(k_group_fill, dim3((unsigned)nb), dim3(kGrpT), 0, s, (const int32_t*)d.g_flag,
                       (const int32_t*)d.g_len, n, few ? nullptr : (const int32_t*)d.g_tmp, nb,
                       (const uint64_t*)d.keys, c.D,
                       (const double*)d.g_box, d.g, d.cnt, d.host_err);
}

}  // namespace pbh
