// core.hip -- core quantities from the 6 nearest neighbours of a particle
// sample (gfx950).
//
// Arnold, Baumgardt & Wang (2021) replace the neighbour-list based core
// estimate with a uniform sample of min(N, sqrt(5000 N)) particles whose 6
// nearest neighbours are found directly (Section 3.2), and feed the core
// density to the regularisation parameters R_min = 4 r_h / (N
// rho_core^(1/3)) and dT_min = 0.01 sqrt(eta / 0.02) sqrt(R_min^3)
// (Section 2.5). With the estimator of Casertano & Hut (1985), per
// sampled particle i:
//   rho_i = (sum of the masses of its 5 nearest neighbours) / ((4 pi/3) r_6^3)
// and over the sample x_d = sum rho x / sum rho, r_c^2 = sum rho^2 |x - x_d|^2
// / sum rho^2, rho_core = sum rho^2 / sum rho; N_core counts all particles
// inside r_c, r_h is the half-mass radius about x_d.
//
// The 6 nearest neighbours are exact (ordered by r^2 = (dx*dx + dy*dy) + dz*dz
// in FP64 without FMA, ties to the lower caller index), but found through the
// octree of the last build instead of a scan over all N: one wave per sampled
// particle seeds its list from the 64 particles around it in key order, then
// walks the tree and opens a node only if its box comes within the current
// 6th distance. The box distance is rounded exactly like a pair distance
// (monotone in every step), so it never exceeds the distance of a particle
// inside the box and no neighbour is pruned.
#include "pbh_internal.hpp"
#include "wave.hpp"

namespace pbh {

namespace {

// LDS traversal stack of one wave. A round takes as many nodes as leave kCoreDeep
// entries free with all their children on it, so a full stack is worked off a node
// at a time, which needs 7 entries a level. The search waits for the loads of its
// rounds, so waves in flight set its rate: 2048 entries without that rule let 18
// share a CU, 1024 let 32 (2^20 particles, 72407 samples: 312 -> 228 us).
constexpr int kCoreStack = 1024;
constexpr int kCoreDeep = 256;     // > 7 levels x 21 + 8

struct CoreParams {
    int64_t n;
    int64_t ns;
    const int32_t* sample;   // [ns] caller indices
    NodePlanes node;         // breadth-first nodes of the last build, root 0
    const double* x;         // sorted coordinates
    const double* y;
    const double* z;
    const int32_t* perm;     // key position -> caller index
    const int32_t* rank;     // caller index -> key position
    const double* mass;      // caller order
    double* rho;             // [ns] out
    unsigned long long* err; // kCore* flag bits
};

__device__ inline double pair_r2(double xj, double yj, double zj, double xi, double yi, double zi) {
#pragma clang fp contract(off)
    const double dx = xj - xi, dy = yj - yi, dz = zj - zi;
    return dx * dx + dy * dy + dz * dz;
}

// smaller of v and the value DPP control CTRL brings from another lane (lanes
// whose source lies outside keep their own)
template <int CTRL, int ROWS>
__device__ inline unsigned long long dpp_min_u64(unsigned long long v) {
    const int lo = (int)(unsigned)v, hi = (int)(unsigned)(v >> 32);
    const unsigned l = (unsigned)__builtin_amdgcn_update_dpp(lo, lo, CTRL, ROWS, 0xf, false);
    const unsigned h = (unsigned)__builtin_amdgcn_update_dpp(hi, hi, CTRL, ROWS, 0xf, false);
    const unsigned long long w = (unsigned long long)h << 32 | l;
    return w < v ? w : v;
}

// minimum over the wave, in every lane: within rows of 16 lanes by row shifts,
// then across the rows by row broadcasts into lane 63 (an exchange through LDS for
// each of the six steps took four times as long)
__device__ inline unsigned long long wave_min_u64(unsigned long long v) {
    v = dpp_min_u64<0x111, 0xf>(v);   // row_shr:1
    v = dpp_min_u64<0x112, 0xf>(v);   // row_shr:2
    v = dpp_min_u64<0x114, 0xf>(v);   // row_shr:4
    v = dpp_min_u64<0x118, 0xf>(v);   // row_shr:8
    v = dpp_min_u64<0x142, 0xa>(v);   // row_bcast:15
    v = dpp_min_u64<0x143, 0xc>(v);   // row_bcast:31
    const unsigned lo = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)v, 63);
    const unsigned hi = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)(v >> 32), 63);
    return (unsigned long long)hi << 32 | lo;
}

__device__ inline int wave_min_i32(int v) {
    for (int o = 32; o > 0; o >>= 1) {
        const int w = __shfl_xor(v, o, 64);
        v = w < v ? w : v;
    }
    return v;
}

// value of another lane, as the compiler's lane reads take 32 bits
__device__ inline double lane_f64(double v, int lane) {
    const unsigned long long b = (unsigned long long)__double_as_longlong(v);
    const unsigned lo = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)b, lane);
    const unsigned hi = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)(b >> 32), lane);
    return __longlong_as_double((long long)((unsigned long long)hi << 32 | lo));
}

// value of the lane before (lane 0 of each row of 16 keeps its own)
__device__ inline int from_lane_before(int v) {
    return __builtin_amdgcn_update_dpp(v, v, 0x111, 0xf, 0xf, false);   // row_shr:1
}

// The wave's current 6 nearest, ascending by (r^2, index): lane t < 6 holds entry
// t, empty entries are infinitely far with an index above any. An insertion is one
// comparison in all lanes and a shift by one lane (the whole list in every lane,
// with static selections, took 250 us against 228 at 2^20 particles, 72407
// samples).
struct Top6 {
    double d = __builtin_inf();
    int id = 0x7fffffff;
    double d5 = __builtin_inf();   // entry 5, in every lane
    int id5 = 0x7fffffff;
    // (r2, j) would enter the list
    __device__ bool better(double r2, int j) const { return r2 < d5 || (r2 == d5 && j < id5); }
    // insert the wave-uniform (r2, j); the 7th entry falls off
    __device__ void insert(double r2, int j) {
        const int lane = threadIdx.x;
        const uint64_t before = __ballot(d < r2 || (d == r2 && id < j)) & 0x3full;
        const int pos = __popcll(before);
        const unsigned long long b = (unsigned long long)__double_as_longlong(d);
        const unsigned lo = (unsigned)from_lane_before((int)(unsigned)b);
        const unsigned hi = (unsigned)from_lane_before((int)(unsigned)(b >> 32));
        const int idb = from_lane_before(id);
        const double db = __longlong_as_double((long long)((unsigned long long)hi << 32 | lo));
        d = lane > pos ? db : (lane == pos ? r2 : d);
        id = lane > pos ? idb : (lane == pos ? j : id);
        d5 = lane_f64(d, 5);
        id5 = __builtin_amdgcn_readlane(id, 5);
    }
    // merge the lanes' candidates (valid lanes with distance r2, index j, each
    // particle once in a search): the nearest enters until none beats entry 5
    __device__ void merge(bool valid, double r2, int j) {
        bool c = valid;
        for (int it = 0; it < 6; ++it) {
            c = c && better(r2, j);
            uint64_t who = __ballot(c);
            if (!who) return;
            if (who & (who - 1)) {   // several: the nearest, of equal ones the lowest index
                const unsigned long long key = c ? (unsigned long long)__double_as_longlong(r2) : ~0ull;
                const unsigned long long mk = wave_min_u64(key);
                const bool at = c && key == mk;
                who = __ballot(at);
                if (who & (who - 1)) {
                    const int mj = wave_min_i32(at ? j : 0x7fffffff);
                    who = __ballot(at && j == mj);
                }
            }
            const int l = __ffsll((unsigned long long)who) - 1;
            insert(lane_f64(r2, l), __builtin_amdgcn_readlane(j, l));
            c = c && (int)threadIdx.x != l;
        }
    }
};

__global__ __launch_bounds__(64) void k_core_knn(CoreParams p) {
    __shared__ int s_stack[kCoreStack];
    __shared__ int s_ex[64];
    __shared__ int s_beg[64];
    const int lane = threadIdx.x;
    const int64_t s = blockIdx.x;
    const int64_t i = p.sample[s];
    if ((uint64_t)i >= (uint64_t)p.n) {   // wave-uniform
        if (lane == 0) p.rho[s] = __builtin_nan("");
        atomicOr(p.err, lane == 0 ? kCoreBadSample : 0ull);
        return;
    }
    const int64_t k = p.rank[i];
    const double xi = p.x[k], yi = p.y[k], zi = p.z[k];
    Top6 T;
    // seed: the 64 key positions around i (n >= 7 gives at least 6 others)
    int64_t lo = k - 32;
    if (lo + 64 > p.n) lo = p.n - 64;
    if (lo < 0) lo = 0;
    {
        const int64_t q = lo + lane;
        const bool ok = q < p.n && q != k;
        const int64_t qq = q < p.n ? q : k;
        const double r2 = pair_r2(p.x[qq], p.y[qq], p.z[qq], xi, yi, zi);
        T.merge(ok, r2, p.perm[qq]);
    }
    // tree walk from the root, opening nodes within the current 6th distance
    bool overflow = false;
    s_stack[0] = 0;
    int top = 1;
    while (top > 0) {
        __syncthreads();
        const int room = (kCoreStack - kCoreDeep - top) / 7;
        const int npop = uni(min(top, room < 1 ? 1 : (room < 64 ? room : 64)));
        top -= npop;
        const bool has = lane < npop;
        const int nd = has ? s_stack[top + lane] : 0;
        __syncthreads();
        WNode w;
        p.node.box(nd, w.lo, w.hi);
        const int4 rg = p.node.range(nd);
        w.begin = rg.x; w.count = rg.y; w.first_child = rg.z; w.nchild = rg.w;
        const double c[3] = {xi, yi, zi};
        const bool open = has && !(box_pt_d2(w.lo, w.hi, c) > T.d5);
        const bool leaf = w.nchild == 0;
        const int nch = (open && !leaf) ? w.nchild : 0;
        const int incl = wave_incl_scan(nch, lane);
        const int tot = last_lane(incl);
        if (top + tot > kCoreStack) {
            overflow = true;
            break;
        }
        for (int q = 0; q < nch; ++q) s_stack[top + incl - nch + q] = w.first_child + q;
        top = uni(top + tot);
        // particles of opened leaves, 64 at a time
        const int v = (open && leaf) ? w.count : 0;
        const int li = wave_incl_scan(v, lane);
        const int total = last_lane(li);
        if (total == 0) continue;
        __syncthreads();
        s_ex[lane] = li - v;
        s_beg[lane] = w.begin;
        __syncthreads();
        for (int base = 0; base < total; base += 64) {
            const int sidx = base + lane;
            int f = 0;
#pragma unroll
            for (int st = 32; st > 0; st >>= 1)
                if (s_ex[f + st] <= sidx) f += st;
            const bool ok = sidx < total;
            const int64_t q = ok ? (int64_t)s_beg[f] + (sidx - s_ex[f]) : k;
            const double r2 = pair_r2(p.x[q], p.y[q], p.z[q], xi, yi, zi);
            T.merge(ok && (uint64_t)(q - lo) >= 64, r2, p.perm[q]);   // (the seed's are merged already)
        }
    }
    if (overflow) atomicOr(p.err, lane == 0 ? kCoreStackFull : 0ull);
    {
#pragma clang fp contract(off)
        const double m = lane < 5 ? p.mass[T.id] : 0.0;
        double m5 = 0.0;
        for (int t = 0; t < 5; ++t) m5 += lane_f64(m, t);
        const double r6 = sqrt(T.d5);
        if (lane == 0)
            p.rho[s] = overflow ? __builtin_nan("") : m5 / (4.0 / 3.0 * 3.14159265358979323846 * (T.d5 * r6));
    }
}

// rank[perm[k]] = k
__global__ void k_core_rank(int64_t n, const int32_t* __restrict__ perm, int32_t* __restrict__ rank) {
    const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (k < n) rank[perm[k]] = (int32_t)k;
}

// Sums over the sample in two levels, each in a fixed order: a workgroup of
// kStatT threads sums a chunk of kStatCh consecutive samples (thread t takes
// samples t, t + kStatT, ... of the chunk in that order, loads issued
// together, then a fixed tree over the threads), and one workgroup sums the
// chunk totals in chunk order the same way. First the density centre
// (sum rho, sum rho x), then the core density and radius (sum rho^2,
// sum rho^2 |x - x_d|^2). out: [0..2] x_d, [3] rho_core, [4] r_c, ...
// part: [0] the sum of rho; [8 + 4 c ..] the totals of chunk c.
constexpr int kStatT = 256;
constexpr int kStatB = 8;
constexpr int kStatCh = kStatT * kStatB;   // samples per chunk

__device__ inline double block_sum(double v, double* red) {
    const int t = threadIdx.x;
    __syncthreads();
    red[t] = v;
    __syncthreads();
    for (int h = kStatT / 2; h > 0; h >>= 1) {
        if (t < h) red[t] += red[t + h];
        __syncthreads();
    }
    return red[0];
}

// the samples of thread t in chunk c: caller index (-1: none or out of range,
// flagged by the search and never read), density and position
__device__ inline void chunk_samples(int64_t n, int64_t ns, const int32_t* __restrict__ sample,
                                     const double* __restrict__ pos, const double* __restrict__ rho,
                                     int64_t c, int t, int64_t (&iv)[kStatB], double (&rv)[kStatB],
                                     double (&xv)[kStatB], double (&yv)[kStatB], double (&zv)[kStatB]) {
#pragma unroll
    for (int u = 0; u < kStatB; ++u) {
        const int64_t s = c * kStatCh + t + (int64_t)kStatT * u;
        iv[u] = s < ns ? (int64_t)sample[s] : -1;
    }
#pragma unroll
    for (int u = 0; u < kStatB; ++u) {
        const int64_t s = c * kStatCh + t + (int64_t)kStatT * u;
        const bool ok = (uint64_t)iv[u] < (uint64_t)n;
        if (!ok) iv[u] = -1;
        const int64_t i = ok ? iv[u] : 0;
        rv[u] = ok ? rho[s] : 0.0;
        xv[u] = pos[3 * i];
        yv[u] = pos[3 * i + 1];
        zv[u] = pos[3 * i + 2];
    }
}

__global__ __launch_bounds__(kStatT) void k_core_sum1(int64_t n, int64_t ns, const int32_t* __restrict__ sample,
                                                      const double* __restrict__ pos,
                                                      const double* __restrict__ rho, double* __restrict__ part) {
#pragma clang fp contract(off)
    __shared__ double red[kStatT];
    int64_t iv[kStatB];
    double rv[kStatB], xv[kStatB], yv[kStatB], zv[kStatB];
    chunk_samples(n, ns, sample, pos, rho, blockIdx.x, threadIdx.x, iv, rv, xv, yv, zv);
    double sr = 0, sx = 0, sy = 0, sz = 0;
#pragma unroll
    for (int u = 0; u < kStatB; ++u) {
        if (iv[u] < 0) continue;
        sr += rv[u];
        sx += rv[u] * xv[u];
        sy += rv[u] * yv[u];
        sz += rv[u] * zv[u];
    }
    sr = block_sum(sr, red);
    sx = block_sum(sx, red);
    sy = block_sum(sy, red);
    sz = block_sum(sz, red);
    if (threadIdx.x == 0) {
        double* q = part + 8 + 4 * (int64_t)blockIdx.x;
        q[0] = sr; q[1] = sx; q[2] = sy; q[3] = sz;
    }
}

// totals of the first k (<= 4) values of every chunk, in chunk order
template <int K>
__device__ inline void chunk_totals(int64_t nc, const double* __restrict__ part, double* red, double (&tot)[K]) {
    double v[K];
    for (int k = 0; k < K; ++k) v[k] = 0.0;
    for (int64_t c = threadIdx.x; c < nc; c += kStatT)
        for (int k = 0; k < K; ++k) v[k] += part[8 + 4 * c + k];
    for (int k = 0; k < K; ++k) tot[k] = block_sum(v[k], red);
}

__global__ __launch_bounds__(kStatT) void k_core_centre(int64_t nc, double* __restrict__ part,
                                                        double* __restrict__ out) {
#pragma clang fp contract(off)
    __shared__ double red[kStatT];
    double tot[4];
    chunk_totals<4>(nc, part, red, tot);
    if (threadIdx.x == 0) {
        part[0] = tot[0];
        out[0] = tot[1] / tot[0];
        out[1] = tot[2] / tot[0];
        out[2] = tot[3] / tot[0];
    }
}

__global__ __launch_bounds__(kStatT) void k_core_sum2(int64_t n, int64_t ns, const int32_t* __restrict__ sample,
                                                      const double* __restrict__ pos,
                                                      const double* __restrict__ rho,
                                                      const double* __restrict__ out, double* __restrict__ part) {
#pragma clang fp contract(off)
    __shared__ double red[kStatT];
    const double xd = out[0], yd = out[1], zd = out[2];
    int64_t iv[kStatB];
    double rv[kStatB], xv[kStatB], yv[kStatB], zv[kStatB];
    chunk_samples(n, ns, sample, pos, rho, blockIdx.x, threadIdx.x, iv, rv, xv, yv, zv);
    double s2 = 0, s2d = 0;
#pragma unroll
    for (int u = 0; u < kStatB; ++u) {
        if (iv[u] < 0) continue;
        const double r = rv[u];
        const double dx = xv[u] - xd, dy = yv[u] - yd, dz = zv[u] - zd;
        const double dd = dx * dx + dy * dy + dz * dz;
        s2 += r * r;
        s2d += r * r * dd;
    }
    s2 = block_sum(s2, red);
    s2d = block_sum(s2d, red);
    if (threadIdx.x == 0) {
        double* q = part + 8 + 4 * (int64_t)blockIdx.x;
        q[0] = s2; q[1] = s2d;
    }
}

__global__ __launch_bounds__(kStatT) void k_core_radius(int64_t nc, const double* __restrict__ part,
                                                        double* __restrict__ out) {
#pragma clang fp contract(off)
    __shared__ double red[kStatT];
    double tot[2];
    chunk_totals<2>(nc, part, red, tot);
    if (threadIdx.x == 0) {
        out[3] = tot[0] / part[0];        // rho_core
        out[4] = sqrt(tot[1] / tot[0]);   // r_c
    }
}

// distance keys about x_d for the half-mass radius, and the core count (one
// device atomic per workgroup: atomics on one address serialise)
constexpr int kDistGrid = 1024;

__global__ __launch_bounds__(256) void k_core_dist(int64_t n, const double* __restrict__ pos,
                                                   const double* __restrict__ st,
                                                   uint64_t* __restrict__ key,
                                                   unsigned long long* __restrict__ ncore) {
#pragma clang fp contract(off)
    __shared__ unsigned long long s_cnt[4];
    const double xd = st[0], yd = st[1], zd = st[2], rc = st[4];
    unsigned long long cnt = 0;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
        const double dx = pos[3 * i] - xd, dy = pos[3 * i + 1] - yd, dz = pos[3 * i + 2] - zd;
        const double dd = dx * dx + dy * dy + dz * dz;
        cnt += dd < rc * rc ? 1ull : 0ull;
        key[i] = (uint64_t)__double_as_longlong(dd);   // dd >= 0: bit order is numeric order
    }
    for (int o = 32; o > 0; o >>= 1) cnt += __shfl_xor(cnt, o, 64);
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    if (lane == 0) s_cnt[w] = cnt;
    __syncthreads();
    if (w == 0) {   // all lanes of wave 0 take part; lane 0 adds the workgroup's count
        const unsigned long long tot = s_cnt[0] + s_cnt[1] + s_cnt[2] + s_cnt[3];
        if (tot) atomicAdd(ncore, lane == 0 ? tot : 0ull);
    }
}

// masses in distance order, summed per block of kCrossBlk (fixed order)
constexpr int kCrossBlk = 1024;

__global__ __launch_bounds__(kCrossBlk) void k_core_bsum(int64_t n, const int32_t* __restrict__ order,
                                                         const double* __restrict__ mass,
                                                         double* __restrict__ bsum) {
    __shared__ double red[kCrossBlk];
    const int64_t i = (int64_t)blockIdx.x * kCrossBlk + threadIdx.x;
    red[threadIdx.x] = i < n ? mass[order[i]] : 0.0;
    __syncthreads();
    for (int h = kCrossBlk / 2; h > 0; h >>= 1) {
        if ((int)threadIdx.x < h) red[threadIdx.x] += red[threadIdx.x + h];
        __syncthreads();
    }
    if (threadIdx.x == 0) bsum[blockIdx.x] = red[0];
}

// Replaces v[0 .. e - 1] by its running sums, added in order to cum, and returns
// the last (one thread; v holds zeros from e to the next multiple of 16). The
// chain of additions sets the pace: the next 16 values are read while it runs and
// no branch or comparison stands in it.
__device__ inline double run_in_order(double* v, int e, double cum) {
    double x[16];
#pragma unroll
    for (int u = 0; u < 16; ++u) x[u] = v[u];
    for (int k0 = 0; k0 < e; k0 += 16) {
        double nx[16];
        const int k1 = k0 + 16 < e ? k0 + 16 : k0;
#pragma unroll
        for (int u = 0; u < 16; ++u) nx[u] = v[k1 + u];
#pragma unroll
        for (int u = 0; u < 16; ++u) {
            cum += x[u];
            x[u] = cum;
        }
#pragma unroll
        for (int u = 0; u < 16; ++u) {
            v[k0 + u] = x[u];
            x[u] = nx[u];
        }
    }
    return cum;
}

// Half-mass radius (first distance at which the running mass reaches half the
// total) and the regularisation parameters, in one workgroup. Running sums are
// taken in order by one thread, kCrossBlk values at a time in LDS: of the block
// sums (left in bsum) and, once every thread has looked for the half among
// those, of the masses of the block that holds it. Searching while summing, one
// value read at a time, and a second pass of sums took 110 us at 2^20, this 34.
__global__ __launch_bounds__(kCrossBlk) void k_core_final(int64_t n, int64_t nblk, const int32_t* __restrict__ order,
                                                          const uint64_t* __restrict__ key,
                                                          const double* __restrict__ mass, double* __restrict__ bsum,
                                                          const unsigned long long* ncore, double eta,
                                                          double* __restrict__ st) {
#pragma clang fp contract(off)
    __shared__ double v[kCrossBlk];
    __shared__ double s_cum;
    __shared__ unsigned long long s_b, s_k;
    const int t = threadIdx.x;
    if (t == 0) {
        s_cum = 0.0;
        s_b = (unsigned long long)(nblk - 1);
    }
    for (int64_t c0 = 0; c0 < nblk; c0 += kCrossBlk) {
        const bool in = c0 + t < nblk;
        v[t] = in ? bsum[c0 + t] : 0.0;
        __syncthreads();
        if (t == 0) s_cum = run_in_order(v, nblk - c0 < kCrossBlk ? (int)(nblk - c0) : kCrossBlk, s_cum);
        __syncthreads();
        if (in) bsum[c0 + t] = v[t];
        __syncthreads();
    }
    const double half = 0.5 * s_cum;
    // the first block whose running sum is not below the half, or the last one
    for (int64_t k = t; k < nblk - 1; k += kCrossBlk)
        if (!(bsum[k] < half)) {
            atomicMin(&s_b, (unsigned long long)k);
            break;
        }
    __syncthreads();
    const int64_t b = (int64_t)s_b;
    const int64_t beg = b * kCrossBlk;
    const int len = (int)((b + 1) * kCrossBlk < n ? kCrossBlk : n - beg);
    v[t] = t < len ? mass[order[beg + t]] : 0.0;
    if (t == 0) s_k = (unsigned long long)(len - 1);
    __syncthreads();
    if (t == 0) run_in_order(v, len, b > 0 ? bsum[b - 1] : 0.0);
    __syncthreads();
    if (t < len - 1 && v[t] >= half) atomicMin(&s_k, (unsigned long long)t);
    __syncthreads();
    if (t == 0) {
        const double rh = sqrt(__longlong_as_double((long long)key[beg + (int64_t)s_k]));
        const double rmin = 4.0 * rh / ((double)n * cbrt(st[3]));
        st[5] = (double)*ncore;
        st[6] = rh;
        st[7] = rmin;
        st[8] = 0.01 * sqrt(eta / 0.02) * sqrt(rmin * rmin * rmin);
    }
}

}  // namespace

void launch_core(const CoreLaunch& c, hipStream_t s) {
    const int64_t n = c.n;
    hipLaunchKernelGGL(k_core_rank, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, n, c.perm, c.rank);
    CoreParams p;
    p.n = n;
    p.ns = c.ns;
    p.sample = c.sample;
    p.node = c.node;
    p.x = c.x; p.y = c.y; p.z = c.z;
    p.perm = c.perm;
    p.rank = c.rank;
    p.mass = c.mass;
    p.rho = c.rho;
    p.err = c.err;
    hipLaunchKernelGGL(k_core_knn, dim3((unsigned)c.ns), dim3(64), 0, s, p);
    const int64_t nc = (c.ns + kStatCh - 1) / kStatCh;   // sample chunks (ns >= 1)
    hipLaunchKernelGGL(k_core_sum1, dim3((unsigned)nc), dim3(kStatT), 0, s, n, c.ns, c.sample, c.pos,
                       (const double*)c.rho, c.bsum);
    hipLaunchKernelGGL(k_core_centre, dim3(1), dim3(kStatT), 0, s, nc, c.bsum, c.stats);
    hipLaunchKernelGGL(k_core_sum2, dim3((unsigned)nc), dim3(kStatT), 0, s, n, c.ns, c.sample, c.pos,
                       (const double*)c.rho, (const double*)c.stats, c.bsum);
    hipLaunchKernelGGL(k_core_radius, dim3(1), dim3(kStatT), 0, s, nc, (const double*)c.bsum, c.stats);
    const int64_t nb = (n + 255) / 256;
    hipLaunchKernelGGL(k_core_dist, dim3((unsigned)(nb < kDistGrid ? nb : kDistGrid)), dim3(256), 0, s, n, c.pos,
                       (const double*)c.stats, sort_iota_in_alt(n) ? c.keys_alt : c.keys, c.ncore);
    sort_iota(c.keys, c.vals, c.keys_alt, c.vals_alt, n, 64, c.hist, c.scan_tmp, c.sort_tmp, s);
    const int64_t nblk = (n + kCrossBlk - 1) / kCrossBlk;
    hipLaunchKernelGGL(k_core_bsum, dim3((unsigned)nblk), dim3(kCrossBlk), 0, s, n, (const int32_t*)c.vals,
                       c.mass, c.bsum);
    hipLaunchKernelGGL(k_core_final, dim3(1), dim3(kCrossBlk), 0, s, n, nblk, (const int32_t*)c.vals,
                       (const uint64_t*)c.keys, c.mass, c.bsum,
                       (const unsigned long long*)c.ncore, c.eta, c.stats);
}

// the cross-block sums of the half-mass search, and before them the sample
// sums' chunk totals (n >= the sample size)
int64_t core_bsum_len(int64_t n) {
    const int64_t a = (n + kCrossBlk - 1) / kCrossBlk, b = 8 + 4 * ((n + kStatCh - 1) / kStatCh);
    return a > b ? a : b;
}

}  // namespace pbh
