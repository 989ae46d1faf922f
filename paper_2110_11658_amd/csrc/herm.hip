// herm.hip -- Hermite integration of the irregular force with block time
// steps over one regular step, the inner loop of the P3T scheme (gfx950).
//
// Arnold, Baumgardt & Wang (2021), Section 2.2: between two regular kicks
// every particle moves under its irregular force F_I, integrated with the
// Hermite scheme on individual block steps. Per particle the state is x, v,
// a = F_I, j = dF_I/dt, its time tau_i and step dt_i = dt_max / 2^k, with
// dt_max = T / 4 (eq. dtmax) for a regular step T. Times are integer ticks of
// dt_max / 2^kHermK, so block times add exactly. One block:
//   tau' = min(tau_i + dt_i); the active particles and the members of their
//   neighbour lists are predicted to tau' with the P3T predictor (eq.
//   p3t-jpred-x, -dx: no regular force, the kicks carry it)
//     x_p = x + d v + d^2/2 a + d^3/6 j,   v_p = v + d a + d^2/2 j;
//   the active particles (tau_i + dt_i = tau') get F_I and its derivative at
//   the predicted state from their neighbour lists, then the 4th-order Hermite
//   corrector (d = dt_i, da = a - a1)
//     a2 = (-6 da - d (4 j + 2 j1)) / d^2,  a3 = (12 da + 6 d (j + j1)) / d^3
//     x = x_p + d^4/24 a2 + d^5/120 a3,     v = v_p + d^3/6 a2 + d^4/24 a3
//   and a new step from eq. dt (eta) with a^(0) = a1 + F_R, a^(1) = j1,
//   a^(2) = a2 + d a3, a^(3) = a3: at most twice the old step and dt_max,
//   rounded down to dt_max / 2^k dividing tau'. The corrector is the standard
//   Hermite one (Makino & Aarseth 1992).
// First steps (Section 2.1, after eq. dt: the higher derivatives are computed
// and the fourth-order criterion sets the initial step; steps are set afresh
// after every regular kick): with a = F_I and j = dF_I/dt of every particle
// at the start, the second and third derivatives of F_I along the motion
// under F_I come from the neighbour lists (relative accelerations a_j - a_i,
// relative jerks j_j - j_i), and eq. dt with a^(0) = a + F_R, a^(1) = j and
// those derivatives gives the first step; dt_max where its denominator is 0
// (no pair inside r_out). Expressions are evaluated as written (no contraction).
//
// A block is at most one launch: the next block time and its active particles from
// the level counts, prediction of each active particle and its list members in
// registers, force, corrector, new step, move to the new bucket. Particles are
// kept in one bucket per level, so it does not pass over all n particles. Blocks of
// few particles, which are most, follow one another inside one workgroup.
#include "irr_pair.hpp"
#include "pbh_internal.hpp"
#include "wave.hpp"

namespace pbh {

namespace {

__device__ inline double norm3(double x, double y, double z) {
#pragma clang fp contract(off)
    return sqrt(x * x + y * y + z * z);
}

// Block schedule by level. A particle at level k has dt_i = 2^(kHermK - k)
// ticks, and its time tau_i is a multiple of dt_i (the new step is chosen to
// divide the block time), with tau_i <= t < tau_i + dt_i at the current block
// time t. Its next time tau_i + dt_i is then the first multiple of dt_i after
// t, so the next block time tn = min(tau_i + dt_i) is the first multiple of
// the smallest occupied step after t, and particle i is active at tn exactly
// when dt_i divides tn, i.e. when k >= k* = kHermK - ctz(tn) (0 if that is
// negative). Particles are therefore kept in one bucket per level and a block
// takes whole buckets: no pass over all n particles per block. The corrected
// particles of a block (levels >= k*) move to their new levels, which are
// >= k* - 1 (the step at most doubles): buckets >= k* are refilled from zero
// and bucket k* - 1 is appended to.
//
// No workgroup reads what another one of its launch writes. Level counts, block
// time and k* have two slots by launch parity q: a launch reads slot q and writes
// q ^ 1. The counts of the corrected particles per level (new) have four by launch
// number: a launch reads its own, which the one before filled, appends to the next
// and clears the one after that. Buckets of the active levels are read from one of two buffers
// (bit k of the mask) and refilled in the other. And a particle's state has two
// records: a block reads the newest with a time before its own, and writes the
// corrected state over the older one, whose time (old or, once written, the
// block's own) never qualifies, so members that are corrected at the same moment
// are read as they were.
//
// A launch's first block may have any number of active particles. If they are few
// (kHermSolo), workgroup 0 takes them all, the others end, and it goes on with the
// following blocks as long as those are few as well, with nothing between them but
// a barrier of the workgroup; it stops before a large block and leaves the counts
// for the next launch. Deep levels hold few particles and make most of the blocks:
// of 617 in a regular step at 2^20 three quarters have at most 18 active. A block
// is a chain of dependent loads (bucket entry, list bounds, list entry, the times of
// the member's records, its record) and the corrector's divisions and roots, about
// 4 us in a row of small blocks; one of a launch of its own takes 7 to 12 us, and
// took 19 when prediction and force were two launches (regular step at 2^20 with two
// forces: 28.2 -> 20.6 ms; 16384 particles: 2.87 -> 1.23 ms). Two records side by
// side and the record's number in the bucket entry leave out one load and most
// of the address misses (22.0 -> 21.0 ms).
//
// Launches are enqueued in batches without waiting; once every particle has
// reached the end of the regular step the remaining launches are empty
// (kHermDone), and the one that finds it also sets a host-visible flag,
// which the host reads after a batch while the next one runs.
constexpr int kHermT = 512;       // threads per workgroup of a block
constexpr int kHermGrid = 512;    // workgroups
constexpr int kHermLanes = 8;     // lanes per active particle while that fits the grid, else one
constexpr int kHermSolo = 128;    // active particles of a block that one workgroup takes (64: the same time, 256: 1 % more)
constexpr int kHermInner = 64;    // blocks in a launch at most
constexpr int kSlotShift = 26;    // per-item scratch: level << 26 | rank in its workgroup
constexpr uint32_t kSlotMask = (1u << kSlotShift) - 1;
static_assert(kHermK < 63, "levels fit one wave");

__device__ inline unsigned long long* lev_cnt(const HermParams& p, int q) { return p.lev + kLevCnt + 64 * q; }
__device__ inline unsigned long long* lev_new(const HermParams& p, int b) { return p.lev + kLevNew + 64 * (b & 3); }

// One particle's state at its own time, as 16-byte pieces of its record:
// x y | z vx | vy vz | ax ay | az jx | jy jz | m tau | dt -
struct HermState {
    double x[3], v[3], a[3], j[3], m;
    int64_t tau, dt;
};

__device__ inline HermState load_state(const double2* __restrict__ r) {
    HermState s;
    const double2 q0 = r[0], q1 = r[1], q2 = r[2], q3 = r[3], q4 = r[4], q5 = r[5], q6 = r[6], q7 = r[7];
    s.x[0] = q0.x; s.x[1] = q0.y; s.x[2] = q1.x;
    s.v[0] = q1.y; s.v[1] = q2.x; s.v[2] = q2.y;
    s.a[0] = q3.x; s.a[1] = q3.y; s.a[2] = q4.x;
    s.j[0] = q4.y; s.j[1] = q5.x; s.j[2] = q5.y;
    s.m = q6.x;
    s.tau = __double_as_longlong(q6.y);
    s.dt = __double_as_longlong(q7.x);
    return s;
}

__device__ inline void store_state(double2* r, const HermState& s) {
    r[0] = make_double2(s.x[0], s.x[1]);
    r[1] = make_double2(s.x[2], s.v[0]);
    r[2] = make_double2(s.v[1], s.v[2]);
    r[3] = make_double2(s.a[0], s.a[1]);
    r[4] = make_double2(s.a[2], s.j[0]);
    r[5] = make_double2(s.j[1], s.j[2]);
    r[6] = make_double2(s.m, __longlong_as_double((long long)s.tau));
    r[7] = make_double2(__longlong_as_double((long long)s.dt), 0.0);
}

// Record `buf` (0 or 1) of particle i; the two are neighbours.
__device__ inline double2* record(const HermParams& p, int64_t i, int buf) { return p.rec + 8 * (2 * i + buf); }

__device__ inline int64_t record_time(const HermParams& p, int64_t i, int buf) {
    return __double_as_longlong(record(p, i, buf)[6].y);
}

// The record of particle i to read at block time tn: the newest with an earlier time.
__device__ inline int state_buffer(const HermParams& p, int64_t i, int64_t tn) {
    const int64_t t0 = record_time(p, i, 0), t1 = record_time(p, i, 1);
    return t1 < tn && (t0 >= tn || t1 > t0) ? 1 : 0;
}

// A bucket entry: the particle, and in the sign bit which record holds its state.
constexpr int32_t kInRec1 = (int32_t)0x80000000;

// The predicted position and velocity at time tn (the P3T predictor).
__device__ inline void predict(const HermParams& p, const HermState& s, int64_t tn, double* xp, double* vp) {
#pragma clang fp contract(off)
    const double d = (double)(tn - s.tau) * p.unit;
    const double d2 = d * d, d3 = d2 * d;
    for (int k = 0; k < 3; ++k) {
        xp[k] = s.x[k] + d * s.v[k] + 0.5 * d2 * s.a[k] + d3 / 6.0 * s.j[k];
        vp[k] = s.v[k] + d * s.a[k] + 0.5 * d2 * s.j[k];
    }
}

// The count of level k after a block that took the levels >= ks, from the count
// before it and the corrected particles `add` it left on the level.
__device__ inline long long merged_count(long long old, long long add, int ks, int k) {
    return k >= ks ? add : (k == ks - 1 ? old + add : old);
}

// The next block from the level counts (one wave, lane k holding count c of
// level k) and the current time t: its time tn, k*, the number of active
// particles and lane k's end in the active list (levels >= k* in order).
struct BlockPlan {
    long long tn;
    int nact, end, ks;
    bool done;
};

__device__ inline BlockPlan plan_block(long long c, long long t, unsigned long long tend) {
    const int k = threadIdx.x & 63;
    BlockPlan b;
    const int kmax = 63 - __clzll(__ballot(c > 0));   // deepest occupied level (n >= 1)
    b.done = t >= (long long)tend;
    const int sh = kHermK - kmax;
    b.tn = b.done ? (long long)tend : (((t >> sh) + 1) << sh);
    const int tz = __ffsll((unsigned long long)b.tn) - 1;
    b.ks = b.done ? kHermK + 1 : (tz >= kHermK ? 0 : kHermK - tz);
    const int a = k >= b.ks ? (int)c : 0;   // (n < 2^31)
    const int incl = wave_incl_scan(a, k);
    b.nact = last_lane(incl);
    b.end = incl;
    return b;
}

__device__ inline int32_t* bucket_of(const HermParams& p, int buf, int k) {
    return p.bucket + ((int64_t)buf * (kHermK + 1) + k) * p.n;
}

// entry t of the active list: level buckets ks, ks + 1, ... in turn, each in the
// buffer of its mask bit. end[k]: entries of levels up to k (0 below ks); its 16
// groups of four are read until one ends past t.
__device__ inline int32_t active_at(const HermParams& p, const int4* end, int ks, uint64_t mask, int t) {
    int k = ks & ~3, first = 0;
    int4 e = end[k >> 2];
    while (e.w <= t) {   // t < nact = end[63]
        first = e.w;
        k += 4;
        e = end[k >> 2];
    }
    if (t >= e.z) { k += 3; first = e.z; }
    else if (t >= e.y) { k += 2; first = e.y; }
    else if (t >= e.x) { k += 1; first = e.x; }
    return bucket_of(p, (int)((mask >> k) & 1), k)[t - first];
}

// Each workgroup takes one contiguous chunk of the n_items items (a multiple of
// its lane groups, so a small set is one workgroup): `step(have, i, buf)` advances
// the particle of bucket entry item(k), whose state is in record buf, to the other
// record and returns its new level in lane 0 of its group of LH lanes; the workgroup ranks its items per level in LDS, reserves room in each
// bucket with one device atomic per level (buckets >= ks restart from zero in
// their other buffer, bucket ks - 1 keeps its `keep` members), then stores the
// particles there. Same-address device atomics serialise, so one per workgroup
// and level, not per wave. `step` runs in every lane of a wave that holds an item.
template <int LH, int T, class Item, class Step>
__device__ inline void step_and_bucket(const HermParams& p, unsigned long long* newcnt, int ks, long long keep_cnt,
                                       uint64_t mask_new, int64_t n_items, Item item, Step step) {
    constexpr int TG = T / LH;
    __shared__ int s_h[64];
    __shared__ long long s_b[64];
    const int64_t per = ((n_items + gridDim.x - 1) / gridDim.x + TG - 1) / TG * TG;
    const int64_t c0 = (int64_t)blockIdx.x * per, c1 = c0 + per < n_items ? c0 + per : n_items;
    if (c0 >= c1) return;   // workgroup-uniform
    if (threadIdx.x < 64) s_h[threadIdx.x] = 0;
    __syncthreads();
    const int tg = threadIdx.x / LH;
    const bool head = threadIdx.x % LH == 0;
    // a group's first item stays in registers; later ones go through p.slot
    int lv0 = -1, r0 = 0;
    int32_t i0 = 0;
    for (int64_t k0 = c0; k0 < c1; k0 += TG) {
        const int64_t k = k0 + tg;
        const bool have = k < c1;
        if (__ballot(have) == 0) break;   // this wave holds no more items
        const int32_t i = have ? item(k) : 0;
        const int level = step(have, i & ~kInRec1, i & kInRec1 ? 1 : 0);
        if (have && head) {
            const int r = atomicAdd(&s_h[level], 1);
            if (k0 == c0) {
                lv0 = level;
                r0 = r;
                i0 = i;
            } else {
                p.slot[k] = ((uint32_t)level << kSlotShift) | (uint32_t)r;
            }
        }
    }
    __syncthreads();
    if (threadIdx.x <= kHermK && s_h[threadIdx.x] > 0) {
        const int k = threadIdx.x;
        s_b[k] = (k == ks - 1 ? keep_cnt : 0) + (long long)atomicAdd(newcnt + k, (unsigned long long)s_h[k]);
    }
    __syncthreads();
    auto put = [&](int level, int64_t r, int32_t i) {
        bucket_of(p, (int)((mask_new >> level) & 1), level)[s_b[level] + r] = i ^ kInRec1;
    };
    if (lv0 >= 0) put(lv0, r0, i0);
    if (head)
        for (int64_t k = c0 + TG + tg; k < c1; k += TG) {   // the same later items per group
            const uint32_t v = p.slot[k];
            put((int)(v >> kSlotShift), (int64_t)(v & kSlotMask), item(k));
        }
}

// The same by one workgroup for every item: ranks are places in the buckets at
// once, without a barrier. count[64] (LDS): particles per new level, zero at first.
template <int LH, int T, class Item, class Step>
__device__ inline void step_solo(const HermParams& p, int* count, int ks, long long keep_cnt, uint64_t mask_new,
                                 int n_items, Item item, Step step) {
    constexpr int TG = T / LH;
    for (int k0 = 0; k0 < n_items; k0 += TG) {
        const int k = k0 + (int)threadIdx.x / LH;
        const bool have = k < n_items;
        if (__ballot(have) == 0) break;   // this wave holds no more items
        const int32_t i = have ? item(k) : 0;
        const int level = step(have, i & ~kInRec1, i & kInRec1 ? 1 : 0);
        if (have && threadIdx.x % LH == 0) {
            const long long at = (level == ks - 1 ? keep_cnt : 0) + atomicAdd(&count[level], 1);
            bucket_of(p, (int)((mask_new >> level) & 1), level)[at] = i ^ kInRec1;
        }
    }
}

// block step in ticks: dt_max / 2^k not above `want` (k <= kHermK), dividing tau
// (the largest power of two dividing tau > 0 is its lowest set bit). With
// dt_max >= want the exponents give k or k - 1.
__device__ inline int64_t block_step(double want, double dtmax, int64_t tau) {
    int k = 0;
    if (dtmax > want) {
        k = want > 0.0 ? __builtin_amdgcn_frexp_exp(dtmax) - __builtin_amdgcn_frexp_exp(want) : kHermK;
        if (k < kHermK && __builtin_ldexp(dtmax, -k) > want) ++k;
        k = k < kHermK ? k : kHermK;
    }
    int64_t t = (int64_t)1 << (kHermK - k);
    const int64_t low = tau & -tau;
    if (tau != 0 && low < t) t = low;
    return t;
}

__device__ inline int step_level(int64_t t) { return kHermK - (63 - __clzll((unsigned long long)t)); }

// Second and third time derivatives of one pair term m K(s) d / s^3 of F_I,
// added to f2, f3. d, u, w, z: relative position, velocity, acceleration and
// jerk (j's minus i's); s^2 = |d|^2 + eps^2. The Newtonian part A = m d / s^3
// follows the usual recurrences in
//   al = d.u / s^2,  be = (u.u + d.w) / s^2 + al^2,
//   ga = (3 u.w + d.z) / s^2 + al (3 be - 4 al^2):
//   dA = m u / s^3 - 3 al A,  d2A = m w / s^3 - 6 al dA - 3 be A,
//   d3A = m z / s^3 - 9 al d2A - 9 be dA - 3 ga A;
// along the motion s has the derivatives al s, (be - 2 al^2) s and
// s ((3 u.w + d.z) / s^2 - 3 al (be - 2 al^2)); in the band the weight has
// dK/ds = -g1(x)/D, d2K/ds2 = -g2(x)/D^2, d3K/ds3 = -g3(x)/D^3 with
// g1 = 140 x^3 (1-x)^3, g2 = 420 x^2 (1-x)^2 (1-2x), g3 = 840 x (1-x) (1-5x+5x^2),
// and the product rule gives the second and third derivatives of K A.
__device__ inline void pair_d23(const ClusterParams& cp, double eps2, const double* d, const double* u,
                                const double* w, const double* z, double m, double* f2, double* f3) {
#pragma clang fp contract(off)
    const double s2 = d[0] * d[0] + d[1] * d[1] + d[2] * d[2] + eps2;
    if (!(s2 < cp.rout2)) return;   // K = 0 with all its derivatives
    const double s = sqrt(s2);
    const double i2 = 1.0 / s2;
    const double mi3 = m / (s2 * s);
    const double du = d[0] * u[0] + d[1] * u[1] + d[2] * u[2];
    const double uu = u[0] * u[0] + u[1] * u[1] + u[2] * u[2];
    const double dw = d[0] * w[0] + d[1] * w[1] + d[2] * w[2];
    const double uw = u[0] * w[0] + u[1] * w[1] + u[2] * w[2];
    const double dz = d[0] * z[0] + d[1] * z[1] + d[2] * z[2];
    const double al = du * i2;
    const double be = (uu + dw) * i2 + al * al;
    const double ga = (3.0 * uw + dz) * i2 + al * (3.0 * be - 4.0 * al * al);
    double K = 1.0, K1 = 0.0, K2 = 0.0, K3 = 0.0;   // K and its time derivatives
    if (s >= cp.r_in && cp.inv_delta > 0.0) {
        const double x = (s - cp.r_in) * cp.inv_delta, o = 1.0 - x;
        const double x2 = x * x;
        const double id = cp.inv_delta;
        K = 1.0 - x2 * x2 * (35.0 + x * (-84.0 + x * (70.0 - 20.0 * x)));
        const double ks1 = -140.0 * x2 * x * o * o * o * id;
        const double ks2 = -420.0 * x2 * o * o * (1.0 - 2.0 * x) * id * id;
        const double ks3 = -840.0 * x * o * (1.0 - 5.0 * x + 5.0 * x2) * id * id * id;
        const double sd1 = al * s;
        const double q = be - 2.0 * al * al;
        const double sd2 = q * s;
        const double sd3 = s * ((3.0 * uw + dz) * i2 - 3.0 * al * q);
        K1 = ks1 * sd1;
        K2 = ks2 * sd1 * sd1 + ks1 * sd2;
        K3 = ks3 * sd1 * sd1 * sd1 + 3.0 * ks2 * sd1 * sd2 + ks1 * sd3;
    }
    for (int c = 0; c < 3; ++c) {
        const double A0 = mi3 * d[c];
        const double A1 = mi3 * u[c] - 3.0 * al * A0;
        const double A2 = mi3 * w[c] - 6.0 * al * A1 - 3.0 * be * A0;
        const double A3 = mi3 * z[c] - 9.0 * al * A2 - 9.0 * be * A1 - 3.0 * ga * A0;
        f2[c] += K * A2 + 2.0 * K1 * A1 + K2 * A0;
        f3[c] += K * A3 + 3.0 * K1 * A2 + 3.0 * K2 * A1 + K3 * A0;
    }
}

// First steps: one lane per particle sums the derivatives over its list (in
// list order; lists from the regular-force walk are short), then eq. dt.
__global__ __launch_bounds__(256) void k_herm_start(HermParams p, IrrParams ip) {
    // block 0's counts, every level filled (ks = 0) in buffer 0, the states in record 0
    step_and_bucket<1, 256>(p, lev_new(p, 0), 0, 0, 0ull, p.n,
                                   [](int64_t k) { return (int32_t)k | kInRec1; }, [&](bool have, int32_t i, int) {
#pragma clang fp contract(off)
        if (!have) return 0;   // a lane without an item
        const int64_t i3 = 3 * (int64_t)i;
        double xi[3], vi[3], ai[3], ji[3], f2[3] = {0.0, 0.0, 0.0}, f3[3] = {0.0, 0.0, 0.0};
        for (int c = 0; c < 3; ++c) {
            xi[c] = p.x[i3 + c];
            vi[c] = p.v[i3 + c];
            ai[c] = p.a[i3 + c];
            ji[c] = p.j[i3 + c];
        }
        int64_t b = p.off[i], e = p.off[i + 1];
        if (b < 0 || e < b || e > p.cap) {   // malformed offsets: flagged, list not read
            atomicOr(ip.err, kIrrBadOffsets);
            e = b;
        }
        for (int64_t q = b; q < e; ++q) {
            const int32_t jj = p.idx[q];
            if ((uint64_t)(int64_t)jj >= (uint64_t)p.n) {
                atomicOr(ip.err, kIrrBadIndex);
                continue;
            }
            if (jj == i) continue;
            const int64_t j3 = 3 * (int64_t)jj;
            double d[3], u[3], w[3], z[3];
            for (int c = 0; c < 3; ++c) {
                d[c] = p.x[j3 + c] - xi[c];
                u[c] = p.v[j3 + c] - vi[c];
                w[c] = p.a[j3 + c] - ai[c];
                z[c] = p.j[j3 + c] - ji[c];
            }
            pair_d23(ip.cp0, ip.eps2, d, u, w, z, ip.mass[jj], f2, f3);
        }
        double at[3];
        for (int c = 0; c < 3; ++c) at[c] = ai[c] + (p.fr ? p.fr[i3 + c] : 0.0);
        const double n0 = norm3(at[0], at[1], at[2]);
        const double n1 = norm3(ji[0], ji[1], ji[2]);
        const double n2 = norm3(f2[0], f2[1], f2[2]);
        const double n3 = norm3(f3[0], f3[1], f3[2]);
        const double num = n0 * n2 + n1 * n1, den = n1 * n3 + n2 * n2;
        const double want = den > 0.0 ? sqrt(p.eta * num / den) : p.dtmax;
        const int64_t t = block_step(want, p.dtmax, 0);
        HermState s;
        for (int c = 0; c < 3; ++c) {
            s.x[c] = xi[c];
            s.v[c] = vi[c];
            s.a[c] = ai[c];
            s.j[c] = ji[c];
        }
        s.m = ip.mass[i];
        s.tau = 0;
        s.dt = t;
        store_state(record(p, i, 0), s);
        record(p, i, 1)[6] = make_double2(0.0, __longlong_as_double(-1ll));   // none yet: a time before any
        p.dt0[i] = t;
        return step_level(t);
    });
}

// One active particle i with its state in record buf (a group of LH lanes; have
// false: a group without one, which takes part in the exchange): F_I and its derivative a1, j1 at the predicted
// states (the pair terms of the irregular-force kernel; lane g sums list entries
// g, g + LH, ... in order, then the group's butterfly), the 4th-order corrector
// and the new block step; returns the new level.
template <int LH>
__device__ inline int force_correct(const HermParams& p, const IrrParams& ip, bool have, int32_t i, int buf, int64_t tn) {
#pragma clang fp contract(off)
    const int g = threadIdx.x % LH;
    IrrSums S;   // (the pair sums carry their own contraction setting)
    HermState s = {};
    double xp[3] = {0.0, 0.0, 0.0}, vp[3] = {0.0, 0.0, 0.0}, fr[3] = {0.0, 0.0, 0.0};
    if (have) {
        const int64_t i3 = 3 * (int64_t)i;
        int64_t b = p.off[i], e = p.off[i + 1];
        s = load_state(record(p, i, buf));
        if (p.fr)
            for (int c = 0; c < 3; ++c) fr[c] = p.fr[i3 + c];
        predict(p, s, tn, xp, vp);
        const PartJ me = {xp[0], xp[1], xp[2], s.m, vp[0], vp[1], vp[2]};
        const IrrK K = irr_constants(ip.cp0);
        if (b < 0 || e < b || e > p.cap) {   // malformed offsets: flagged, list not read
            atomicOr(ip.err, kIrrBadOffsets);
            e = b;
        }
        for (int64_t m = b + g; m < e; m += LH) {
            const int64_t j = p.idx[m];
            if ((uint64_t)j >= (uint64_t)p.n) {
                atomicOr(ip.err, kIrrBadIndex);
                continue;
            }
            if (j == i) continue;
            const HermState o = load_state(record(p, j, state_buffer(p, j, tn)));
            double xj[3], vj[3];
            predict(p, o, tn, xj, vj);
            pair_irr<true, false, false>(K, ip.eps2, me, PartJ{xj[0], xj[1], xj[2], o.m, vj[0], vj[1], vj[2]}, true, S);
        }
    }
    if (LH > 1) {
        double* const w[6] = {&S.ax, &S.ay, &S.az, &S.jx, &S.jy, &S.jz};
        for (int k = 0; k < 6; ++k)
            for (int o = LH / 2; o > 0; o >>= 1) *w[k] += __shfl_xor(*w[k], o, 64);
    }
    if (!have || g != 0) return 0;
    const double a1v[3] = {S.ax, S.ay, S.az}, j1v[3] = {S.jx, S.jy, S.jz};
    const double d = (double)s.dt * p.unit, d2 = d * d, d3 = d2 * d, d4 = d3 * d, d5 = d4 * d;
    double a2[3], a3[3], a2e[3], at[3];
    for (int c = 0; c < 3; ++c) {
        const double a1 = a1v[c], j1 = j1v[c];
        const double da = s.a[c] - a1;
        a2[c] = (-6.0 * da - d * (4.0 * s.j[c] + 2.0 * j1)) / d2;
        a3[c] = (12.0 * da + 6.0 * d * (s.j[c] + j1)) / d3;
        s.x[c] = xp[c] + d4 / 24.0 * a2[c] + d5 / 120.0 * a3[c];
        s.v[c] = vp[c] + d3 / 6.0 * a2[c] + d4 / 24.0 * a3[c];
        s.a[c] = a1;
        s.j[c] = j1;
        a2e[c] = a2[c] + d * a3[c];
        at[c] = a1 + fr[c];
    }
    const double n0 = norm3(at[0], at[1], at[2]);
    const double n1 = norm3(j1v[0], j1v[1], j1v[2]);
    const double n2 = norm3(a2e[0], a2e[1], a2e[2]);
    const double n3 = norm3(a3[0], a3[1], a3[2]);
    const double num = n0 * n2 + n1 * n1, den = n1 * n3 + n2 * n2;
    double want = den > 0.0 ? sqrt(p.eta * num / den) : p.dtmax;
    if (want > 2.0 * d) want = 2.0 * d;
    const int64_t t = block_step(want, p.dtmax, tn);
    s.tau = tn;
    s.dt = t;
    store_state(record(p, i, buf ^ 1), s);
    return step_level(t);
}

// One launch (number b in its batch): every workgroup computes the next block
// time and the active buckets from the level counts; then the grid takes that
// block, or workgroup 0 that one and those after it while they are few, and
// workgroup 0 leaves counts, time and buckets for the next launch.
__global__ __launch_bounds__(kHermT) void k_herm_block(HermParams p, IrrParams ip, int b) {
    __shared__ long long s_cnt[64];
    __shared__ int4 s_end[16];
    __shared__ int s_new[64];   // of the last block of a row
    __shared__ long long s_tn;
    __shared__ int s_nact, s_ks;
    const int q = b & 1;
    uint64_t mask = p.lev[kLevMask + q];
    // wave 0, lane k: the count of level k, the levels the last block filled
    // (its corrected particles; the first block's are the start levels, which
    // count for no statistics), and the statistics of this launch
    const int lane = threadIdx.x;
    const bool wave0 = lane < 64;
    long long c = 0, t = 0;
    int last = 0, deepest = -1;
    unsigned long long blocks = 0, steps = 0;
    auto plan = [&](long long old, long long add, int kp) {
        c = lane <= kHermK ? merged_count(old, add, kp, lane) : 0;
        const uint64_t app = __ballot(lane <= kHermK && add > 0);
        if (t > 0 && app) {
            const int dl = 63 - __clzll(app);
            deepest = dl > deepest ? dl : deepest;
        }
        const BlockPlan B = plan_block(c, t, p.tend);
        s_cnt[lane] = c;
        (&s_end[0].x)[lane] = B.end;
        if (lane == 0) {
            s_tn = B.done ? -1 : B.tn;
            s_nact = B.done ? 0 : B.nact;
            s_ks = B.ks;
        }
        return B;
    };
    // for the next launch: the counts before the last block, its time, its k* and
    // the buckets after it
    auto publish = [&](long long tn, int ks, uint64_t mask_new, bool done) {
        if (lane <= kHermK) {
            lev_cnt(p, q ^ 1)[lane] = (unsigned long long)c;
            lev_new(p, b + 2)[lane] = 0ull;
        }
        if (lane != 0) return;
        p.lev[kLevT + (q ^ 1)] = (unsigned long long)tn;
        p.lev[kLevKs + (q ^ 1)] = (unsigned long long)ks;
        p.lev[kLevMask + (q ^ 1)] = mask_new;
        if (deepest >= 0 && (unsigned long long)deepest > p.ctl[kHermKmax])
            p.ctl[kHermKmax] = (unsigned long long)deepest;
        const unsigned long long all = p.ctl[kHermBlocks] + blocks;
        p.ctl[kHermBlocks] = all;
        p.ctl[kHermSteps] += steps;
        if (done) p.ctl[kHermDone] = 1ull;
        // read by the host while later launches run
        if (p.done_host && (done || all > kHermMaxBlocks)) *p.done_host = all > kHermMaxBlocks ? 2ull : 1ull;
    };
    if (wave0) {
        s_new[lane] = 0;
        t = (long long)p.lev[kLevT + q];
        const long long old = lane <= kHermK ? (long long)lev_cnt(p, q)[lane] : 0;
        const long long add = lane <= kHermK ? (long long)lev_new(p, b)[lane] : 0;
        plan(old, add, (int)p.lev[kLevKs + q]);
    }
    __syncthreads();
    long long tn = s_tn;
    int nact = s_nact, ks = s_ks;
    auto item = [&](int64_t k) { return active_at(p, s_end, ks, mask, (int)k); };
    if (nact == 0) {
        if (wave0 && blockIdx.x == 0) publish((long long)p.tend, kHermK + 1, mask, true);
        return;
    }
    if (nact > kHermSolo) {
        const uint64_t mask_new = mask ^ (~0ull << ks);
        if (wave0 && blockIdx.x == 0) {
            blocks = 1;
            steps = (unsigned long long)nact;
            publish(tn, ks, mask_new, false);
        }
        const long long keep = ks > 0 ? s_cnt[ks - 1] : 0;
        unsigned long long* const newcnt = lev_new(p, b + 1);
        // eight lanes share a particle's list while the grid has lanes for all
        if ((long long)nact * kHermLanes <= (long long)gridDim.x * kHermT)
            step_and_bucket<kHermLanes, kHermT>(
                p, newcnt, ks, keep, mask_new, nact, item,
                [&](bool have, int32_t i, int buf) { return force_correct<kHermLanes>(p, ip, have, i, buf, tn); });
        else
            step_and_bucket<1, kHermT>(p, newcnt, ks, keep, mask_new, nact, item,
                                              [&](bool have, int32_t i, int buf) { return force_correct<1>(p, ip, have, i, buf, tn); });
        return;
    }
    if (blockIdx.x != 0) return;
    for (int it = 1;; ++it) {
        const uint64_t mask_new = mask ^ (~0ull << ks);
        step_solo<kHermLanes, kHermT>(
            p, s_new, ks, ks > 0 ? s_cnt[ks - 1] : 0, mask_new, nact, item,
            [&](bool have, int32_t i, int buf) { return force_correct<kHermLanes>(p, ip, have, i, buf, tn); });
        blocks += 1;
        steps += (unsigned long long)nact;
        __syncthreads();   // every record, bucket entry and count of the block is stored
        const long long before = c;
        if (wave0) {
            last = s_new[lane];
            s_new[lane] = 0;
            t = tn;
            plan(before, last, ks);
        }
        __syncthreads();
        if (it < kHermInner && s_nact > 0 && s_nact <= kHermSolo) {
            nact = s_nact;
            tn = s_tn;
            ks = s_ks;
            mask = mask_new;
            continue;
        }
        if (wave0) {   // (the next launch plans that block again)
            c = before;
            if (lane <= kHermK) lev_new(p, b + 1)[lane] = (unsigned long long)last;
            publish(tn, ks, mask_new, false);
        }
        return;
    }
}

// the states of the end of the regular step into the caller's arrays
__global__ __launch_bounds__(256) void k_herm_finish(HermParams p) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= p.n) return;
    const HermState s = load_state(record(p, i, record_time(p, i, 1) > record_time(p, i, 0) ? 1 : 0));
    for (int c = 0; c < 3; ++c) {
        p.x[3 * i + c] = s.x[c];
        p.v[3 * i + c] = s.v[c];
    }
}

// pot_tot = pot_r + pot_i
__global__ void k_add(int64_t n, const double* a, const double* b, double* out) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) out[i] = a[i] + b[i];
}

}  // namespace

void launch_herm_start(const HermParams& p, const IrrParams& ip, hipStream_t s) {
    const int64_t g = (p.n + 255) / 256;
    hipLaunchKernelGGL(k_herm_start, dim3((unsigned)(g < 1024 ? g : 1024)), dim3(256), 0, s, p, ip);
}

void launch_herm_block(const HermParams& p, const IrrParams& ip, int b, hipStream_t s) {
    const int64_t g = (p.n * kHermLanes + kHermT - 1) / kHermT;
    hipLaunchKernelGGL(k_herm_block, dim3((unsigned)(g < kHermGrid ? g : kHermGrid)), dim3(kHermT), 0, s, p, ip, b);
}

void launch_herm_finish(const HermParams& p, hipStream_t s) {
    hipLaunchKernelGGL(k_herm_finish, dim3((unsigned)((p.n + 255) / 256)), dim3(256), 0, s, p);
}

void launch_add(int64_t n, const double* a, const double* b, double* out, hipStream_t s) {
    hipLaunchKernelGGL(k_add, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, n, a, b, out);
}

}  // namespace pbh
