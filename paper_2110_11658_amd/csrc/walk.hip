// walk.hip -- grouped Barnes-Hut walk for the regular force (gfx950).
//
// Regular acceleration of particle i (Arnold, Baumgardt & Wang 2021, Section
// 2.1, eq. fi with F_R = total - F_I and eq. duncan):
//   a_i = sum_j m_j W(s_ij) d_ij / s_ij^3,  d = x_j - x_i,  s^2 = r^2 + eps^2,
// and the regular potential Phi_R (dPhi_R/ds = W/s^2). Far nodes are taken as
// monopole + traceless quadrupole about their centre of mass (Section 2.4:
// Barnes-Hut with opening angle theta).
//
// One wavefront walks one group (a run of <= 64 sorted particles, one per
// lane), or with few groups a team of four does (see TeamMem). Persistent
// workgroups pull groups from global counters.
// Per step the wave pops up to 64 nodes from its stack (one per lane) and
// classifies them in FP64 without FMA, exactly like the definition:
//   near   box-box distance^2 < R^2, or the boxes touch (R = r_out + r_buff,
//          the neighbour-list radius; R = r_out without a buffer)
//   accept not near, theta > 0, distance^2(group box, COM) > rcrit^2
//   open   otherwise: a leaf becomes particle-particle work, an inner node
//          pushes its children.
// Accepted nodes are compacted with ballot + prefix sums into LDS tiles of TC
// entries (64, 96 or 128; FP32 in the mixed path: positions relative to the group
// centre, formed in FP64 first), leaf particles as runs of their tile; a tile is
// evaluated just before it would overflow, every lane reading each entry by LDS
// broadcast. Only then are the particles of its runs loaded, all in one go (a step
// adds few, and loading them there cost it a search and a memory latency: 128k
// particles 813 -> 803 us, 2^20 5.12 -> 5.07 ms, 4096 190 -> 184). Tile partial sums are
// folded into FP32 (hi, lo) pairs with TwoSum and returned in FP64.
#include <type_traits>

#include "pbh_internal.hpp"
#include "wave.hpp"

namespace pbh {

namespace {

// Tile capacity TC (a template parameter, 64, 96 or 128). A far or near tile
// is evaluated just before it would overflow; the multipole tile holds TC + 32
// entries and is evaluated at the start of a traversal step once it holds more
// than TC - 32 (one step adds at most 64), where the least state is live. One
// traversal step adds at most 64 entries of a kind, so TC >= 64.
//
// The first kWalkStackLds traversal stack entries live in LDS (the rest in the
// wave's spill region).
constexpr int kWalkStackLds = 640;
//
// Near entries of the FP64 walk keep their original coordinates for the
// neighbour test; the mixed walk keeps the sorted index instead and reads the
// coordinates from global memory in the rare case the FP64 test is needed
// (under 10 KB of LDS per wave with TC = 64: 16 waves per CU).
template <typename R, int TC>
struct NearExtra {
    double nx[TC], ny[TC], nz[TC];
};
template <int TC>
struct NearExtra<float, TC> {
    int nears[TC];     // sorted index
};

template <typename R, int TC>
struct alignas(16) Tiles : NearExtra<R, TC> {
    static_assert(TC >= 64, "one traversal step adds up to 64 entries");
    static constexpr int kCap = TC;
    R pn[TC + 32][12];   // cx cy cz M | qxx qyy qzz qxy | qxz qyz - -  (room for one more step)
    // Far and near tiles are filled just before they are evaluated; until then their
    // storage holds the runs of sorted particles that make them up: [0] a run's first
    // entry, [1] its first particle minus that entry
    union {
        R far[TC][4];    // x y z m (relative to the group centre)
        int far_run[2][TC];
    };
    union {
        R nearp[TC][4];
        int near_run[2][TC];
    };
    int nearj[TC];       // caller index: skips the self pair, and is the neighbour index
};

struct WalkParams {
    NodePlanes node;
    Mom32Planes q32;
    Mom64Planes q64;
    const double* x;
    const double* y;
    const double* z;
    const double* m;
    const int32_t* perm;
    const int32_t* g_begin;
    const int32_t* g_count;
    const int32_t* g_root;
    const int32_t* g_cluster;
    const double* g_lo;
    const double* g_hi;
    const ClusterParams* cp;
    const unsigned long long* G;   // device-side group count
    int use_theta;
    double eps2;
    double* acc;
    double* pot;
    int32_t* stack;
    int stack_cap;
    unsigned long long* cnt;
    unsigned long long* queues;     // [kQueues] group queue heads, kQueueStride apart
    unsigned long long* walk_cnt;   // [kWalkCntLines] lines of six interaction counters
    unsigned long long* wave_log;   // per workgroup: groups walked, steady-clock ticks
    unsigned long long* wave_cyc;   // per workgroup: core clock cycles over the same span
    int32_t* nbr_cnt;               // neighbour counts per caller index, or null
    int32_t* stage;                 // neighbour staging rows per sorted particle, or null
    int scap;                       // entries per staging row
    int8_t* stage_k;                // per sorted particle: 1 = list staged, 0 = left to the fill pass
    int32_t* fill_list;             // groups left to the fill pass
    int max_copies;                 // most sub-wave copies of a small group (1..64)
    const double* cpos;             // caller's pos [n][3] and mass [n]: compared with the
    const double* cmass;            // build's sorted copy (changed in place: kErrStale), or null
    void* part_sum;                 // partial sums of the shared groups' waves, [slot][word][lane]
    unsigned* part_done;            // waves of a shared group that have stored theirs
};

__device__ inline void two_sum_acc(float& hi, float& lo, float v) {
    const float s = hi + v;
    const float bp = s - hi;
    const float e = (hi - (s - bp)) + (v - bp);
    hi = s;
    lo += e;
}

// Partial sums of one tile evaluation (one lane).
template <typename R>
struct Part {
    R x, y, z, p;
};

template <typename R>
struct Acc;

template <>
struct Acc<float> {
    float hx = 0, hy = 0, hz = 0, hp = 0, lx = 0, ly = 0, lz = 0, lp = 0;
    static constexpr int kWords = 8;
    __device__ void add(float ax, float ay, float az, float ph) {
        two_sum_acc(hx, lx, ax);
        two_sum_acc(hy, ly, ay);
        two_sum_acc(hz, lz, az);
        two_sum_acc(hp, lp, ph);
    }
    __device__ void add(const Part<float>& q) { add(q.x, q.y, q.z, q.p); }
    __device__ void store(float* w) const {
        w[0] = hx; w[1] = lx; w[2] = hy; w[3] = ly; w[4] = hz; w[5] = lz; w[6] = hp; w[7] = lp;
    }
    __device__ void load(const float* w) {
        hx = w[0]; lx = w[1]; hy = w[2]; ly = w[3]; hz = w[4]; lz = w[5]; hp = w[6]; lp = w[7];
    }
    // adds another (hi, lo) set: TwoSum of the high parts, plain sum of the low parts
    __device__ void merge(const float* w) {
        two_sum_acc(hx, lx, w[0]); lx += w[1];
        two_sum_acc(hy, ly, w[2]); ly += w[3];
        two_sum_acc(hz, lz, w[4]); lz += w[5];
        two_sum_acc(hp, lp, w[6]); lp += w[7];
    }
    __device__ double gx() const { return (double)hx + (double)lx; }
    __device__ double gy() const { return (double)hy + (double)ly; }
    __device__ double gz() const { return (double)hz + (double)lz; }
    __device__ double gp() const { return (double)hp + (double)lp; }
};

template <>
struct Acc<double> {
    double x = 0, y = 0, z = 0, p = 0;
    static constexpr int kWords = 4;
    __device__ void add(double ax, double ay, double az, double ph) {
        x += ax; y += ay; z += az; p += ph;
    }
    __device__ void add(const Part<double>& q) { add(q.x, q.y, q.z, q.p); }
    __device__ void store(double* w) const { w[0] = x; w[1] = y; w[2] = z; w[3] = p; }
    __device__ void load(const double* w) { x = w[0]; y = w[1]; z = w[2]; p = w[3]; }
    __device__ void merge(const double* w) { x += w[0]; y += w[1]; z += w[2]; p += w[3]; }
    __device__ double gx() const { return x; }
    __device__ double gy() const { return y; }
    __device__ double gz() const { return z; }
    __device__ double gp() const { return p; }
};

// the value of lane L ^ 32: lane p < 32 receives lane p + 32's
template <typename R>
__device__ inline R shfl_down32(R v) { return __shfl_xor(v, 32, 64); }

__device__ inline float rsq(float v) { return __builtin_amdgcn_rsqf(v); }
__device__ inline double rsq(double v) { return rsqrt(v); }
__device__ inline float lnr(float v) { return __logf(v); }
__device__ inline double lnr(double v) { return log(v); }

// Sub-wave split of the tile entries. A group of g <= 32 particles occupies
// ksub = 64 / g copies of itself in the wave (lane = sub * g + particle); the
// copy `sub` evaluates tile entries sub, sub + ksub, sub + 2 ksub, ... and the
// copies' partial sums are merged once per group. ksub = 1 is the plain
// one-particle-per-lane walk. `body(e)` evaluates entry e for this lane.
template <int U, typename F>
__device__ inline void for_entries(int cnt, int ksub, int sub, F&& body) {
    if (ksub == 1) {
#pragma unroll U
        for (int e = 0; e < cnt; ++e) body(e);
    } else {
        int e2 = 0;
#pragma unroll 2
        for (; e2 + ksub <= cnt; e2 += ksub) body(e2 + sub);
        if (e2 + sub < cnt) body(e2 + sub);
    }
}

// Loop iterations of for_entries, ceil(cnt / ksub), as a multiply and shift:
// with rcp = ceil(2^16 / ksub), floor(v * rcp / 2^16) = floor(v / ksub) for
// v < 2^16 / 64 (the error v * (rcp - 2^16 / ksub) / 2^16 stays below 1 / ksub).
__device__ inline unsigned rounds_rcp(int ksub) { return (65536u + (unsigned)ksub - 1u) / (unsigned)ksub; }
__device__ inline int entry_rounds(int cnt, int ksub, unsigned rcp) {
    return (int)(((unsigned)(cnt + ksub - 1) * rcp) >> 16);
}

// Monopole + traceless quadrupole: phi = -M/s - (R^T Q R)/(2 s^5), a = -grad phi
//   a = -(M/s^3 + (5/2) (R^T Q R)/s^7) R + Q R / s^5,   R = x_i - COM
template <typename R, int TC>
__device__ inline Part<R> eval_pn(const Tiles<R, TC>& T, int cnt, int ksub, int sub, R px, R py, R pz,
                                  R eps2) {
    R ax = 0, ay = 0, az = 0, ph = 0;
    for_entries<2>(cnt, ksub, sub, [&](int e) {
        const R* q = T.pn[e];
        const R Rx = px - q[0], Ry = py - q[1], Rz = pz - q[2];
        const R s2 = Rx * Rx + Ry * Ry + Rz * Rz + eps2;
        const R inv = rsq(s2);
        const R inv2 = inv * inv;
        const R inv3 = inv * inv2;
        const R inv5 = inv3 * inv2;
        const R inv7 = inv5 * inv2;
        const R qx = q[4] * Rx + q[7] * Ry + q[8] * Rz;
        const R qy = q[7] * Rx + q[5] * Ry + q[9] * Rz;
        const R qz = q[8] * Rx + q[9] * Ry + q[6] * Rz;
        const R rqr = Rx * qx + Ry * qy + Rz * qz;
        const R cr = -q[3] * inv3 - R(2.5) * rqr * inv7;
        ax += cr * Rx + qx * inv5;
        ay += cr * Ry + qy * inv5;
        az += cr * Rz + qz * inv5;
        ph += -q[3] * inv - R(0.5) * rqr * inv5;
    });
    return Part<R>{ax, ay, az, ph};
}

// FP32 form written as explicit FMA chains (33 VALU + 1 rsqrt per entry). The
// tile holds Q' = 2.5 Q, so with q' = Q' R and t' = R.q' / s^5 (= 2.5 t):
//   cr = M/s^3 + t'/s^2,  a += 0.4 q'/s^5 - cr R,  phi += -M/s - 0.2 t'.
// The q'/s^5 terms are summed apart and scaled by 0.4 once per tile.
template <int TC>
__device__ inline Part<float> eval_pn_f32(const Tiles<float, TC>& T, int cnt, int ksub, int sub, float px,
                                          float py, float pz, float eps2) {
    float ax = 0.f, ay = 0.f, az = 0.f, ph = 0.f;
    float bx = 0.f, by = 0.f, bz = 0.f;
    for_entries<4>(cnt, ksub, sub, [&](int e) {
        const float4 a = *reinterpret_cast<const float4*>(&T.pn[e][0]);   // cx cy cz M
        const float4 b = *reinterpret_cast<const float4*>(&T.pn[e][4]);   // qxx qyy qzz qxy
        const float2 c = *reinterpret_cast<const float2*>(&T.pn[e][8]);   // qxz qyz
        const float Rx = px - a.x, Ry = py - a.y, Rz = pz - a.z;
        const float s2 = fmaf(Rz, Rz, fmaf(Ry, Ry, fmaf(Rx, Rx, eps2)));
        const float inv = __builtin_amdgcn_rsqf(s2);
        const float inv2 = inv * inv;
        const float qx = fmaf(c.x, Rz, fmaf(b.w, Ry, b.x * Rx));
        const float qy = fmaf(c.y, Rz, fmaf(b.y, Ry, b.w * Rx));
        const float qz = fmaf(b.z, Rz, fmaf(c.y, Ry, c.x * Rx));
        const float rqr = fmaf(Rz, qz, fmaf(Ry, qy, Rx * qx));
        const float inv3 = inv * inv2;
        const float inv5 = inv3 * inv2;
        const float t = rqr * inv5;
        const float cr = fmaf(t, inv2, a.w * inv3);
        bx = fmaf(qx, inv5, bx);
        by = fmaf(qy, inv5, by);
        bz = fmaf(qz, inv5, bz);
        ax = fmaf(-cr, Rx, ax);
        ay = fmaf(-cr, Ry, ay);
        az = fmaf(-cr, Rz, az);
        ph = fmaf(-a.w, inv, fmaf(-0.2f, t, ph));
    });
    return Part<float>{fmaf(0.4f, bx, ax), fmaf(0.4f, by, ay), fmaf(0.4f, bz, az), ph};
}

// Pairs of far leaves: every pair is at r >= R >= r_out, where W = 1.
template <typename R, int TC>
__device__ inline Part<R> eval_far(const Tiles<R, TC>& T, int cnt, int ksub, int sub, R px, R py, R pz,
                                   R eps2) {
    R ax = 0, ay = 0, az = 0, ph = 0;
    for_entries<4>(cnt, ksub, sub, [&](int e) {
        const R* q = T.far[e];
        const R dx = q[0] - px, dy = q[1] - py, dz = q[2] - pz;
        const R s2 = dx * dx + dy * dy + dz * dz + eps2;
        const R inv = rsq(s2);
        const R mi = q[3] * inv;
        const R mi3 = mi * inv * inv;
        ax += mi3 * dx;
        ay += mi3 * dy;
        az += mi3 * dz;
        ph -= mi;
    });
    return Part<R>{ax, ay, az, ph};
}

template <int TC>
__device__ inline Part<float> eval_far_f32(const Tiles<float, TC>& T, int cnt, int ksub, int sub,
                                           float px, float py, float pz, float eps2) {
    float ax = 0.f, ay = 0.f, az = 0.f, ph = 0.f;
    for_entries<4>(cnt, ksub, sub, [&](int e) {
        const float4 q = *reinterpret_cast<const float4*>(&T.far[e][0]);
        const float dx = q.x - px, dy = q.y - py, dz = q.z - pz;
        const float s2 = fmaf(dz, dz, fmaf(dy, dy, fmaf(dx, dx, eps2)));
        const float inv = __builtin_amdgcn_rsqf(s2);
        const float mi = q.w * inv;
        const float mi3 = mi * (inv * inv);
        ax = fmaf(mi3, dx, ax);
        ay = fmaf(mi3, dy, ay);
        az = fmaf(mi3, dz, az);
        ph -= mi;
    });
    return Part<float>{ax, ay, az, ph};
}

template <typename R>
struct NearK {
    R r_in, r_out, inv_delta, c0, d0, l1, inner;
    R e[6];
    bool pole;   // r_in > 0: the -d0/s and log terms are present
    // FP32 neighbour pre-test (mixed path): R^2 (list radius) in FP32 and the half-width
    // of the band around it inside which the FP64 test decides (infinite:
    // always FP64)
    float rlist2f, band;
    const double* x;   // sorted FP64 coordinates (the FP64 neighbour test of the mixed walk)
    const double* y;
    const double* z;
};

// Neighbour test of the CSR lists: r^2 < R^2 (list radius) in FP64 from the original
// coordinates, ((dx*dx + dy*dy) + dz*dz) without FMA.
__device__ inline bool is_neighbour(double xj, double yj, double zj, double xi, double yi, double zi,
                                    double rlist2) {
#pragma clang fp contract(off)
    const double dx = xj - xi, dy = yj - yi, dz = zj - zi;
    const double r2 = dx * dx + dy * dy + dz * dz;
    return r2 < rlist2;
}

// Pairs of near leaves: changeover weight W(s) and the regular potential;
// optionally also counts the neighbours inside the list radius R (FP64 test).
// optionally also stores them in the lane's staging row (`srow`, at most
// `scap` entries, kStageStride apart).
template <typename R, int TC>
__device__ inline Part<R> eval_near(const Tiles<R, TC>& T, int cnt, int ksub, int sub, R px, R py, R pz,
                                    R eps2, int self, const NearK<R>& K, bool count_nbr, bool force, int me,
                                    double rlist2, int& nbr, int32_t* srow, int scap) {
    const double xi = K.x[me], yi = K.y[me], zi = K.z[me];
    R ax = 0, ay = 0, az = 0, ph = 0;
    for_entries<1>(cnt, ksub, sub, [&](int e) {
        const R* q = T.nearp[e];
        const int oj = T.nearj[e];
        const bool is_self = oj == self;
        if (count_nbr) {
            const bool nb = !is_self && is_neighbour(T.nx[e], T.ny[e], T.nz[e], xi, yi, zi, rlist2);
            if (nb && nbr < scap) srow[nbr * kStageStride] = oj;
            nbr += nb ? 1 : 0;
        }
        if (!force) return;
        const R dx = q[0] - px, dy = q[1] - py, dz = q[2] - pz;
        const R s2 = dx * dx + dy * dy + dz * dz + eps2;
        const R inv = rsq(s2);
        const R s = s2 > R(0) ? s2 * inv : R(0);
        const R xx = (s - K.r_in) * K.inv_delta;
        const R x2 = xx * xx;
        const R gpoly = x2 * x2 * (R(35) + xx * (R(-84) + xx * (R(70) - R(20) * xx)));
        const R W = s >= K.r_out ? R(1) : (s < K.r_in ? R(0) : gpoly);
        const R f = (W > R(0) && !is_self) ? q[3] * W * inv * inv * inv : R(0);
        ax += f * dx;
        ay += f * dy;
        az += f * dz;
        const R t = s * K.inv_delta;
        R mid = K.c0 + t * (K.e[0] + t * (K.e[1] + t * (K.e[2] + t * (K.e[3] + t * (K.e[4] + t * K.e[5])))));
        if (K.pole) mid += -K.d0 * inv + K.l1 * lnr(s);
        const R phi = s >= K.r_out ? -inv : (s < K.r_in ? K.inner : mid);
        ph += is_self ? R(0) : q[3] * phi;
    });
    return Part<R>{ax, ay, az, ph};
}

// Whether the near pair e (dr = r^2 - R^2 in FP32) is inside the list radius:
// FP32 decides outside the band (where it provably agrees with the FP64
// definition), the FP64 test inside it.
template <int TC>
__device__ inline bool near_listed(const Tiles<float, TC>& T, int e, float dr, const NearK<float>& K, int me,
                                   double rlist2) {
    const double* __restrict__ gx = K.x;
    const double* __restrict__ gy = K.y;
    const double* __restrict__ gz = K.z;
    const bool band = fabsf(dr) <= K.band;
    bool nb = dr < 0.f;
    if (__ballot(band)) {
        if (band) {
            const int js = T.nears[e];
            nb = is_neighbour(gx[js], gy[js], gz[js], gx[me], gy[me], gz[me], rlist2);
        }
    }
    return nb;
}

// FP32 form without per-lane branches: the neighbour count and the pole
// terms (-d0/s + l1 ln s, present when r_in > 0) are compile-time switches,
// ln s = log2(s) ln 2, and the boundary cases of W and Phi_R are selects.
// Each entry yields a force factor f and a potential term, taken either from
// the far-pair formula (every lane beyond the list radius) or from the
// changeover forms; the sums are updated in one place after either.
// Without FORCE only the neighbours are found.
template <bool CNT, bool FORCE, bool POLE, int TC>
__device__ inline Part<float> eval_near_f32(const Tiles<float, TC>& T, int cnt, int ksub, int sub,
                                            float px, float py, float pz, float eps2, int self,
                                            const NearK<float>& K, int me, double rlist2, int& nbr,
                                            int32_t* srow, int scap) {
    float ax = 0.f, ay = 0.f, az = 0.f, ph = 0.f;
    const float l1 = K.l1 * 0.693147180559945309f;
    const float x0 = -K.r_in * K.inv_delta;   // x = (s - r_in) / delta = s / delta + x0
    // s^2 >= 1e-30 keeps 1/s and 1/s^2 finite: a pair at s = 0 only arises with
    // eps = 0 (where W = 0 and the self pair is masked); for eps^2 >= 2^-76 the
    // added term is below half an ulp of s^2 and changes nothing
    const float e2 = eps2 + 1e-30f;
    for_entries<2>(cnt, ksub, sub, [&](int e) {
        const float4 q = *reinterpret_cast<const float4*>(&T.nearp[e][0]);
        const float dx = q.x - px, dy = q.y - py, dz = q.z - pz;
        const float r2 = fmaf(dz, dz, fmaf(dy, dy, dx * dx));
        const float s2 = r2 + e2;
        const float dr = r2 - K.rlist2f;
        if (!FORCE) {
            if (__ballot(dr <= K.band) == 0) return;
            const int oj = T.nearj[e];
            bool nb = near_listed(T, e, dr, K, me, rlist2);
            nb = nb & (oj != self);
            if (nb & (nbr < scap)) srow[nbr * kStageStride] = oj;
            nbr += nb ? 1 : 0;
            return;
        }
        const float inv = __builtin_amdgcn_rsqf(s2);
        float f, pt;
        if (__ballot(dr <= K.band) == 0) {
            // every lane's pair lies beyond R >= r_out by more than the rounding band:
            // no neighbour, W = 1 and Phi_R = -1/s (the far-pair formula)
            const float mi = q.w * inv;
            f = mi * (inv * inv);
            pt = -mi;
        } else {
            // changeover forms first (every lane evaluates them), then the
            // neighbour test, then the selects
            const float s = s2 * inv;
            const float xx = fmaf(s, K.inv_delta, x0);
            const float x2 = xx * xx;
            const float gp = (x2 * x2) * fmaf(xx, fmaf(xx, fmaf(-20.f, xx, 70.f), -84.f), 35.f);
            const float t = s * K.inv_delta;
            float mid = fmaf(t, fmaf(t, fmaf(t, fmaf(t, fmaf(t, K.e[5], K.e[4]), K.e[3]), K.e[2]), K.e[1]),
                             K.e[0]);
            mid = fmaf(t, mid, K.c0);
            if (POLE) mid = fmaf(-K.d0, inv, fmaf(l1, __builtin_amdgcn_logf(s), mid));
            // (the empty asm statements keep the polynomial and the selects in
            // place: sunk under a divergent branch on s < r_out, they cost more in
            // exec-mask handling than they save)
            asm volatile("" : "+v"(mid));
            const bool outer = s >= K.r_out, inner = s < K.r_in;
            float phi = inner ? K.inner : mid;
            asm volatile("" : "+v"(phi));
            phi = outer ? -inv : phi;
            const int oj = T.nearj[e];
            const bool other = oj != self;
            if (CNT) {
                bool nb = near_listed(T, e, dr, K, me, rlist2);
                nb = nb & other;
                if (nb & (nbr < scap)) srow[nbr * kStageStride] = oj;
                nbr += nb ? 1 : 0;
            }
            const float mq = other ? q.w : 0.f;
            const float W = outer ? 1.f : (inner ? 0.f : gp);
            // W first: W = 0 gives f = 0 without forming m / s^3
            f = ((W * mq) * inv) * (inv * inv);
            pt = mq * phi;
        }
        ax = fmaf(f, dx, ax);
        ay = fmaf(f, dy, ay);
        az = fmaf(f, dz, az);
        ph += pt;
    });
    return Part<float>{ax, ay, az, ph};
}

// Only the neighbours of a near tile, in entry order, for the list wave of a team:
// a lane's four next entries are read and tested together (one at a time, the LDS
// reads and branches set its pace: walk of 4096 particles 146 us, 138 so; with four
// groups on a SIMD that is covered and the larger code costs 2 to 5 %).
template <int TC>
__device__ inline void find_near_f32(const Tiles<float, TC>& T, int cnt, int ksub, int sub, float px, float py,
                                     float pz, int self, const NearK<float>& K, int me, double rlist2, int& nbr,
                                     int32_t* srow, int scap) {
    for (int e0 = 0; e0 < cnt; e0 += 4 * ksub) {
        float dr[4];
        int oj[4];
        bool band = false, any = false;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int e = e0 + u * ksub + sub, ec = e < cnt ? e : cnt - 1;
            const float4 q = *reinterpret_cast<const float4*>(&T.nearp[ec][0]);
            const float dx = q.x - px, dy = q.y - py, dz = q.z - pz;
            oj[u] = T.nearj[ec];
            dr[u] = e < cnt ? fmaf(dz, dz, fmaf(dy, dy, dx * dx)) - K.rlist2f : INFINITY;
            band = band || (e < cnt && fabsf(dr[u]) <= K.band);
            any = any || dr[u] < 0.f;
        }
        if (__ballot(band || any) == 0) continue;
        const bool exact = __ballot(band) != 0;   // (wave-uniform)
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int e = e0 + u * ksub + sub;
            bool nb = dr[u] < 0.f;
            if (exact && e < cnt) nb = near_listed(T, e, dr[u], K, me, rlist2);
            nb = nb && oj[u] != self;
            if (nb && nbr < scap) srow[nbr * kStageStride] = oj[u];
            nbr += nb ? 1 : 0;
        }
    }
}

// The mixed walk's forms (explicit FMA chains above), chosen per precision.
template <int TC>
__device__ inline Part<float> eval_pn(const Tiles<float, TC>& T, int cnt, int ksub, int sub, float px,
                                      float py, float pz, float eps2) {
    return eval_pn_f32<TC>(T, cnt, ksub, sub, px, py, pz, eps2);
}

template <int TC>
__device__ inline Part<float> eval_far(const Tiles<float, TC>& T, int cnt, int ksub, int sub, float px,
                                       float py, float pz, float eps2) {
    return eval_far_f32<TC>(T, cnt, ksub, sub, px, py, pz, eps2);
}

template <int TC>
__device__ inline Part<float> eval_near(const Tiles<float, TC>& T, int cnt, int ksub, int sub,
                                        float px, float py, float pz, float eps2, int self,
                                        const NearK<float>& K, bool count_nbr, bool force, int me, double rlist2,
                                        int& nbr, int32_t* srow, int scap) {
    if (!force)   // (only with count_nbr)
        return eval_near_f32<true, false, false, TC>(T, cnt, ksub, sub, px, py, pz, eps2, self, K, me, rlist2,
                                                     nbr, srow, scap);
    if (count_nbr) {
        if (K.pole)
            return eval_near_f32<true, true, true, TC>(T, cnt, ksub, sub, px, py, pz, eps2, self, K, me, rlist2,
                                                       nbr, srow, scap);
        return eval_near_f32<true, true, false, TC>(T, cnt, ksub, sub, px, py, pz, eps2, self, K, me, rlist2,
                                                    nbr, srow, scap);
    }
    if (K.pole)
        return eval_near_f32<false, true, true, TC>(T, cnt, ksub, sub, px, py, pz, eps2, self, K, me, rlist2,
                                                    nbr, srow, scap);
    return eval_near_f32<false, true, false, TC>(T, cnt, ksub, sub, px, py, pz, eps2, self, K, me, rlist2, nbr,
                                                 srow, scap);
}

// How many groups at the end of each queue are shared by two waves. With few
// groups the chip is idle but for the longest one, so all are; with many, sharing
// the last ones makes the end of the walk finer-grained (a group is up to a
// millisecond of one wave) at the price of traversing for them twice, which costs
// the FP64 walk less. q: groups per queue, w: waves per queue (512 for the mixed
// walk). Walk times in us, one wave a group, sharing none / the rule's / all:
//   215 groups 245 / 205 / 205, 1523: 461 / 374 / 375, 3177: 552 / 521 / 576,
//   6141: 892 / 805 / 899, 26611: 5128 / 5098 / -, FP64 4782: 2012 / 1786 / 1835
// and with 103236 groups sharing only costs (14090 / 14150).
// A team (see TeamMem) shares all groups or none: 16384 particles 225 / 231, 32768
// 339 (three eighths) / 322. With tiles of 128 entries ten waves share a CU, not
// sixteen, and the second traversal costs them more: none are shared beyond 1.5 groups
// a wave (1.2 groups a wave, none / three eighths: 571 / 529; 1.5: 1309 / 1368; 1.9:
// 754 / 797; 2.4: 901 / 986; 3.6: 1202 / 1327).
template <bool MIXED, int TC, int TEAM>
__device__ inline int walk_shared(int64_t G) {
    const int64_t q = (G + kQueues - 1) / kQueues, w = gridDim.x / kQueues;
    if (q > 8 * w || (MIXED && TC == 128 && 2 * q > 3 * w)) return 0;
    const int64_t t = 8 * q <= 5 * w ? q : (TEAM > 1 ? 0 : (MIXED ? q * 3 / 8 : q * 5 / 8));
    return (int)(t < kWalkShared / kQueues ? t : kWalkShared / kQueues);
}

// The next work item of a persistent wave. A queue (one contiguous range of
// groups, one per XCD) hands out its groups one by one; its last `tail` groups
// are handed out twice, to the two waves that share them.
struct WalkItem {
    int64_t g;        // group, < 0: no work left
    int part, parts;  // this wave's part of it
    int slot;         // its place among the shared groups' partial sums (parts > 1)
};

// A wave's first item is its own by its place in the grid, with no queue access
// (4096 waves starting on one line of queue heads waited 50 us for it, and every
// other access to that memory channel with them); the heads count from there
// on, each on a line of its own.
__device__ inline WalkItem walk_next(unsigned long long* q, int64_t G, int tail, int& home, bool first,
                                     int lane) {
    WalkItem it;
    it.part = 0;
    it.parts = 1;
    it.slot = 0;
    for (int k = 0; k < kQueues; ++k) {
        const int qi = (home + k) % kQueues;
        const int64_t lo = G * qi / kQueues, hi = G * (qi + 1) / kQueues;
        const int64_t shared = hi - lo < tail ? hi - lo : tail, single = hi - lo - shared;
        const int64_t given = ((int64_t)gridDim.x - qi + kQueues - 1) / kQueues;   // first items of its waves
        const int64_t items = single + 2 * shared;
        int64_t t;
        if (first && k == 0) {
            t = blockIdx.x / kQueues;
        } else {
            if (items <= given) continue;   // nothing queued beyond the first items
            unsigned long long* head = q + qi * kQueueStride;
            if (k > 0 && (int64_t)__builtin_amdgcn_readfirstlane((int)(*head + given < (unsigned long long)items)) == 0)
                continue;   // range already drained: skip the atomic
            t = given + (int64_t)uni((int)atomicAdd(head, lane == 0 ? 1ull : 0ull));
        }
        if (t < items) {
            home = qi;
            if (t < single) {
                it.g = lo + t;
            } else {
                const int u = (int)(t - single), j = u >> 1;
                it.g = lo + single + j;
                it.part = u & 1;
                it.parts = 2;
                it.slot = (qi * tail + j) * 2;
            }
            return it;
        }
    }
    it.g = -1;
    return it;
}

// The kernel's arguments, read again where they are used: the empty asm keeps
// the compiler from loading all of them at the start, which spilled 150 scalar
// registers into vector ones.
typedef const __attribute__((address_space(4))) WalkParams* WalkArgs;
__device__ inline WalkArgs walk_args() {
    WalkArgs a = (WalkArgs)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(a));
    return a;
}

// A lane's part in the walk of a group: which particles it evaluates for, and how
// the tiles' entries are shared with its copies. By default a group of g particles
// takes one pass over every tile with ksub = min(64 / g, cap) copies, lane = copy *
// g + particle (see for_entries; lanes beyond ksub * g repeat copy 0 and are
// ignored at the merge), and the copies are merged once per group. A group of
// 33..53 particles takes two passes over every multipole tile instead (split):
// pass A holds particles 0..31 in two copies (particle lane & 31, copy lane >> 5),
// pass B the other rB = g - 32 in kB = min(64 / rB, cap, 8) >= 3 copies counted
// from lane 32, so that lane 32 + q holds particle 32 + q in copy 0. Their copies
// are merged after every tile into lane p < g, which owns particle p and takes the
// group's far and near tiles in one pass.
template <typename R>
struct Role {
    int gb, gcnt, cl;
    double ctr[3];          // group centre
    double rlist2;          // neighbour-list radius R = r_out + r_buff, squared
    bool near_exact;        // every neighbour test in FP64 (see the band in tile_near)
    bool active, split;
    int rB, kB, ksubA, subA, copyA, subB;
    int ksubN, subN, me;    // far and near pairs, neighbour list and outputs: this lane's particle
    int wrow, scap;
    bool real, hiB, ownerB;
    R pAx, pAy, pAz, pBx, pBy, pBz;

    __device__ __forceinline__ void set(WalkArgs a, int64_t g, int lane, const double* glo, const double* ghi) {
        gb = uni(a->g_begin[g]);
        gcnt = uni(a->g_count[g]);
        cl = uni(a->g_cluster[g]);
        // a group this large against the list radius R takes every neighbour test in FP64
        double h = 0.0;
        for (int k = 0; k < 3; ++k) {
            ctr[k] = (glo[k] + ghi[k]) * 0.5;
            h = fmax(h, (ghi[k] - glo[k]) * 0.5);
        }
        near_exact = __builtin_amdgcn_readfirstlane((int)(h > 64.0 * a->cp[cl].rlist)) != 0;
        rlist2 = a->cp[cl].rlist2;
        active = lane < gcnt;
        rB = gcnt - 32;
        kB = 0;
        if (rB >= 1 && rB <= 21) {
            const int kfit = 64 / rB;
            kB = kfit < a->max_copies ? kfit : a->max_copies;
            kB = kB < 8 ? kB : 8;
        }
        split = kB >= 3;
        int plA, plB = 0;
        subB = 0;
        if (split) {
            ksubA = 2;
            copyA = lane >> 5;
            subA = copyA;
            plA = lane & 31;
            const int q = (lane - 32) & 63;
            const int cB = q / rB;
            plB = 32 + (q - cB * rB);
            subB = cB < kB ? cB : 0;
        } else {
            const int kfit = 64 / gcnt;
            ksubA = kfit < a->max_copies ? kfit : a->max_copies;
            copyA = lane / gcnt;
            plA = lane - copyA * gcnt;
            subA = copyA < ksubA ? copyA : 0;
        }
        // the particle whose far and near pairs, neighbour list and outputs
        // this lane handles (a stand-in for the idle lanes of a split group)
        const int own = split ? (active ? lane : 0) : plA;
        ksubN = split ? 1 : ksubA;
        subN = split ? 0 : subA;
        me = gb + own;
        // Neighbour staging. A particle's row holds a->scap entries; a lane
        // that holds it whole (ksubN = 1) uses it whole, copies of a small group
        // each get a sub-row of wrow = a->scap / ksubN entries (joined into one
        // list after the walk). Lanes that hold no particle of their own, or
        // repeat copy 0, store nothing (scap = 0).
        real = split ? active : copyA < ksubA;
        wrow = a->scap / ksubN;
        scap = (a->stage == nullptr || !real) ? 0 : (ksubN == 1 ? a->scap : wrow);
        // positions relative to the group centre: pass A (also the far and
        // near tiles, except on lanes >= 32 of a split group) and pass B
        pAx = (R)(a->x[gb + plA] - ctr[0]);
        pAy = (R)(a->y[gb + plA] - ctr[1]);
        pAz = (R)(a->z[gb + plA] - ctr[2]);
        const int pbi = split ? gb + plB : me;
        pBx = (R)(a->x[pbi] - ctr[0]);
        pBy = (R)(a->y[pbi] - ctr[1]);
        pBz = (R)(a->z[pbi] - ctr[2]);
        hiB = split && lane >= 32;   // lanes whose own particle is pass B's copy 0
        ownerB = hiB && active;
    }
};

// The LDS accesses of one wave complete in order; this keeps the compiler to it.
__device__ inline void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// One evaluation of a tile of each kind by one wave (all lanes run it).
template <typename R, int TC>
__device__ __forceinline__ Part<R> tile_pn(Tiles<R, TC>& T, const Role<R>& r, int lane, int cnt, R eps2) {
    Part<R> pa = eval_pn(T, cnt, r.ksubA, r.subA, r.pAx, r.pAy, r.pAz, eps2);
    if (r.split) {
        const Part<R> pb = eval_pn(T, cnt, r.kB, r.subB, r.pBx, r.pBy, r.pBz, eps2);
        // pass A: copy 1 (lane p + 32) into lane p
        pa.x += shfl_down32(pa.x);
        pa.y += shfl_down32(pa.y);
        pa.z += shfl_down32(pa.z);
        pa.p += shfl_down32(pa.p);
        // pass B: copies in copy order into lane 32 + q, through the
        // tile's storage (every lane has read the tile)
        wave_sync();
        Part<R>* red = reinterpret_cast<Part<R>*>(&T.pn[0][0]);
        red[lane] = pb;
        wave_sync();
        Part<R> sb{R(0), R(0), R(0), R(0)};
        if (r.ownerB) {
            for (int c = 0; c < r.kB; ++c) {
                const Part<R> v = red[(lane + c * r.rB) & 63];
                sb.x += v.x; sb.y += v.y; sb.z += v.z; sb.p += v.p;
            }
        }
        wave_sync();
        if (r.hiB) pa = sb;   // idle lanes add zero
    }
    return pa;
}

// Fills a far or near tile of cnt entries from its runs of particles.
template <bool NEAR, typename R, int TC>
__device__ __forceinline__ void fill_tile(Tiles<R, TC>& T, const WalkParams& p, const double (&ctr)[3], int lane,
                                          int cnt, int runs) {
    constexpr int H = (TC + 63) / 64;
    int (&run)[2][TC] = NEAR ? T.near_run : T.far_run;
    int j[H];
    wave_sync();
#pragma unroll
    for (int h = 0; h < H; ++h) {
        const int e = h * 64 + lane;
        int f = 0;   // the last run that begins at or before entry e
#pragma unroll
        for (int st = H * 32; st > 0; st >>= 1)
            if (f + st < runs && run[0][f + st] <= e) f += st;
        j[h] = run[1][f] + e;
    }
    wave_sync();
#pragma unroll
    for (int h = 0; h < H; ++h) {
        const int e = h * 64 + lane;
        if (e >= cnt) continue;
        const int64_t k = j[h];
        R* q = NEAR ? T.nearp[e] : T.far[e];
        q[0] = (R)(p.x[k] - ctr[0]);
        q[1] = (R)(p.y[k] - ctr[1]);
        q[2] = (R)(p.z[k] - ctr[2]);
        q[3] = (R)p.m[k];
        if (NEAR) {
            T.nearj[e] = p.perm[k];
            if constexpr (std::is_same<R, float>::value) {
                T.nears[e] = (int)k;
            } else {
                T.nx[e] = p.x[k];
                T.ny[e] = p.y[k];
                T.nz[e] = p.z[k];
            }
        }
    }
    wave_sync();
}

template <typename R, int TC>
__device__ __forceinline__ Part<R> tile_far(const Tiles<R, TC>& T, const Role<R>& r, int cnt, R eps2) {
    return eval_far(T, cnt, r.ksubN, r.subN, r.hiB ? r.pBx : r.pAx, r.hiB ? r.pBy : r.pAy,
                    r.hiB ? r.pBz : r.pAz, eps2);
}

template <bool LIST_WAVE, typename R, int TC>
__device__ __forceinline__ Part<R> tile_near(const Tiles<R, TC>& T, const Role<R>& r, const WalkParams& p, int cnt,
                                             R eps2, bool count_nbr, bool force, int& nbr) {
    constexpr bool MIXED = std::is_same<R, float>::value;
    // The changeover constants are read for each near tile (about ten a
    // group): kept in registers they would crowd the multipole loop. The
    // empty asm keeps the loads here.
    const ClusterParams* cpp = p.cp + r.cl;
    asm volatile("" : "+s"(cpp));
    const ClusterParams& cp = *cpp;
    NearK<R> K;
    if (MIXED) {
        K.r_in = cp.f_r_in; K.r_out = cp.f_r_out; K.inv_delta = cp.f_inv_delta;
        K.c0 = cp.f_c0; K.d0 = cp.f_d0; K.l1 = cp.f_l1; K.inner = cp.f_inner;
        for (int k = 0; k < 6; ++k) K.e[k] = cp.f_e[k];
    } else {
        K.r_in = cp.r_in; K.r_out = cp.r_out; K.inv_delta = cp.inv_delta;
        K.c0 = cp.c0; K.d0 = cp.d0; K.l1 = cp.l1; K.inner = cp.inner;
        for (int k = 0; k < 6; ++k) K.e[k] = cp.e[k];
    }
    K.pole = cp.d0 != 0.0;
    {
        // Band of the FP32 neighbour pre-test against the list radius R.
        // Relative coordinates are FP64 differences rounded once to FP32, so
        // with |p| <= h (group box half side) and a pair at r <= 2 R each
        // component of d errs by at most 2^-24 (2h + 2.01 r); with h <= 64 R
        // the error of r^2 (squares, FMA rounding, R^2 in FP32) stays below
        // 928 * 2^-24 R^2, and for r > 2 R far below r^2 - R^2. The band is
        // 2048 * 2^-24 R^2; larger groups always take the FP64 test.
        K.rlist2f = (float)r.rlist2;
        K.x = p.x; K.y = p.y; K.z = p.z;
        K.band = r.near_exact ? INFINITY : (float)(2048.0 * 0x1p-24 * r.rlist2);
    }
    int32_t* srow = p.stage != nullptr
                        ? p.stage + stage_index(r.me, (r.ksubN == 1 ? 0 : r.subN * r.wrow), p.scap)
                        : nullptr;
    if constexpr (LIST_WAVE && MIXED) {
        find_near_f32(T, cnt, r.ksubN, r.subN, r.hiB ? r.pBx : r.pAx, r.hiB ? r.pBy : r.pAy, r.hiB ? r.pBz : r.pAz,
                      p.perm[r.me], K, r.me, r.rlist2, nbr, srow, r.scap);
        return Part<R>{0, 0, 0, 0};
    }
    return eval_near(T, cnt, r.ksubN, r.subN, r.hiB ? r.pBx : r.pAx, r.hiB ? r.pBy : r.pAy,
                     r.hiB ? r.pBz : r.pAz, eps2, p.perm[r.me], K, count_nbr, force, r.me, r.rlist2, nbr, srow,
                     r.scap);
}

// Team walk: with few groups a workgroup of four waves walks one group. The first
// traverses and makes tiles; full tiles go as jobs to the others, who take them as
// they come free. Neighbour lists are jobs of their own for the last wave, which
// keeps the counts. Jobs are numbered in the order in which one wave alone would
// evaluate them; a job's partial sums come back through slot (number mod
// kTeamRing) and the first wave folds them into the accumulators in that order, so
// the results are those of one wave. A tile of each kind has kTeamBufs buffers; the
// first wave waits for a slot or buffer it needs, the others for jobs. Every wait is
// for a wave of the same workgroup that runs on, and the end flag ends the others.
constexpr int kTeamWaves = 4;
constexpr int kTeamBufs = 3;
constexpr int kTeamRing = 8;
enum { kJobPn = 0, kJobFar = 1, kJobNear = 2 };

template <typename R, int TEAM>
struct TeamMem {
    Part<R> res[kTeamRing][64];
    int done[kTeamRing];       // number + 1 of the job whose sums the slot holds
    int head, take;            // jobs given, jobs taken
    int4 job[kTeamRing];       // kind, buffer, entries | runs << 16, list job that fills the tile (0: none)
    int last[3][kTeamBufs];    // last job on each buffer of each kind
    int list_head, list_filled, list_done;   // list jobs given, their tiles filled, ended
    int2 list_job[kTeamBufs + 1];            // buffer, entries | runs << 16
    int list_last[kTeamBufs];                // list jobs up to the last one on each near buffer
    int nbr[64];               // neighbours found by the lanes of the last wave
    int group, turn, end;      // group of the jobs, its turn; no more jobs
};
template <typename R>
struct TeamMem<R, 1> {};

__device__ inline int lds_load(int* p) {
    return uni(__hip_atomic_load(p, __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_WORKGROUP));
}
__device__ inline void lds_store(int* p, int v) {   // (all lanes the same value)
    __hip_atomic_store(p, v, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_WORKGROUP);
}
__device__ inline void lds_wait(int* p, int v) {   // until *p >= v
    while (lds_load(p) < v) __builtin_amdgcn_s_sleep(1);
}

__device__ inline void group_box(WalkArgs a, int64_t g, double* lo, double* hi) {
    for (int k = 0; k < 3; ++k) {
        lo[k] = a->g_lo[3 * g + k];
        hi[k] = a->g_hi[3 * g + k];
    }
}

// A wave that evaluates; `lists`: also the neighbour lists.
template <typename R, int TC, int TEAM>
__device__ __forceinline__ void team_evaluate(Tiles<R, TC>* T, TeamMem<R, TEAM>& tm, const WalkParams& p, bool lists,
                                              int lane, R eps2) {
    int turn = 0, list = 0, nbr = 0;
    Role<R> r;
    auto follow = [&]() {   // the group that jobs are given for
        const int now = uni(tm.turn);
        if (now == turn) return;
        turn = now;
        const WalkArgs a = walk_args();
        const int64_t g = uni(tm.group);
        double glo[3], ghi[3];
        group_box(a, g, glo, ghi);
        r.set(a, g, lane, glo, ghi);
        nbr = 0;
    };
    for (;;) {
        // (the jobs seen here come after the list jobs seen next, which fill their tiles)
        const int head = lds_load(&tm.head);
        if (lists && list < lds_load(&tm.list_head)) {
            follow();
            const int2 job = tm.list_job[list % (kTeamBufs + 1)];
            Tiles<R, TC>& t = T[uni(job.x)];
            const int cnt = uni(job.y) & 0xffff;
            fill_tile<true>(t, p, r.ctr, lane, cnt, uni(job.y) >> 16);
            lds_store(&tm.list_filled, ++list);
            tile_near<true>(t, r, p, cnt, eps2, true, false, nbr);
            tm.nbr[lane] = nbr;
            lds_store(&tm.list_done, list);
            continue;
        }
        const int num = lds_load(&tm.take);
        if (num < head) {
            if (uni(atomicCAS(&tm.take, lane == 0 ? num : -1, num + 1)) != num) continue;   // (another wave has it)
            follow();
            const int4 job = tm.job[num % kTeamRing];
            const int kind = uni(job.x), cnt = uni(job.z) & 0xffff, runs = uni(job.z) >> 16, filler = uni(job.w);
            Tiles<R, TC>& t = T[uni(job.y)];
            Part<R> v;
            if (kind == kJobPn) {
                v = tile_pn(t, r, lane, cnt, eps2);
            } else if (kind == kJobFar) {
                fill_tile<false>(t, p, r.ctr, lane, cnt, runs);
                v = tile_far(t, r, cnt, eps2);
            } else {
                if (filler) lds_wait(&tm.list_filled, filler);
                else fill_tile<true>(t, p, r.ctr, lane, cnt, runs);
                int none = 0;
                v = tile_near<false>(t, r, p, cnt, eps2, false, true, none);
            }
            tm.res[num % kTeamRing][lane] = v;
            lds_store(&tm.done[num % kTeamRing], num + 1);
            continue;
        }
        if (lds_load(&tm.end)) break;
        __builtin_amdgcn_s_sleep(1);
    }
}

// Four waves per SIMD (16 per compute unit, which the 64-entry mixed walk's
// LDS allows): the register budget is held to 128, which this kernel fits
// but for a few registers of its set-up; left free, the compiler takes more and halves nothing but
// occupancy. Larger tiles and the FP64 walk are held lower by their LDS; the mixed
// 96-entry tiles leave room for 13 waves, which the compiler takes for four a SIMD as
// well: held to three they keep 148 registers and spill none (131072 particles, theta
// 0.3, 2053 -> 1743 us; the 128-entry tiles are better left alone, 2059 / 2188).
constexpr int walk_waves(bool mixed, int tc) { return mixed && tc == 96 ? 3 : 4; }

template <bool MIXED, int TC, int TEAM>
__global__ __launch_bounds__(64 * TEAM) __attribute__((amdgpu_waves_per_eu(walk_waves(MIXED, TC), walk_waves(MIXED, TC)))) void k_walk(WalkParams p) {
    using R = typename std::conditional<MIXED, float, double>::type;
    constexpr int TCAP = TC;
    __shared__ Tiles<R, TC> s_tiles[TEAM == 1 ? 1 : kTeamBufs];
    __shared__ int s_stack[kWalkStackLds + 1];   // (and an entry for what is not pushed)
    __shared__ TeamMem<R, TEAM> tm;
    const int lane = threadIdx.x & 63;
    const R eps2 = (R)p.eps2;
    if constexpr (TEAM > 1) {
        if (threadIdx.x < kTeamRing) tm.done[threadIdx.x] = 0;
        if (threadIdx.x < 3 * kTeamBufs) (&tm.last[0][0])[threadIdx.x] = -1;
        if (threadIdx.x < kTeamBufs) tm.list_last[threadIdx.x] = 0;
        if (threadIdx.x == 0) tm.head = tm.take = tm.list_head = tm.list_filled = tm.list_done = tm.turn = tm.end = 0;
        __syncthreads();
        // the traversing waves of a CU's teams are spread over its SIMDs
        const int w = uni((int)(threadIdx.x / 64 + blockIdx.x / 256) & (kTeamWaves - 1));
        if (w > 0) {
            team_evaluate<R, TC, TEAM>(s_tiles, tm, p, w == kTeamWaves - 1, lane, eps2);
            return;
        }
    }
    Tiles<R, TC>& T = s_tiles[0];
    const Stack stack{s_stack, p.stack + (int64_t)blockIdx.x * (p.stack_cap - kWalkStackLds), p.stack_cap,
                      kWalkStackLds};
    int home = blockIdx.x % kQueues;
    const int64_t G = (int64_t)*p.G;
    const unsigned long long t_start = wall_clock64();
    const unsigned long long c_start = clock64();
    const int tail = walk_shared<MIXED, TC, TEAM>(G);
    int n_walked = 0;
    // interaction counts of this wave, added to the counters once at its end
    unsigned long long sum_pn = 0, sum_far = 0, sum_near = 0, slot_pn = 0, slot_far = 0, slot_near = 0;
    bool first = true;
    // the team's jobs: next number, first one not yet folded in, those for A1 (a bit
    // per slot), list jobs, the group's turn, and the buffers being filled
    int j_next = 0, j_tail = 0, j_list = 0, j_turn = 0;
    unsigned j_a1 = 0;
    int b_pn = 0, b_far = 0, b_near = 0;
    (void)j_next, (void)j_tail, (void)j_list, (void)j_turn, (void)j_a1;

    for (;;) {
        const WalkItem item = walk_next(p.queues, G, tail, home, first, lane);
        first = false;
        if (item.g < 0) break;
        const int64_t g = item.g;
        // A group's sums are kept in two: A0 takes three of five multipole tiles
        // and the far tiles, A1 the other multipole tiles and the near ones, and
        // the two are added at the end. In a shared group each wave computes one
        // of them: both traverse the tree (the order of the tile entries is the
        // traversal's), each fills and evaluates only the tiles of its own sum, and
        // part 0 finds the neighbours. So the sums do not depend on which groups
        // are shared.
        const int part = uni(item.part), parts = uni(item.parts);
        const bool lead = part == 0;
        n_walked += lead ? 1 : 0;

        const WalkArgs a = walk_args();
        const int root = uni(a->g_root[g]);
        double glo[3], ghi[3];
        group_box(a, g, glo, ghi);
        Role<R> r;
        r.set(a, g, lane, glo, ghi);
        const double (&ctr)[3] = r.ctr;
        const double rlist2 = r.rlist2;
        const bool active = r.active, split = r.split, real = r.real;
        const int gcnt = r.gcnt, ksubA = r.ksubA, ksubN = r.ksubN, kB = r.kB, me = r.me, wrow = r.wrow,
                  scap = r.scap;
        const int orig_me = a->perm[me];
        if (a->cpos && lead) {
            // the caller's arrays must still hold what the build sorted
            const int64_t o3 = 3 * (int64_t)orig_me;
            const bool stale = active && (a->cpos[o3] != a->x[me] || a->cpos[o3 + 1] != a->y[me] ||
                                          a->cpos[o3 + 2] != a->z[me] || a->cmass[orig_me] != a->m[me]);
            if (__ballot(stale)) atomicOr(&a->cnt[kErr], lane == 0 ? kErrStale : 0ull);
        }
        const unsigned rcpA = rounds_rcp(ksubA), rcpB = split ? rounds_rcp(kB) : 0u,
                       rcpN = rounds_rcp(ksubN);
        const bool count_nbr = a->nbr_cnt != nullptr && lead;
        // the tiles this wave fills and evaluates
        int pn_tile = 0, pn_own = 0;                     // multipole tile being filled and its accumulator
        const bool far_mine = lead, near_force = parts == 1 || !lead, near_mine = near_force || count_nbr;
        int npn = 0, nfar = 0, nnear = 0, rfar = 0, rnear = 0;   // tile entries, runs of the far and near tile
        unsigned c_pn = 0, c_far = 0, c_near = 0;   // per group: far below 2^32
        // loop iterations of the evaluations (each occupies all 64 lanes)
        unsigned it_pn = 0, it_far = 0, it_near = 0;
        int nbr = 0;
        Acc<R> A0, A1;
        // one flush of each tile kind; every lane runs it (it_* counts the
        // loop iterations, each of which occupies the 64 lanes)
        auto fold = [&]() {   // the next job's sums
            if constexpr (TEAM > 1) {
                const int slot = j_tail % kTeamRing;
                lds_wait(&tm.done[slot], j_tail + 1);
                const Part<R> v = tm.res[slot][lane];
                if ((j_a1 >> slot) & 1) A1.add(v);
                else A0.add(v);
                ++j_tail;
            }
        };
        // gives buffer b of a kind out as a job, then takes the next buffer
        auto give = [&](int kind, int b, int cnt, int filler, int acc) {
            if constexpr (TEAM > 1) {
                if (j_next - j_tail == kTeamRing) fold();
                const int slot = j_next % kTeamRing;
                j_a1 = (j_a1 & ~(1u << slot)) | ((unsigned)acc << slot);
                tm.job[slot] = make_int4(kind, b, cnt, filler);
                tm.last[kind][b] = j_next;
                lds_store(&tm.head, ++j_next);
            }
        };
        auto next_buffer = [&](int kind, int& b) {
            if constexpr (TEAM > 1) {
                b = b + 1 < kTeamBufs ? b + 1 : 0;
                const int busy = uni(tm.last[kind][b]);
                while (j_tail <= busy) fold();
            }
        };
        auto flush_pn = [&](int cnt) {
            it_pn += entry_rounds(cnt, ksubA, rcpA);
            if (split) it_pn += entry_rounds(cnt, kB, rcpB);
            if constexpr (TEAM > 1) {
                give(kJobPn, b_pn, cnt, 0, pn_own);
                next_buffer(kJobPn, b_pn);
            } else {
                const Part<R> pa = tile_pn(T, r, lane, cnt, eps2);
                if (pn_own == 0) A0.add(pa);
                else A1.add(pa);
            }
        };
        auto flush_far = [&](int cnt, int runs) {
            it_far += entry_rounds(cnt, ksubN, rcpN);
            if constexpr (TEAM > 1) {
                give(kJobFar, b_far, cnt | runs << 16, 0, 0);
                next_buffer(kJobFar, b_far);
            } else {
                fill_tile<false>(T, p, ctr, lane, cnt, runs);
                A0.add(tile_far(T, r, cnt, eps2));
            }
        };
        bool had_lists = false;
        auto flush_near = [&](int cnt, int runs) {
            if (near_force) it_near += entry_rounds(cnt, ksubN, rcpN);
            if constexpr (TEAM > 1) {
                if (count_nbr) {
                    had_lists = true;
                    tm.list_job[j_list % (kTeamBufs + 1)] = make_int2(b_near, cnt | runs << 16);
                    lds_store(&tm.list_head, ++j_list);
                    tm.list_last[b_near] = j_list;
                }
                if (near_force) give(kJobNear, b_near, cnt | runs << 16, count_nbr ? j_list : 0, 1);
                next_buffer(kJobNear, b_near);
                lds_wait(&tm.list_done, uni(tm.list_last[b_near]));
            } else {
                fill_tile<true>(T, p, ctr, lane, cnt, runs);
                const Part<R> v = tile_near<false>(T, r, p, cnt, eps2, count_nbr, near_force, nbr);
                if (near_force) A1.add(v);
            }
        };
        auto group_sync = []() {   // between the lanes of this wave
            if constexpr (TEAM > 1) wave_sync();
            else __syncthreads();
        };
        if constexpr (TEAM > 1) {   // (no job of another group is under way)
            tm.group = (int)g;
            tm.turn = ++j_turn;
        }
        stack.put(0, root);   // every lane stores the same value
        int top = 1;
        bool overflow = false;

        while (top > 0) {
            // multipole tile: evaluated here, where no node state is live,
            // once it could not take another step's entries (up to 64)
            if (npn > TCAP - 32) {
                if (parts == 1 || pn_own == part) {
                    group_sync();
                    flush_pn(npn);
                    group_sync();
                }
                npn = 0;
                pn_tile = pn_tile < 4 ? pn_tile + 1 : 0;
                pn_own = pn_tile < 3 ? 0 : 1;
            }
            __threadfence_block();
            const int npop = uni(top < 64 ? top : 64);
            top -= npop;
            const bool has = lane < npop;
            int nd = root;
            if (top + npop <= kWalkStackLds) {   // (wave-uniform; the usual case)
                if (has) nd = s_stack[top + lane];
            } else {
                if (has) nd = stack.get(top + lane);
            }
            __threadfence_block();
            const WNode w = p.node.load(nd);
            // (the moments along with the node: one latency a step, and siblings' moments
            // lie side by side, whether or not all of them are accepted)
            Mom32 q32 = {};
            if (MIXED) q32 = p.q32.load(nd);
            double rcrit2 = w.rcrit2;
            asm volatile("" : "+v"(rcrit2));   // (with the other loads, not where it is compared)
            const double dbox2 = box_box_d2(glo, ghi, w.lo, w.hi);
            const bool near = (dbox2 < rlist2) || (dbox2 == 0.0);
            const bool accept = has && !near && p.use_theta && (box_pt_d2(glo, ghi, w.com) > rcrit2);
            const bool open = has && !accept;
            const bool leaf = w.nchild == 0;

            // multipole entries
            const uint64_t mk = __ballot(accept);
            if (mk) {
                const int k = uni(__popcll(mk));
                if (accept && (parts == 1 || pn_own == part)) {
                    R* e = s_tiles[b_pn].pn[npn + popc_below(mk)];
                    e[0] = (R)(w.com[0] - ctr[0]);
                    e[1] = (R)(w.com[1] - ctr[1]);
                    e[2] = (R)(w.com[2] - ctr[2]);
                    if (MIXED) {
                        // quadrupole scaled by 2.5 (see eval_pn<float>)
                        e[3] = q32.M; e[4] = 2.5f * q32.qxx; e[5] = 2.5f * q32.qyy; e[6] = 2.5f * q32.qzz;
                        e[7] = 2.5f * q32.qxy; e[8] = 2.5f * q32.qxz; e[9] = 2.5f * q32.qyz;
                    } else {
                        const Mom64 q = p.q64.load(nd);
                        e[3] = q.M; e[4] = q.qxx; e[5] = q.qyy; e[6] = q.qzz;
                        e[7] = q.qxy; e[8] = q.qxz; e[9] = q.qyz;
                    }
                }
                npn = uni(npn + k);
                c_pn += k;
            }

            // children of opened inner nodes
            const int nch = (open && !leaf) ? w.nchild : 0;
            const int incl = wave_incl_scan(nch, lane);
            const int tot = last_lane(incl);
            if (top + tot > p.stack_cap) {
                overflow = true;
                break;
            }
            if (top + tot <= kWalkStackLds) {   // (wave-uniform; the usual case)
                int* dst = s_stack + top + incl - nch;
#pragma unroll
                for (int k = 0; k < 8; ++k)
                    *(k < nch ? dst + k : s_stack + kWalkStackLds) = w.first_child + k;   // (no branches)
            } else {
                for (int k = 0; k < nch; ++k) stack.put(top + incl - nch + k, w.first_child + k);
            }
            top = uni(top + tot);

            // leaves: far ones (W = 1) and near ones (changeover)
            for (int cls = 0; cls < 2; ++cls) {
                const bool flag = open && leaf && (cls == 0 ? !near : near);
                const uint64_t lm = __ballot(flag);
                if (!lm) continue;
                const int v = flag ? w.count : 0;
                const int li = wave_incl_scan(v, lane);
                const int total = last_lane(li);
                if (cls == 0) c_far += total; else c_near += total;
                int fill = cls == 0 ? nfar : nnear, runs = cls == 0 ? rfar : rnear;
                const bool mine = cls == 0 ? far_mine : near_mine;
                for (int base = 0; base < total; base += 64) {
                    const int add = (total - base) < 64 ? (total - base) : 64;
                    if (fill + add > TCAP) {
                        group_sync();
                        if (cls == 0) {
                            if (far_mine) flush_far(fill, runs);
                        } else {
                            if (near_mine) flush_near(fill, runs);
                        }
                        fill = 0;
                        runs = 0;
                        group_sync();
                    }
                    if (mine) {
                        // the part of the lane's leaf among these entries
                        const int ex = li - v;
                        const int lo = ex > base ? ex : base, hi = li < base + add ? li : base + add;
                        const uint64_t rm = __ballot(lo < hi);
                        if (lo < hi) {
                            Tiles<R, TC>& F = s_tiles[cls == 0 ? b_far : b_near];
                            int (&run)[2][TC] = cls == 0 ? F.far_run : F.near_run;
                            const int k = runs + popc_below(rm), at = fill + lo - base;
                            run[0][k] = at;
                            run[1][k] = w.begin + (lo - ex) - at;
                        }
                        runs = uni(runs + __popcll(rm));
                    }
                    fill = uni(fill + add);
                }
                if (cls == 0) {
                    nfar = fill;
                    rfar = runs;
                } else {
                    nnear = fill;
                    rnear = runs;
                }
            }
        }
        group_sync();
        if (npn && (parts == 1 || pn_own == part)) flush_pn(npn);
        if (nfar && far_mine) flush_far(nfar, rfar);
        if (nnear && near_mine) flush_near(nnear, rnear);
        if constexpr (TEAM > 1) {
            while (j_tail < j_next) fold();
            lds_wait(&tm.list_done, j_list);
            nbr = had_lists ? tm.nbr[lane] : 0;
        }
        group_sync();

        const WalkArgs e = walk_args();
        // a row that overflowed sends the group's lists to the fill pass
        const bool row_full = count_nbr && real && nbr > scap;
        const bool need_fill = count_nbr && (e->stage == nullptr || __ballot(row_full) != 0);
        if (!split && ksubA > 1) {
            const int ksub = ksubA;
            // merge the copies' partial sums in copy order, into copy 0
            R* red = &T.pn[0][0];
            constexpr int W = Acc<R>::kWords + 1;   // odd stride: no LDS bank conflicts
            A0.store(red + W * lane);
            A1.store(red + W * (64 + lane));
            T.nearj[lane] = nbr;
            group_sync();
            // (the barrier also makes the copies' staged entries visible)
            if (active) {
                const bool join = count_nbr && !need_fill;
                int32_t* base = join ? e->stage + stage_index(me, 0, e->scap) : nullptr;
                for (int c = 1; c < ksub; ++c) {
                    A0.merge(red + W * (c * gcnt + lane));
                    A1.merge(red + W * (64 + c * gcnt + lane));
                    const int nc = T.nearj[c * gcnt + lane];
                    // move copy c's sub-row down to follow the list so far;
                    // targets lie below sources, loads of a batch precede its stores
                    if (join) {
                        for (int t0 = 0; t0 < nc; t0 += 8) {
                            int v[8];
#pragma unroll
                            for (int u = 0; u < 8; ++u) {
                                const int t = t0 + u < nc ? t0 + u : nc - 1;
                                v[u] = base[(int64_t)(c * wrow + t) * kStageStride];
                            }
#pragma unroll
                            for (int u = 0; u < 8; ++u)
                                if (t0 + u < nc) base[(int64_t)(nbr + t0 + u) * kStageStride] = v[u];
                        }
                    }
                    nbr += nc;
                }
            }
            group_sync();
        }
        if (overflow) atomicOr(&e->cnt[kErr], lane == 0 ? kErrWalkStack : 0ull);
        if (count_nbr) {
            // lists this walk did not stage completely go to the fill pass
            if (need_fill) {
                // all lanes issue the atomic (lane 0 adds 1): no lane-0-only branch
                const unsigned long long slot =
                    atomicAdd(&e->cnt[kCntFill], lane == 0 ? 1ull : 0ull);
                if (lane == 0) e->fill_list[slot] = (int32_t)g;
            }
            if (active) e->stage_k[me] = (int8_t)(need_fill ? 0 : 1);
        }
        if (active && count_nbr) e->nbr_cnt[e->perm[me]] = nbr;
        bool last = true;
        if (parts == 1) {
            R w[Acc<R>::kWords];
            A1.store(w);
            A0.merge(w);
        } else {
            // The wave that comes last adds up both sums, as one wave would. They
            // cross XCDs, whose L2s are not coherent with each other: device-scope
            // accesses, and the count is raised only after the stores have arrived
            // (a fence at that scope would write back and invalidate a whole L2).
            R* sum = reinterpret_cast<R*>(e->part_sum) + (int64_t)item.slot * (Acc<R>::kWords * 64);
            R w[Acc<R>::kWords];
            if (!lead) A0 = A1;
            A0.store(w);
#pragma unroll
            for (int k = 0; k < Acc<R>::kWords; ++k)
                __hip_atomic_store(sum + (part * Acc<R>::kWords + k) * 64 + lane, w[k], __ATOMIC_RELAXED,
                                   __HIP_MEMORY_SCOPE_AGENT);
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            last = uni((int)atomicAdd(e->part_done + item.slot / 2, lane == 0 ? 1u : 0u)) == 1;
            if (last) {
#pragma unroll
                for (int k = 0; k < Acc<R>::kWords; ++k)
                    w[k] = __hip_atomic_load(sum + ((part ^ 1) * Acc<R>::kWords + k) * 64 + lane, __ATOMIC_RELAXED,
                                             __HIP_MEMORY_SCOPE_AGENT);
                // (the first sum takes the second)
                Acc<R> B;
                B.load(w);
                if (lead) {
                    A0.merge(w);
                } else {
                    A0.store(w);
                    B.merge(w);
                    A0 = B;
                }
            }
        }
        if (active && last) {
            const int orig = e->perm[me];
            e->acc[3 * (int64_t)orig] = A0.gx();
            e->acc[3 * (int64_t)orig + 1] = A0.gy();
            e->acc[3 * (int64_t)orig + 2] = A0.gz();
            e->pot[orig] = A0.gp();
        }
        if (lead) {
            sum_pn += (unsigned long long)c_pn * gcnt;
            sum_far += (unsigned long long)c_far * gcnt;
            sum_near += (unsigned long long)c_near * gcnt;
        }
        slot_pn += it_pn;
        slot_far += it_far;
        slot_near += it_near;
    }
    if constexpr (TEAM > 1) lds_store(&tm.end, 1);   // (no jobs are left)
    const WalkArgs z = walk_args();
    if (!first && (slot_pn | slot_far | slot_near)) {
        // one contribution per wave (lane 0, the others add 0), spread over lines
        unsigned long long* c = z->walk_cnt + (blockIdx.x % kWalkCntLines) * kQueueStride;
        const unsigned long long l0 = lane == 0 ? 1ull : 0ull;
        atomicAdd(c, sum_pn * l0);
        atomicAdd(c + 1, sum_far * l0);
        atomicAdd(c + 2, sum_near * l0);
        atomicAdd(c + 3, slot_pn * 64ull * l0);
        atomicAdd(c + 4, slot_far * 64ull * l0);
        atomicAdd(c + 5, slot_near * 64ull * l0);
    }
    if (z->wave_log) {
        const unsigned long long c_end = clock64();
        z->wave_log[2 * blockIdx.x] = (unsigned long long)n_walked;
        z->wave_log[2 * blockIdx.x + 1] = wall_clock64() - t_start;
        z->wave_cyc[blockIdx.x] = c_end - c_start;
    }
}

// rcrit^2 = (l/theta + delta)^2 per node, l = largest box extent, delta =
// |COM - box centre|; also clears the per-call counters and queues, and stores the
// changeover constants of a single cluster (a launch of its own took them 3 us and a gap of 4).
__global__ void k_rcrit(NodePlanes node, const unsigned long long* __restrict__ n_dev,
                        double theta, unsigned long long* __restrict__ cnt,
                        unsigned long long* __restrict__ queues, unsigned* __restrict__ part_done, int n_part,
                        ClusterParams cp0, ClusterParams* __restrict__ cp_dst) {
#pragma clang fp contract(off)
    const int64_t n = (int64_t)*n_dev;
    if (blockIdx.x == 0) {   // the queue heads, then the counter lines
        for (int k = threadIdx.x; k < kQueueWords; k += blockDim.x) queues[k] = 0;
        if (threadIdx.x == 0) cnt[kCntFill] = 0;
        if (threadIdx.x == 0 && cp_dst) *cp_dst = cp0;
    }
    for (int64_t b = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; b < n_part;
         b += (int64_t)gridDim.x * blockDim.x)
        part_done[b] = 0u;
    for (int64_t b = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; b < n;
         b += (int64_t)gridDim.x * blockDim.x) {
        WNode w;
        node.box(b, w.lo, w.hi);
        node.com(b, w.com);
        double l = 0.0;
        for (int k = 0; k < 3; ++k)
            if (w.hi[k] - w.lo[k] > l) l = w.hi[k] - w.lo[k];
        double dd[3];
        for (int k = 0; k < 3; ++k) dd[k] = w.com[k] - (w.lo[k] + w.hi[k]) * 0.5;
        const double delta = sqrt(dd[0] * dd[0] + dd[1] * dd[1] + dd[2] * dd[2]);
        const double rc = theta > 0.0 ? l / theta + delta : 0.0;
        node.set_rcrit2(b, rc * rc);
    }
}

}  // namespace

void launch_rcrit(Dev& d, const BuildCfg& c, double theta, const ClusterParams* cp0, hipStream_t s) {
    int64_t nb = (c.node_cap + 255) / 256;
    if (nb > 4096) nb = 4096;
    hipLaunchKernelGGL(k_rcrit, dim3(nb), dim3(256), 0, s, d.node,
                       (const unsigned long long*)(d.cnt + kCntNodes), theta, d.cnt, d.queues, d.part_done, kWalkShared,
                       cp0 ? *cp0 : ClusterParams{}, cp0 ? d.cparams : nullptr);
}

template <bool MIXED>
static auto walk_kernel(int tile) {
    return tile == 128 ? k_walk<MIXED, 128, 1> : (tile == 96 ? k_walk<MIXED, 96, 1> : k_walk<MIXED, 64, 1>);
}

// Up to here a team walks each group. Few groups leave the chip idle but for the
// longest ones, whose walk is a chain of latencies that four waves shorten; with
// more, four groups on a SIMD cover each other's latencies and a team's idle waves
// are lost. Walk in us, one wave a group / a team: 700 particles 87 / 73, 4096 184
// / 138, 16384 301 / 226, 32768 358 / 322, 40960 409 / 366 (nbar 200: 827 / 745),
// 49152 440 / 436, 65536 505 / 550, 131072 812 / 970; uniform 28000 159 / 139, 36000
// 180 / 174, 40000 201 / 186; lattice 32768 96 / 91, 35937 113 / 124, 39304 117 / 135.
constexpr int64_t kTeamMaxN = 40960;

bool walk_team(int mixed, int tile, int64_t n) { return mixed && tile == 64 && n <= kTeamMaxN; }

int walk_blocks_per_cu(int mixed, int tile, bool team) {
    int nb = 0;
    if (team) hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, k_walk<true, 64, kTeamWaves>, 64 * kTeamWaves, 0);
    else if (mixed) hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, walk_kernel<true>(tile), 64, 0);
    else hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, walk_kernel<false>(tile), 64, 0);
    return nb > 0 ? nb : 1;
}

void launch_walk(Dev& d, const BuildCfg& c, const WalkCfg& w, double* acc, double* pot,
                 hipStream_t s) {
    WalkParams p;
    p.node = d.node;
    p.q32 = d.q32;
    p.q64 = d.q64;
    p.x = d.x; p.y = d.y; p.z = d.z; p.m = d.m;
    p.perm = d.perm;
    p.g_begin = d.g.begin; p.g_count = d.g.count; p.g_root = d.g.root; p.g_cluster = d.g.cluster;
    p.g_lo = d.g.lo; p.g_hi = d.g.hi;
    p.cp = d.cparams;
    p.G = d.cnt + kCntGroups;
    p.use_theta = w.theta > 0.0;
    p.eps2 = w.eps * w.eps;
    p.acc = acc;
    p.pot = pot;
    p.stack = d.stack;
    p.stack_cap = w.stack_cap;
    p.cnt = d.cnt;
    p.queues = d.queues;
    p.walk_cnt = d.queues + kWalkCntAt;
    p.wave_log = d.wave_log;
    p.wave_cyc = d.wave_cyc;
    p.nbr_cnt = w.count_nbr ? d.nbr_cnt : nullptr;
    p.stage = (w.count_nbr && w.stage_cap > 0) ? d.nbr_stage : nullptr;
    p.scap = w.stage_cap;
    p.stage_k = d.stage_k;
    p.fill_list = d.fill_list;
    p.max_copies = w.max_copies;
    p.cpos = w.cpos;
    p.cmass = w.cmass;
    p.part_sum = d.part_sum;
    p.part_done = d.part_done;
    if (w.team) hipLaunchKernelGGL((k_walk<true, 64, kTeamWaves>), dim3(w.grid), dim3(64 * kTeamWaves), 0, s, p);
    else if (w.mixed) hipLaunchKernelGGL(walk_kernel<true>(w.tile), dim3(w.grid), dim3(64), 0, s, p);
    else hipLaunchKernelGGL(walk_kernel<false>(w.tile), dim3(w.grid), dim3(64), 0, s, p);
}

}  // namespace pbh
