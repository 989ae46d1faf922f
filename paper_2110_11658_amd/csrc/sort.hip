// sort.hip -- device-wide exclusive scan and stable sorts of 64-bit keys (gfx950).
//
// Scan: launches of fixed size (so they can be captured in a graph): per-tile
// sums, then per-tile scans, each tile adding the sums of the tiles before it
// (summed by its own workgroup while there are at most kScanFuseTiles tiles;
// beyond that a single workgroup scans the tile sums in a launch between).
//
// Sorts: a sample sort for the (key, position) pairs of a build and of the core
// quantities up to 2^22 of them, an LSD radix sort beyond that.
//
// Radix sort: 8-bit digits. Per pass a tile
// histogram (LDS atomics), a scan of the digit-major histogram table, and a
// stable scatter in which each wave ranks equal digits with one ballot per
// digit bit (match by bits) and the waves of a workgroup are ordered through
// LDS.
#include "pbh_internal.hpp"
#include "sample_sort.hpp"
#include "wave.hpp"

namespace pbh {

namespace {

constexpr int SCAN_T = 256;
constexpr int SCAN_I = 4;   // 1024 elements per tile (2, 8 and 16 built slower at 2^20; 2 leaves the fused path at 4M)
constexpr int SCAN_TILE = SCAN_T * SCAN_I;

__device__ inline int64_t wave_incl_scan64(int64_t v, int lane) {
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        int64_t t = __shfl_up(v, o, 64);
        if (lane >= o) v += t;
    }
    return v;
}

// exclusive scan over a 256-thread block; returns the exclusive prefix, total in *tot
__device__ inline int64_t block_excl_scan(int64_t v, int64_t* s_wave, int64_t* tot) {
    const int t = threadIdx.x, lane = t & 63, w = t >> 6;
    int64_t inc = wave_incl_scan64(v, lane);
    if (lane == 63) s_wave[w] = inc;
    __syncthreads();
    int64_t base = 0, all = 0;
    for (int k = 0; k < SCAN_T / 64; ++k) {
        if (k < w) base += s_wave[k];
        all += s_wave[k];
    }
    *tot = all;
    __syncthreads();
    return base + inc - v;
}

template <typename T>
__global__ __launch_bounds__(SCAN_T) void k_scan_reduce(const T* __restrict__ in, int64_t n,
                                                        int64_t* __restrict__ tmp) {
    __shared__ int64_t s_wave[SCAN_T / 64];
    const int64_t base = (int64_t)blockIdx.x * SCAN_TILE;
    int64_t v = 0;
#pragma unroll
    for (int k = 0; k < SCAN_I; ++k) {
        int64_t i = base + k * SCAN_T + threadIdx.x;
        if (i < n) v += (int64_t)in[i];
    }
    int64_t tot;
    block_excl_scan(v, s_wave, &tot);
    if (threadIdx.x == 0) tmp[blockIdx.x] = tot;
}

__global__ __launch_bounds__(1024) void k_scan_top(int64_t* __restrict__ tmp, int64_t nb) {
    __shared__ int64_t s_wave[16];
    const int t = threadIdx.x, lane = t & 63, w = t >> 6;
    const int64_t per = (nb + 1023) / 1024;
    const int64_t b0 = t * per;
    int64_t sum = 0;
    for (int64_t k = 0; k < per; ++k)
        if (b0 + k < nb) sum += tmp[b0 + k];
    int64_t inc = wave_incl_scan64(sum, lane);
    if (lane == 63) s_wave[w] = inc;
    __syncthreads();
    int64_t base = 0, all = 0;
    for (int k = 0; k < 16; ++k) {
        if (k < w) base += s_wave[k];
        all += s_wave[k];
    }
    int64_t run = base + inc - sum;
    for (int64_t k = 0; k < per; ++k) {
        if (b0 + k < nb) {
            int64_t v = tmp[b0 + k];
            tmp[b0 + k] = run;
            run += v;
        }
    }
    if (t == 0) tmp[nb] = all;
}

template <typename T, typename O>
__global__ __launch_bounds__(SCAN_T) void k_scan_down(const T* in, int64_t n,
                                                      const int64_t* __restrict__ tmp, O* out,
                                                      int64_t nb) {
    __shared__ int64_t s_val[SCAN_TILE];
    __shared__ int64_t s_wave[SCAN_T / 64];
    const int64_t base = (int64_t)blockIdx.x * SCAN_TILE;
#pragma unroll
    for (int k = 0; k < SCAN_I; ++k) {
        int64_t i = base + k * SCAN_T + threadIdx.x;
        s_val[k * SCAN_T + threadIdx.x] = (i < n) ? (int64_t)in[i] : 0;
    }
    __syncthreads();
    int64_t v[SCAN_I];
    int64_t sum = 0;
#pragma unroll
    for (int k = 0; k < SCAN_I; ++k) {
        v[k] = s_val[threadIdx.x * SCAN_I + k];
        sum += v[k];
    }
    int64_t tot;
    int64_t run = block_excl_scan(sum, s_wave, &tot) + tmp[blockIdx.x];
#pragma unroll
    for (int k = 0; k < SCAN_I; ++k) {
        s_val[threadIdx.x * SCAN_I + k] = run;
        run += v[k];
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < SCAN_I; ++k) {
        int64_t i = base + k * SCAN_T + threadIdx.x;
        if (i < n) out[i] = (O)s_val[k * SCAN_T + threadIdx.x];
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) out[n] = (O)tmp[nb];
}

// Per-tile scan with the tile's offset summed here from the tile sums before
// it (tmp[0 .. blockIdx.x), in index order per thread, then across the
// workgroup); the last tile also writes the total to out[n].
constexpr int64_t kScanFuseTiles = 4096;
constexpr int64_t kScanFewTiles = 8;

template <typename T, typename O>
__global__ __launch_bounds__(SCAN_T) void k_scan_down_fused(const T* in, int64_t n,
                                                            const int64_t* __restrict__ tmp, O* out,
                                                            int64_t nb) {
    __shared__ int64_t s_val[SCAN_TILE];
    __shared__ int64_t s_wave[SCAN_T / 64];
    const int t = threadIdx.x, lane = t & 63, w = t >> 6;
    const int64_t base = (int64_t)blockIdx.x * SCAN_TILE;
    int64_t part = 0;
    if (tmp) {
        for (int64_t k = t; k < (int64_t)blockIdx.x; k += SCAN_T) part += tmp[k];
    } else {   // few tiles, and `in` is not `out`: summed here
#pragma unroll 8
        for (int64_t k = t; k < base; k += SCAN_T) part += (int64_t)in[k];
    }
    for (int o = 32; o > 0; o >>= 1) part += __shfl_xor(part, o, 64);
    if (lane == 0) s_wave[w] = part;
    __syncthreads();
    int64_t off = 0;
    for (int k = 0; k < SCAN_T / 64; ++k) off += s_wave[k];
    __syncthreads();
#pragma unroll
    for (int k = 0; k < SCAN_I; ++k) {
        int64_t i = base + k * SCAN_T + t;
        s_val[k * SCAN_T + t] = (i < n) ? (int64_t)in[i] : 0;
    }
    __syncthreads();
    int64_t v[SCAN_I];
    int64_t sum = 0;
#pragma unroll
    for (int k = 0; k < SCAN_I; ++k) {
        v[k] = s_val[t * SCAN_I + k];
        sum += v[k];
    }
    int64_t tot;
    int64_t run = block_excl_scan(sum, s_wave, &tot) + off;
#pragma unroll
    for (int k = 0; k < SCAN_I; ++k) {
        s_val[t * SCAN_I + k] = run;
        run += v[k];
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < SCAN_I; ++k) {
        int64_t i = base + k * SCAN_T + t;
        if (i < n) out[i] = (O)s_val[k * SCAN_T + t];
    }
    if (blockIdx.x == nb - 1 && t == 0) out[n] = (O)(off + tot);
}

template <typename T, typename O>
void scan_impl(const T* in, O* out, int64_t n, int64_t* tmp, hipStream_t s) {
    const int64_t nb = (n + SCAN_TILE - 1) / SCAN_TILE;
    if (nb >= 1 && nb <= kScanFuseTiles) {
        // up to kScanFewTiles a workgroup sums the tiles before its own itself: cheaper than
        // a launch (lists of 700 particles 19 -> 16 us, 4096 19.8 -> 17.5). Not in place, where those are being overwritten.
        const bool few = nb <= kScanFewTiles && (const void*)in != (const void*)out;
        if (!few) hipLaunchKernelGGL((k_scan_reduce<T>), dim3(nb), dim3(SCAN_T), 0, s, in, n, tmp);
        hipLaunchKernelGGL((k_scan_down_fused<T, O>), dim3(nb), dim3(SCAN_T), 0, s, in, n,
                           few ? nullptr : (const int64_t*)tmp, out, nb);
        return;
    }
    if (nb == 0) {
        // n == 0: out[0] = 0 through the top kernel with nb = 0
        hipLaunchKernelGGL(k_scan_top, dim3(1), dim3(1024), 0, s, tmp, (int64_t)0);
        hipLaunchKernelGGL((k_scan_down<T, O>), dim3(1), dim3(SCAN_T), 0, s, in, (int64_t)0,
                           (const int64_t*)tmp, out, (int64_t)0);
        return;
    }
    hipLaunchKernelGGL((k_scan_reduce<T>), dim3(nb), dim3(SCAN_T), 0, s, in, n, tmp);
    hipLaunchKernelGGL(k_scan_top, dim3(1), dim3(1024), 0, s, tmp, nb);
    hipLaunchKernelGGL((k_scan_down<T, O>), dim3(nb), dim3(SCAN_T), 0, s, in, n,
                       (const int64_t*)tmp, out, nb);
}

// ---------------------------------------------------------------- radix sort
constexpr int RS_T = 256;
constexpr int RS_R = 16;            // rounds per tile (4096 keys; 4, 8, 12, 20, 24 and 32 built slower at 2^20)
constexpr int RS_TILE = RS_T * RS_R;
constexpr int RS_MAX_BINS = 256;    // bins of the widest digit used

// Tile histogram of one digit (BITS wide, at `shift`), digit-major table.
template <int BITS>
__global__ __launch_bounds__(RS_T) void k_rs_hist(const uint64_t* __restrict__ keys, int64_t n,
                                                  int shift, int64_t* __restrict__ hist, int64_t nblk) {
    constexpr int BINS = 1 << BITS;
    constexpr unsigned MASK = BINS - 1;
    __shared__ int s_h[BINS];
    for (int d = threadIdx.x; d < BINS; d += RS_T) s_h[d] = 0;
    __syncthreads();
    const int64_t base = (int64_t)blockIdx.x * RS_TILE;
    uint64_t k[RS_R];
#pragma unroll
    for (int r = 0; r < RS_R; ++r) {
        const int64_t i = base + r * RS_T + threadIdx.x;
        k[r] = i < n ? keys[i] : 0ull;
    }
#pragma unroll
    for (int r = 0; r < RS_R; ++r) {
        const int64_t i = base + r * RS_T + threadIdx.x;
        if (i < n) atomicAdd(&s_h[(unsigned)(k[r] >> shift) & MASK], 1);
    }
    __syncthreads();
    for (int d = threadIdx.x; d < BINS; d += RS_T) hist[(int64_t)d * nblk + blockIdx.x] = s_h[d];
}

__device__ inline uint64_t lanes_below(int lane) {
    return (lane == 0) ? 0ull : (~0ull >> (64 - lane));
}

template <int BITS>
__global__ __launch_bounds__(RS_T) void k_rs_scatter(const uint64_t* __restrict__ kin,
                                                     const int32_t* __restrict__ vin,
                                                     uint64_t* __restrict__ kout,
                                                     int32_t* __restrict__ vout, int64_t n,
                                                     int shift,
                                                     const int64_t* __restrict__ hist,
                                                     int64_t nblk, int iota) {
    constexpr int BINS = 1 << BITS;
    constexpr unsigned MASK = BINS - 1;
    constexpr int PER = BINS / RS_T;   // bins per thread
    __shared__ int64_t s_goff[BINS];
    __shared__ int s_run[BINS];
    __shared__ int s_wc[RS_T / 64][BINS];
    const int t = threadIdx.x, lane = t & 63, w = t >> 6;
#pragma unroll
    for (int u = 0; u < PER; ++u) {
        s_goff[t + u * RS_T] = hist[(int64_t)(t + u * RS_T) * nblk + blockIdx.x];
        s_run[t + u * RS_T] = 0;
    }
    const int64_t base = (int64_t)blockIdx.x * RS_TILE;
    const uint64_t below = lanes_below(lane);
    // every round's key and value are loaded up front: one memory latency per
    // tile instead of one per round (the rounds are separated by barriers)
    uint64_t keys[RS_R];
    int32_t vals[RS_R];
#pragma unroll
    for (int r = 0; r < RS_R; ++r) {
        const int64_t i = base + r * RS_T + t;
        const bool valid = i < n;
        keys[r] = valid ? kin[i] : 0ull;
        vals[r] = valid ? (iota ? (int32_t)i : vin[i]) : 0;
    }
#pragma unroll
    for (int r = 0; r < RS_R; ++r) {
        const int64_t i = base + r * RS_T + t;
        const bool valid = i < n;
        const uint64_t key = keys[r];
        const int32_t val = vals[r];
        const unsigned d = (unsigned)(key >> shift) & MASK;
#pragma unroll
        for (int u = 0; u < PER; ++u)
            for (int k = 0; k < RS_T / 64; ++k) s_wc[k][t + u * RS_T] = 0;
        __syncthreads();
        uint64_t peers = __ballot(valid);
#pragma unroll
        for (int b = 0; b < BITS; ++b) {
            const bool bit = (d >> b) & 1u;
            const uint64_t m = __ballot(bit);
            peers &= bit ? m : ~m;
        }
        const int rank = __popcll(peers & below);
        if (valid && rank == 0) s_wc[w][d] = __popcll(peers);
        __syncthreads();
#pragma unroll
        for (int u = 0; u < PER; ++u) {
            const int bin = t + u * RS_T;
            int run = s_run[bin];
            for (int k = 0; k < RS_T / 64; ++k) {
                int c = s_wc[k][bin];
                s_wc[k][bin] = run;
                run += c;
            }
            s_run[bin] = run;
        }
        __syncthreads();
        if (valid) {
            const int64_t dst = s_goff[d] + s_wc[w][d] + rank;
            kout[dst] = key;
            vout[dst] = val;
        }
        __syncthreads();
    }
}

__global__ void k_copy_pairs(const uint64_t* __restrict__ ks, const int32_t* __restrict__ vs,
                             uint64_t* __restrict__ kd, int32_t* __restrict__ vd, int64_t n) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x) {
        kd[i] = ks[i];
        vd[i] = vs[i];
    }
}

// --------------------------------------------------------------- sample sort
// Stable sort of up to kSsMaxN (key, index) pairs, the indices being 0..n-1 on
// entry. Up to kSsCap keys: one workgroup sorts them in LDS. More: the keys are
// split into S buckets of 1024 to 2048 keys on average by S - 1 splitters (every
// kSsOver-th of S * kSsOver samples in sorted order, a sample drawn from each of
// as many equal stretches of the keys, see ss_sample_at), scattered to their
// buckets in a stable order, and one workgroup sorts each bucket in LDS. Keys are
// compared as (key, index) pairs, so equal keys spread over buckets like any
// others. A bucket passes kSsCap, 4 to 8 times the average, where the samples drawn
// misrepresent the keys that much: with probability 3e-6 a bucket for places drawn
// at random. Such a bucket is sorted by its workgroup in global memory.
//
// Against the 8-bit LSD radix sort (8 passes of 4 launches over the whole array
// for 63-bit keys) a key moves through global memory twice instead of sixteen
// times, in 6 launches instead of 32: 105 us against 243 us for 2^20 Morton
// keys, 53 against 200 for 2^17, 29 against 165 for 4096 (kernel times). What is
// left is latency: the sort of the buckets takes half of it, five digit passes
// of barriers and LDS round trips in each of 512 workgroups.
constexpr int kSsT = 1024;          // threads of a workgroup that sorts in LDS
constexpr int kSsR = kSsCap / kSsT; // keys per thread

__device__ inline uint64_t ss_lanes_below(int lane) { return (lane == 0) ? 0ull : (~0ull >> (64 - lane)); }

// the m samples, side by side (read in place by every workgroup of the ranking,
// each on a 128-byte line of its own)
__global__ __launch_bounds__(256) void k_ss_gather(const uint64_t* __restrict__ keys, int64_t n, int m,
                                                   uint64_t* __restrict__ sample) {
    const int j = blockIdx.x * 256 + threadIdx.x;
    if (j < m) sample[j] = keys[ss_sample_at(j, n, m)];
}

// Ranks 32 of the m samples per workgroup by counting, 32 threads a sample,
// each over a slice of the samples, which pass through LDS in chunks. Equal
// samples rank in their order: those before this one count when not above it,
// those after it when below it. A sample whose rank is a multiple of kSsOver is
// a splitter.
constexpr int kRankChunk = 4096;
__global__ __launch_bounds__(1024) void k_ss_split(const uint64_t* __restrict__ sample, int64_t n, int m,
                                                   uint64_t* __restrict__ sp_key, int32_t* __restrict__ sp_idx) {
    __shared__ uint64_t s_k[kRankChunk];
    __shared__ int s_cnt[32];
    const int t = threadIdx.x, q = t & 31, part = t >> 5;
    if (t < 32) s_cnt[t] = 0;
    const int me = blockIdx.x * 32 + q;   // m is a multiple of 32
    const uint64_t mk = sample[me];
    int below = 0;
    for (int c0 = 0; c0 < m; c0 += kRankChunk) {
        const int len = m - c0 < kRankChunk ? m - c0 : kRankChunk;
        __syncthreads();
        for (int u = t; u < len; u += 1024) s_k[u] = sample[c0 + u];
        __syncthreads();
        const int per = len / 32;   // len is a multiple of 32
        const int u0 = part * per, u1 = u0 + per;
        const int mid = min(max(me - c0, u0), u1);
#pragma unroll 4
        for (int u = u0; u < mid; ++u) below += s_k[u] <= mk ? 1 : 0;
#pragma unroll 4
        for (int u = mid; u < u1; ++u) below += s_k[u] < mk ? 1 : 0;
    }
    atomicAdd(&s_cnt[q], below);
    __syncthreads();
    if (t < 32) {
        const int r = s_cnt[t];
        if (r > 0 && r % kSsOver == 0) {
            sp_key[r / kSsOver] = mk;
            sp_idx[r / kSsOver] = (int32_t)ss_sample_at(me, n, m);
        }
    }
}

// Bucket of (key, i): the number of splitters 1 .. S-1 not above it.
__device__ inline int ss_bucket(const uint64_t* s_sp, const int32_t* __restrict__ sp_idx, int S, uint64_t key,
                                int64_t i) {
    int k = 0;
    for (int st = S >> 1; st > 0; st >>= 1)   // S is a power of two; entry 0 is not a splitter
        if (s_sp[k + st] <= key) k += st;
    // splitters with this very key: the index decides
    if (k > 0 && s_sp[k] == key) {
        int lo = 0;
        for (int st = S >> 1; st > 0; st >>= 1)
            if (lo + st <= k && (s_sp[lo + st] < key || (int64_t)sp_idx[lo + st] <= i)) lo += st;
        k = lo;
    }
    return k;
}

// Partition, first half: buckets of a tile of T * R keys and the tile's count
// per bucket, table[tile][bucket]. In both halves wave w of a tile holds its
// keys w * 64 R .. and key 64 r + lane of them in its round r.
template <int T, int R>
__global__ __launch_bounds__(T) void k_ss_count(const uint64_t* __restrict__ keys, int64_t n, int S,
                                                const uint64_t* __restrict__ sp_key,
                                                const int32_t* __restrict__ sp_idx, uint16_t* __restrict__ bucket,
                                                int32_t* __restrict__ table) {
    extern __shared__ uint64_t s_dyn[];
    uint64_t* s_sp = s_dyn;                         // [S]
    int* s_h = reinterpret_cast<int*>(s_dyn + S);   // [S]
    const int t = threadIdx.x;
    const int64_t base = (int64_t)blockIdx.x * (T * R) + (t >> 6) * (64 * R) + (t & 63);
    uint64_t k[R];
#pragma unroll
    for (int r = 0; r < R; ++r) k[r] = base + r * 64 < n ? keys[base + r * 64] : 0ull;
    for (int b = t; b < S; b += T) {
        s_sp[b] = b ? sp_key[b] : 0ull;
        s_h[b] = 0;
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int64_t i = base + r * 64;
        if (i < n) {
            const int b = ss_bucket(s_sp, sp_idx, S, k[r], i);
            bucket[i] = (uint16_t)b;
            atomicAdd(&s_h[b], 1);
        }
    }
    __syncthreads();
    for (int b = t; b < S; b += T) table[(int64_t)blockIdx.x * S + b] = s_h[b];
}

// Exclusive prefix over the tiles for every bucket, in place, and the bucket
// totals: 16 buckets a workgroup, 64 threads a bucket with a run of tiles each.
__global__ __launch_bounds__(1024) void k_ss_scan(int32_t* __restrict__ table, int ntile, int S,
                                                  int32_t* __restrict__ total) {
    __shared__ int s_sum[64][16];
    const int q = threadIdx.x & 15, c = threadIdx.x >> 4;
    const int b = blockIdx.x * 16 + q;
    const int per = (ntile + 63) / 64;
    const int t0 = c * per, t1 = t0 + per < ntile ? t0 + per : ntile;
    int sum = 0;
    if (b < S) {
#pragma unroll 8
        for (int t = t0; t < t1; ++t) sum += table[(int64_t)t * S + b];
    }
    s_sum[c][q] = sum;
    __syncthreads();
    if (threadIdx.x < 16) {
        int run = 0;
        for (int k = 0; k < 64; ++k) {
            const int v = s_sum[k][threadIdx.x];
            s_sum[k][threadIdx.x] = run;
            run += v;
        }
        if (blockIdx.x * 16 + (int)threadIdx.x < S) total[blockIdx.x * 16 + threadIdx.x] = run;
    }
    __syncthreads();
    if (b < S) {
        int run = s_sum[c][q];
#pragma unroll 8
        for (int t = t0; t < t1; ++t) {
            const int v = table[(int64_t)t * S + b];
            table[(int64_t)t * S + b] = run;
            run += v;
        }
    }
}

// exclusive scan of v[0 .. len) in LDS by the workgroup's NT threads; s_w has
// NT / 64 entries
template <int NT>
__device__ inline void ss_lds_scan(int* v, int len, int* s_w) {
    const int t = threadIdx.x, lane = t & 63, w = t >> 6;
    const int per = (len + NT - 1) / NT, b0 = t * per;
    int sum = 0;
    for (int k = 0; k < per; ++k)
        if (b0 + k < len) sum += v[b0 + k];
    const int inc = wave_incl_scan(sum, lane);
    if (lane == 63) s_w[w] = inc;
    __syncthreads();
    int run = inc - sum;
    for (int k = 0; k < w; ++k) run += s_w[k];
    for (int k = 0; k < per; ++k)
        if (b0 + k < len) {
            const int u = v[b0 + k];
            v[b0 + k] = run;
            run += u;
        }
    __syncthreads();
}

// lanes of this wave that hold a valid item with the same `bits` low bits of d
__device__ inline uint64_t ss_peers(unsigned d, bool valid, int bits) {
    uint64_t peers = __ballot(valid);
    for (int b = 0; b < bits; ++b) {
        const bool on = (d >> b) & 1u;
        const uint64_t m = __ballot(on);
        peers &= on ? m : ~m;
    }
    return peers;
}

// Partition, second half: every key to its bucket, in tile and key order (a
// wave ranks equal buckets with one ballot per bucket bit, the waves of a tile
// are ordered through their counts in LDS). The tile's keys are put in bucket
// order in LDS first, so that neighbouring lanes store to neighbouring
// addresses. Workgroup 0 writes the bucket offsets for the sort of the buckets.
template <int T, int R>
__global__ __launch_bounds__(T) void k_ss_scatter(const uint64_t* __restrict__ keys, int64_t n, int S, int bits,
                                                  const uint16_t* __restrict__ bucket,
                                                  const int32_t* __restrict__ table,
                                                  const int32_t* __restrict__ total, int32_t* __restrict__ base_out,
                                                  uint64_t* __restrict__ kout, int32_t* __restrict__ vout) {
    constexpr int NW = T / 64;
    extern __shared__ uint64_t s_dyn[];
    uint64_t* s_key = s_dyn;                                             // [T R] tile in bucket order
    uint16_t* s_at = reinterpret_cast<uint16_t*>(s_key + T * R);         // [T R] position in the tile
    uint16_t* s_bk = s_at + T * R;                                       // [T R] bucket
    int* s_base = reinterpret_cast<int*>(s_bk + T * R);                  // [S] bucket's place in the output
    int* s_loc = s_base + S;                                             // [S] its place in the tile
    uint16_t* s_wc = reinterpret_cast<uint16_t*>(s_loc + S);             // [NW][S]
    __shared__ int s_w[NW];
    const int t = threadIdx.x, lane = t & 63, w = t >> 6;
    const int64_t tile0 = (int64_t)blockIdx.x * (T * R);
    const int at0 = w * (64 * R) + lane;
    const int cnt = n - tile0 < T * R ? (int)(n - tile0) : T * R;
    uint64_t k[R];
    uint32_t b[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const bool in = at0 + r * 64 < cnt;
        k[r] = in ? keys[tile0 + at0 + r * 64] : 0ull;
        b[r] = in ? bucket[tile0 + at0 + r * 64] : 0u;
    }
    for (int q = t; q < S; q += T) {
        s_base[q] = total[q];
        for (int v = 0; v < NW; ++v) s_wc[v * S + q] = 0;
    }
    __syncthreads();
    ss_lds_scan<T>(s_base, S, s_w);
    if (blockIdx.x == 0) {
        for (int q = t; q < S; q += T) base_out[q] = s_base[q];
        if (t == 0) base_out[S] = (int32_t)n;
    }
    const uint64_t below = ss_lanes_below(lane);
    uint16_t* wc = s_wc + w * S;
    uint32_t rank[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const bool valid = at0 + r * 64 < cnt;
        const uint64_t peers = ss_peers(b[r], valid, bits);
        // the wave's keys of this bucket before this round, then in it
        const int run = valid ? wc[b[r]] : 0;
        rank[r] = (uint32_t)(run + __popcll(peers & below));
        __builtin_amdgcn_wave_barrier();
        if (valid && (peers & below) == 0) wc[b[r]] = (uint16_t)(run + __popcll(peers));
        __builtin_amdgcn_wave_barrier();
    }
    __syncthreads();
    const int32_t* row = table + (int64_t)blockIdx.x * S;
    for (int q = t; q < S; q += T) {
        int run = 0;
        for (int v = 0; v < NW; ++v) {
            const int c = s_wc[v * S + q];
            s_wc[v * S + q] = (uint16_t)run;
            run += c;
        }
        s_loc[q] = run;
        s_base[q] += row[q];
    }
    __syncthreads();
    ss_lds_scan<T>(s_loc, S, s_w);
#pragma unroll
    for (int r = 0; r < R; ++r) {
        if (at0 + r * 64 < cnt) {
            const int p = s_loc[b[r]] + wc[b[r]] + (int)rank[r];
            s_key[p] = k[r];
            s_at[p] = (uint16_t)(at0 + r * 64);
            s_bk[p] = (uint16_t)b[r];
        }
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int p = r * T + t;
        if (p < cnt) {
            const int q = s_bk[p];
            const int64_t dst = (int64_t)s_base[q] + (p - s_loc[q]);
            kout[dst] = s_key[p];
            vout[dst] = (int32_t)(tile0 + s_at[p]);
        }
    }
}

// LDS of the sort of one bucket. A word holds the digits sorted at first (up to
// 40 bits) above the key's place in the bucket.
constexpr int kSsPos = 13;   // bits of the place
struct SsLds {
    uint64_t word[kSsCap];
    uint16_t wc[kSsT / 64][256];
    int w4[kSsT / 64];
    int fix;
    unsigned long long diff;
};
static_assert((1 << kSsPos) >= kSsCap, "a place fits its bits");

// One digit pass over the len words held by the workgroup (word 64 r + lane of
// wave w's 64 * rounds): offsets per wave and digit by wave-private counting,
// the sorted order through LDS.
__device__ inline void ss_local_pass(SsLds& L, uint64_t (&k)[kSsR], int rounds, int len, int shift) {
    const int t = threadIdx.x, lane = t & 63, w = t >> 6;
    const uint64_t below = ss_lanes_below(lane);
    // (two counters a store; the type keeps their loads behind it)
    typedef uint32_t __attribute__((may_alias)) pair_of_counts;
    for (int q = lane; q < 128; q += 64) reinterpret_cast<pair_of_counts*>(L.wc[w])[q] = 0u;
    __builtin_amdgcn_wave_barrier();
    int rank[kSsR];
#pragma unroll
    for (int r = 0; r < kSsR; ++r) {
        if (r < rounds) {
            const bool valid = w * (64 * rounds) + r * 64 + lane < len;
            const unsigned d = (unsigned)(k[r] >> shift) & 255u;
            uint64_t peers = __ballot(valid);
#pragma unroll
            for (int b = 0; b < 8; ++b) {
                const bool on = (d >> b) & 1u;
                const uint64_t m = __ballot(on);
                peers &= on ? m : ~m;
            }
            const int run = valid ? L.wc[w][d] : 0;
            rank[r] = run + __popcll(peers & below);
            __builtin_amdgcn_wave_barrier();
            if (valid && (peers & below) == 0) L.wc[w][d] = (uint16_t)(run + __popcll(peers));
            __builtin_amdgcn_wave_barrier();
        }
    }
    __syncthreads();
    // Offsets: the counts in the order (digit, wave) are scanned as one array of
    // 256 x 16, four consecutive ones a thread.
    {
        const int d = t >> 2, q = (t & 3) * 4;
        int c[4], sum = 0;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            c[u] = L.wc[q + u][d];
            sum += c[u];
        }
        const int inc = wave_incl_scan(sum, lane);
        if (lane == 63) L.w4[w] = inc;
        __syncthreads();
        int run = inc - sum;
        for (int v = 0; v < w; ++v) run += L.w4[v];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            L.wc[q + u][d] = (uint16_t)run;
            run += c[u];
        }
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < kSsR; ++r)
        if (r < rounds && w * (64 * rounds) + r * 64 + lane < len)
            L.word[L.wc[w][(unsigned)(k[r] >> shift) & 255u] + rank[r]] = k[r];
    __syncthreads();
#pragma unroll
    for (int r = 0; r < kSsR; ++r) {
        const int i = w * (64 * rounds) + r * 64 + lane;
        if (r < rounds && i < len) k[r] = L.word[i];
    }
    // (the next pass writes L.word only after its own barriers)
}
static_assert(kSsT == 1024, "four counts a thread");

// LSD passes of the workgroup over the len pairs in (ka, va), by way of (kb,
// vb) in global memory, the result in (kb, vb): a bucket beyond kSsCap, or one
// with many keys alike in the digits sorted at first. diff: bits in which its
// keys differ.
__device__ inline void ss_global_sort(SsLds& L, uint64_t* ka, int32_t* va, uint64_t* kb, int32_t* vb, int64_t len,
                                      unsigned long long diff) {
    const int t = threadIdx.x, lane = t & 63, w = t >> 6;
    constexpr int NW = kSsT / 64;
    uint64_t *ki = ka, *ko = kb;
    int32_t *vi = va, *vo = vb;
    int* off = reinterpret_cast<int*>(L.word);             // [256] running offset of each digit
    int* dst0 = off + 256;                                 // [NW][256]
    for (int shift = 0; shift < 64; shift += 8) {
        if (((diff >> shift) & 255ull) == 0) continue;   // workgroup-uniform
        __syncthreads();
        if (t < 256) off[t] = 0;
        __syncthreads();
        for (int64_t i = t; i < len; i += kSsT) atomicAdd(&off[(unsigned)(ki[i] >> shift) & 255u], 1);
        __syncthreads();
        if (t == 0) {
            int run = 0;
            for (int d = 0; d < 256; ++d) {
                const int c = off[d];
                off[d] = run;
                run += c;
            }
        }
        for (int64_t c0 = 0; c0 < len; c0 += kSsT) {
            for (int q = lane; q < 256; q += 64) L.wc[w][q] = 0;
            __syncthreads();
            const int64_t i = c0 + t;
            const bool valid = i < len;
            const uint64_t k = valid ? ki[i] : 0ull;
            const int32_t v = valid ? vi[i] : 0;
            const unsigned d = (unsigned)(k >> shift) & 255u;
            const uint64_t peers = ss_peers(d, valid, 8);
            const int r = __popcll(peers & ss_lanes_below(lane));
            if (valid && r == 0) L.wc[w][d] = (uint16_t)__popcll(peers);
            __syncthreads();
            if (t < 256) {
                int run = off[t];
                for (int q = 0; q < NW; ++q) {
                    dst0[q * 256 + t] = run;
                    run += L.wc[q][t];
                }
                off[t] = run;
            }
            __syncthreads();
            if (valid) {
                const int dst = dst0[w * 256 + d] + r;
                ko[dst] = k;
                vo[dst] = v;
            }
            __syncthreads();
        }
        uint64_t* tk = ki; ki = ko; ko = tk;
        int32_t* tv = vi; vi = vo; vo = tv;
    }
    __syncthreads();
    if (ki != kb)
        for (int64_t i = t; i < len; i += kSsT) {
            kb[i] = ki[i];
            vb[i] = vi[i];
        }
    __syncthreads();
}

// Sort of one bucket per workgroup, from (kin, vin) to (kout, vout), two
// different pairs; iota: the values in vin are the positions, and are written
// there by this kernel if it needs them. The keys of a bucket lie close
// together, so the 32 bits below their common prefix (40 where a bucket
// straddles a boundary near the top of the key) tell nearly all of them apart:
// those digits are sorted in LDS, then the runs that agree in them, by insertion
// on the whole keys, unless every run is in order as it is (equal keys are). A run
// beyond kSsRun then sends the bucket to ss_global_sort (1000000 keys, each 100
// times: 201 us in this kernel when equal keys did too, 65 now).
constexpr int kSsRun = 16;
constexpr int kSsLong = 1, kSsUnsorted = 2;   // SsLds::fix
__global__ __launch_bounds__(kSsT) void k_ss_local(uint64_t* __restrict__ kin_all, int32_t* __restrict__ vin_all,
                                                   const int32_t* __restrict__ base, int64_t n, int iota,
                                                   uint64_t* __restrict__ kout_all, int32_t* __restrict__ vout_all) {
    __shared__ SsLds L;
    const int t = threadIdx.x, lane = t & 63, w = t >> 6;
    const int64_t b0 = base ? base[blockIdx.x] : 0, b1 = base ? base[blockIdx.x + 1] : n;
    const int64_t len64 = b1 - b0;
    if (len64 <= 0) return;   // workgroup-uniform
    uint64_t* kin = kin_all + b0;
    int32_t* vin = vin_all + b0;
    uint64_t* kout = kout_all + b0;
    int32_t* vout = vout_all + b0;
    if (t == 0) {
        L.diff = 0ull;
        L.fix = 0;
    }
    const uint64_t k0 = kin[0];
    unsigned long long x = 0;
    if (len64 > kSsCap) {   // (only behind a partition: the values are in vin)
        for (int64_t i = t; i < len64; i += kSsT) x |= kin[i] ^ k0;
        __syncthreads();
        if (x) atomicOr(&L.diff, x);
        __syncthreads();
        const unsigned long long d = L.diff;
        __syncthreads();
        ss_global_sort(L, kin, vin, kout, vout, len64, d);
        return;
    }
    const int len = (int)len64;
    const int rounds = (len + kSsT - 1) / kSsT;
    uint64_t k[kSsR];
#pragma unroll
    for (int r = 0; r < kSsR; ++r) {
        const int i = w * (64 * rounds) + r * 64 + lane;
        k[r] = r < rounds && i < len ? kin[i] : k0;
        x |= k[r] ^ k0;
    }
    for (int o = 32; o > 0; o >>= 1) x |= __shfl_xor(x, o, 64);
    __syncthreads();
    if (lane == 0 && x) atomicOr(&L.diff, x);
    __syncthreads();
    const unsigned long long diff = L.diff;
    const int hb = diff ? 63 - __clzll(diff) : -1;
    const int low = hb >= 54 ? hb - 39 : (hb >= 32 ? hb - 31 : 0);   // lowest bit sorted at first
    const uint64_t mask = hb < 0 ? 0ull : ~0ull >> (63 - (hb - low));
#pragma unroll
    for (int r = 0; r < kSsR; ++r)
        k[r] = ((k[r] >> low) & mask) << kSsPos | (uint64_t)(w * (64 * rounds) + r * 64 + lane);
    for (int shift = low; shift <= hb; shift += 8)
        if ((diff >> shift) & 255ull) ss_local_pass(L, k, rounds, len, shift - low + kSsPos);
    if (low > 0 && (diff & ((1ull << low) - 1ull))) {   // workgroup-uniform
        // (L.word holds the order of the last pass)
        constexpr uint64_t kPos = (1ull << kSsPos) - 1ull;
        bool head[kSsR];
#pragma unroll
        for (int r = 0; r < kSsR; ++r) {
            const int i = w * (64 * rounds) + r * 64 + lane;
            head[r] = false;
            if (r < rounds && i + 1 < len) {
                const uint64_t p = k[r] >> kSsPos, next = L.word[i + 1];
                if (next >> kSsPos == p) {
                    int fix = kin[next & kPos] < kin[k[r] & kPos] ? kSsUnsorted : 0;
                    if (!(i > 0 && L.word[i - 1] >> kSsPos == p)) {
                        int e = i + 2;   // the run [i, e)
                        while (e < len && e - i <= kSsRun && L.word[e] >> kSsPos == p) ++e;
                        head[r] = true;
                        fix |= e - i > kSsRun ? kSsLong : 0;
                    }
                    if (fix) atomicOr(&L.fix, fix);
                }
            }
        }
        __syncthreads();
        const int fix = L.fix;
        __syncthreads();
        if (fix == (kSsLong | kSsUnsorted)) {
            if (iota)
                for (int i = t; i < len; i += kSsT) vin[i] = (int32_t)(b0 + i);
            ss_global_sort(L, kin, vin, kout, vout, len, diff);
            return;
        }
        if (fix == kSsUnsorted) {
#pragma unroll
            for (int r = 0; r < kSsR; ++r) {
                if (head[r]) {
                    const int i = w * (64 * rounds) + r * 64 + lane;
                    const uint64_t p = k[r] >> kSsPos;
                    for (int a = i + 1; a < len && L.word[a] >> kSsPos == p; ++a) {
                        const uint64_t wa = L.word[a], ka = kin[wa & kPos];
                        int b = a;
                        for (; b > i && kin[L.word[b - 1] & kPos] > ka; --b) L.word[b] = L.word[b - 1];
                        L.word[b] = wa;
                    }
                }
            }
            __syncthreads();
#pragma unroll
            for (int r = 0; r < kSsR; ++r) {
                const int i = w * (64 * rounds) + r * 64 + lane;
                if (r < rounds && i < len) k[r] = L.word[i];
            }
        }
    }
#pragma unroll
    for (int r = 0; r < kSsR; ++r) {
        const int i = w * (64 * rounds) + r * 64 + lane;
        if (r < rounds && i < len) {
            const int at = (int)(k[r] & ((1ull << kSsPos) - 1ull));
            kout[i] = kin[at];
            vout[i] = iota ? (int32_t)(b0 + at) : vin[at];
        }
    }
}

}  // namespace

int64_t scan_tmp_need(int64_t n) { return (n + SCAN_TILE - 1) / SCAN_TILE + 2; }

void exclusive_scan_i32_to_i64(const int32_t* in, int64_t* out, int64_t n, int64_t* tmp,
                               hipStream_t s) {
    scan_impl<int32_t, int64_t>(in, out, n, tmp, s);
}

int64_t radix_hist_need(int64_t n) {
    const int64_t nblk = (n + RS_TILE - 1) / RS_TILE;
    return nblk * RS_MAX_BINS + 1;
}

// 8-bit digits (9-bit digits would save a pass on 63-bit keys, 7 instead of 8,
// but cost more per pass than that pass at 2^20)
constexpr int RS_BITS = 8;

// Stable LSD radix sort of the n keys on bits [0, nbits), vals[k] = the original
// position of the k-th; the alternate pair is scratch, in which an odd number
// of passes ends.
static void radix_sort_iota(uint64_t* keys, int32_t* vals, uint64_t* keys_alt, int32_t* vals_alt, int64_t n,
                            int nbits, int64_t* hist, int64_t* scan_tmp, hipStream_t s) {
    const int64_t nblk = (n + RS_TILE - 1) / RS_TILE;
    const int passes = (nbits + RS_BITS - 1) / RS_BITS;
    uint64_t* ki = keys;
    int32_t* vi = vals;
    uint64_t* ko = keys_alt;
    int32_t* vo = vals_alt;
    for (int p = 0; p < passes; ++p) {
        const int shift = RS_BITS * p;
        hipLaunchKernelGGL(k_rs_hist<RS_BITS>, dim3(nblk), dim3(RS_T), 0, s, (const uint64_t*)ki, n, shift, hist, nblk);
        scan_impl<int64_t, int64_t>(hist, hist, nblk << RS_BITS, scan_tmp, s);
        hipLaunchKernelGGL(k_rs_scatter<RS_BITS>, dim3(nblk), dim3(RS_T), 0, s, (const uint64_t*)ki,
                           (const int32_t*)vi, ko, vo, n, shift, (const int64_t*)hist, nblk, (int)(p == 0));
        uint64_t* tk = ki; ki = ko; ko = tk;
        int32_t* tv = vi; vi = vo; vo = tv;
    }
    if (ki != keys)
        hipLaunchKernelGGL(k_copy_pairs, dim3(4096), dim3(256), 0, s, (const uint64_t*)ki, (const int32_t*)vi, keys,
                           vals, n);
}

// Scratch of sort_iota in int32 words for any array of up to n keys: samples,
// splitters (key and index), bucket totals and offsets, and the tile table (at
// most 512 tiles up to 2^20 keys, tiles of 4096 keys beyond).
int64_t sort_scratch_need(int64_t n) {
    if (n > kSsMaxN) n = kSsMaxN;
    const int64_t S = ss_buckets(n), tiles = (n + 4095) / 4096;
    return (2 * kSsOver + 5) * S + 16 + S * (tiles < 512 ? 512 : tiles);
}

struct SsBufs {
    const uint64_t* keys;
    uint64_t* kalt;
    int32_t* valt;
    uint16_t* bucket;
    const uint64_t* sp_key;
    const int32_t* sp_idx;
    int32_t *total, *base, *table;
};

template <int T, int R>
static void ss_partition(const SsBufs& q, int64_t n, int S, hipStream_t s) {
    const int nt = (int)((n + T * R - 1) / (T * R));
    int bits = 0;
    while ((1 << bits) < S) ++bits;
    hipLaunchKernelGGL((k_ss_count<T, R>), dim3(nt), dim3(T), (size_t)S * 12, s, q.keys, n, S, q.sp_key, q.sp_idx,
                       q.bucket, q.table);
    hipLaunchKernelGGL(k_ss_scan, dim3((S + 15) / 16), dim3(1024), 0, s, q.table, nt, S, q.total);
    hipLaunchKernelGGL((k_ss_scatter<T, R>), dim3(nt), dim3(T),
                       (size_t)T * R * 12 + (size_t)S * (8 + 2 * (T / 64)), s, q.keys, n, S, bits,
                       (const uint16_t*)q.bucket, (const int32_t*)q.table, (const int32_t*)q.total, q.base, q.kalt,
                       q.valt);
}

bool sort_iota_in_alt(int64_t n) { return n <= kSsCap; }

void sort_iota(uint64_t* keys, int32_t* vals, uint64_t* keys_alt, int32_t* vals_alt, int64_t n, int nbits,
               int64_t* hist, int64_t* scan_tmp, int32_t* scratch, hipStream_t s) {
    if (n <= 0) return;
    if (n > kSsMaxN) {
        radix_sort_iota(keys, vals, keys_alt, vals_alt, n, nbits, hist, scan_tmp, s);
        return;
    }
    if (n <= kSsCap) {
        // one workgroup, between the two pairs: the keys were put in the alternate
        hipLaunchKernelGGL(k_ss_local, dim3(1), dim3(kSsT), 0, s, keys_alt, vals_alt, (const int32_t*)nullptr, n, 1,
                           keys, vals);
        return;
    }
    const int S = ss_buckets(n), m = S * kSsOver;
    uint64_t* sample = reinterpret_cast<uint64_t*>(scratch);   // [m]
    uint64_t* sp_key = sample + m;                             // [S]
    int32_t* sp_idx = reinterpret_cast<int32_t*>(sp_key + S);  // [S]
    SsBufs q;
    q.keys = keys;
    q.kalt = keys_alt;
    q.valt = vals_alt;
    q.bucket = reinterpret_cast<uint16_t*>(vals);   // free until the buckets are sorted into it
    q.sp_key = sp_key;
    q.sp_idx = sp_idx;
    q.total = sp_idx + S;        // [S]
    q.base = q.total + S;        // [S + 1]
    q.table = q.base + S + 8;
    hipLaunchKernelGGL(k_ss_gather, dim3((m + 255) / 256), dim3(256), 0, s, (const uint64_t*)keys, n, m, sample);
    hipLaunchKernelGGL(k_ss_split, dim3(m / 32), dim3(1024), 0, s, (const uint64_t*)sample, n, m, sp_key, sp_idx);
    // Tiles: 512 keys up to 2^18 keys (to occupy the chip), then 2048, then 4096. A tile
    // takes 12 bytes of LDS a key and each bucket 8 and 2 a wave: 60 KB for 4096 keys in
    // eight waves and 512 buckets, four waves beyond (64 KB for 1024 buckets, 80 for 2048
    // of the 160 a CU has).
    if (n <= (1 << 18)) ss_partition<256, 2>(q, n, S, s);
    else if (n <= (1 << 19)) ss_partition<512, 4>(q, n, S, s);
    else if (S <= 512) ss_partition<512, 8>(q, n, S, s);
    else ss_partition<256, 16>(q, n, S, s);
    hipLaunchKernelGGL(k_ss_local, dim3(S), dim3(kSsT), 0, s, keys_alt, vals_alt, (const int32_t*)q.base, n, 0, keys, vals);
}

}  // namespace pbh
