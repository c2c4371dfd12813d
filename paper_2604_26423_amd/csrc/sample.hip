// Measurement shots (arXiv:2604.26423, Sec. II-B: repeated preparation and
// measurement), reproducible bit for bit:
//   P(x) = re^2 + im^2 in FP64 with no fused multiply-add, q(x) = floor(P 2^62),
//   F(x) = sum_{y<=x} q(y) (uint64), T = F(2^n - 1);
//   shot s: r = word 0 of Philox4x64-10(counter (s,0,0,0), key (seed,0)),
//   u = floor(r T / 2^64), x_s = min { x : F(x) > u }.
// The CDF is never stored.  Pass A writes exclusive prefix sums at three
// levels: 64-amplitude sub-blocks within 8192-amplitude blocks, blocks within
// 2^26-amplitude chunks, and chunks; integer sums make the result independent
// of summation order.  Each shot then descends the three levels and scans 64
// amplitudes.  Small states (n < 13) use a full CDF in LDS.
//
// A sum of 2^64 or more (a norm of 4 or more) cannot be sampled.  Every sum on
// the way to T is checked where it is made: s = a + b wrapped if s < b, and in
// an inclusive scan the first element to wrap is smaller than its own addend.
// No partial sum exceeds T, so a wrap anywhere means T wraps, and T wraps only
// if some partial sum does.  flag[0] = 1: T = 0; flag[1] = 2: T >= 2^64.
#include <algorithm>

#include "device.h"

namespace qs {

namespace {

constexpr int kBlockBits = 13;   // amplitudes per block: 8192
constexpr int kSubBits = 6;      // amplitudes per sub-block: 64
constexpr int kChunkBits = 26;   // amplitudes per chunk
constexpr int kSubPerBlock = 1 << (kBlockBits - kSubBits);            // 128
constexpr int kBlkPerChunk = 1 << (kChunkBits - kBlockBits);          // 8192

// Philox4x64-10 (Salmon, Moraes, Dror, Shaw, SC'11), words 0 and 1 of the
// output for counter (c0, 0, 0, 0) and key (k0, 0).
__device__ __forceinline__ void philox_words01(uint64_t c0, uint64_t k0, uint64_t &w0, uint64_t &w1)
{
    const uint64_t M0 = 0xD2E7470EE14C6C93ULL, M1 = 0xCA5A826395121157ULL;
    const uint64_t W0 = 0x9E3779B97F4A7C15ULL, W1 = 0xBB67AE8584CAA73BULL;
    uint64_t x0 = c0, x1 = 0, x2 = 0, x3 = 0, ka = k0, kb = 0;
#pragma unroll
    for (int round = 0; round < 10; ++round) {
        if (round > 0) {
            ka += W0;
            kb += W1;
        }
        const uint64_t h0 = __umul64hi(M0, x0), l0 = M0 * x0;
        const uint64_t h1 = __umul64hi(M1, x2), l1 = M1 * x2;
        const uint64_t y0 = h1 ^ x1 ^ ka, y2 = h0 ^ x3 ^ kb;
        x0 = y0;
        x1 = l1;
        x2 = y2;
        x3 = l0;
    }
    w0 = x0;
    w1 = x1;
}

__device__ __forceinline__ uint64_t philox_word0(uint64_t c0, uint64_t k0)
{
    uint64_t w0, w1;
    philox_words01(c0, k0, w0, w1);
    return w0;
}

// Inclusive scan across the 64 lanes of a wave.
__device__ __forceinline__ uint64_t wave_scan_u64(uint64_t v, int lane)
{
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const uint64_t t = __shfl_up(v, off, 64);
        if (lane >= off) v += t;
    }
    return v;
}

// Two consecutive amplitudes (an even index): one 16-byte load for complex64.
// Pass A reads each amplitude once: nontemporal (streaming) loads, which
// measured pass A 10% faster at n = 32 in complex64 (6.25 -> 5.65 ms).
template <typename V> struct AmpPair;
template <> struct AmpPair<float2> {
    static __device__ __forceinline__ void load(const float2 *p, float2 &a, float2 &b)
    {
        typedef float f4 __attribute__((ext_vector_type(4)));
        const f4 t = __builtin_nontemporal_load(reinterpret_cast<const f4 *>(p));
        a = float2{t.x, t.y};
        b = float2{t.z, t.w};
    }
};
template <> struct AmpPair<double2> {
    static __device__ __forceinline__ void load(const double2 *p, double2 &a, double2 &b)
    {
        a = load_nt(p);
        b = load_nt(p + 1);
    }
};

// Pass A: one workgroup per block of 8192 amplitudes.  Thread t reads the
// pairs (i 512 + 2 t, +1), i = 0..15, all issued before any arithmetic; the 32
// lanes of half a wave then hold one 64-amplitude sub-block and sum it with
// five shuffles.
template <typename V>
__global__ void __launch_bounds__(256) sample_blocks_kernel(const V *psi, uint64_t *sub, uint64_t *blk,
                                                            int32_t *flag)
{
    constexpr int NL = (1 << kBlockBits) / 512;  // pairs per thread
    int32_t over = 0;
    __shared__ uint64_t ssum[kSubPerBlock];
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    const int64_t b = blockIdx.x;
    const V *blkp = psi + (b << kBlockBits);
    // layout of the block's entries (internal.h): the fold moves bits 4..12 only,
    // so a pair at an even index stays a pair
    const int fb = (int)(swz_fold(b) << kSwzDst);
    V a[NL], c[NL];
#pragma unroll
    for (int i = 0; i < NL; ++i) AmpPair<V>::load(blkp + ((i * 512 + 2 * tid) ^ fb), a[i], c[i]);
#pragma unroll
    for (int i = 0; i < NL; ++i) {
        const uint64_t q1 = qval_of(c[i], &over);
        uint64_t q = qval_of(a[i], &over) + q1;
        over |= q < q1;
#pragma unroll
        for (int off = 16; off >= 1; off >>= 1) {
            const uint64_t t = __shfl_xor(q, off, 64);
            q += t;
            over |= q < t;
        }
        if ((lane & 31) == 0) ssum[i * 8 + 2 * wave + (lane >> 5)] = q;
    }
    __syncthreads();
    if (wave == 0) {
        const uint64_t a0 = ssum[2 * lane], a1 = ssum[2 * lane + 1];
        const uint64_t incl = wave_scan_u64(a0 + a1, lane);
        over |= a0 + a1 < a1 || incl < a0 + a1;
        const uint64_t excl = incl - (a0 + a1);
        sub[b * kSubPerBlock + 2 * lane] = excl;
        sub[b * kSubPerBlock + 2 * lane + 1] = excl + a0;
        if (lane == 63) blk[b] = incl;
    }
    if (over) flag[1] = 2;
}

// Exclusive prefix over the workgroup of one value per thread (1024 threads at
// most); *total: the sum; over: set where a sum wraps.  red: 16 words of LDS.
__device__ __forceinline__ uint64_t block_scan_u64(uint64_t v, uint64_t *red, int tid, uint64_t *total, int32_t &over)
{
    const int wave = tid >> 6, lane = tid & 63, nw = blockDim.x >> 6;
    const uint64_t incl = wave_scan_u64(v, lane);
    if (lane == 63) red[wave] = incl;
    __syncthreads();
    uint64_t before = 0, all = 0;
    for (int w = 0; w < nw; ++w) {
        before += w < wave ? red[w] : 0;
        all += red[w];
    }
    over |= incl < v || before + incl < incl;
    *total = all;
    return before + incl - v;
}

// In-place exclusive scan of block sums within each chunk; chunk sums out.
// One workgroup per chunk: eight consecutive entries per thread, all loaded
// before any is summed (a serial pass of one thread over 256 partial sums took
// 20 us at n = 27, this one 5).
constexpr int kScanThreads = 1024;
__global__ void __launch_bounds__(kScanThreads) scan_blocks_kernel(uint64_t *blk, int64_t nblk, uint64_t *chunk,
                                                                   int32_t *flag)
{
    __shared__ uint64_t red[kScanThreads / 64];
    constexpr int per = kBlkPerChunk / kScanThreads;
    const int tid = threadIdx.x;
    const int64_t lo = (int64_t)blockIdx.x * kBlkPerChunk + (int64_t)tid * per;
    uint64_t v[per], loc = 0, total;
    int32_t over = 0;
#pragma unroll
    for (int k = 0; k < per; ++k) v[k] = lo + k < nblk ? blk[lo + k] : 0;
#pragma unroll
    for (int k = 0; k < per; ++k) {
        loc += v[k];
        over |= loc < v[k];
    }
    uint64_t acc = block_scan_u64(loc, red, tid, &total, over);
    if (over) flag[1] = 2;
#pragma unroll
    for (int k = 0; k < per; ++k) {
        if (lo + k < nblk) blk[lo + k] = acc;
        acc += v[k];
    }
    if (tid == 0) chunk[blockIdx.x] = total;
}

constexpr int kShotThreads = 256;
constexpr int kMaxChunks = 256;  // 2^34 stored amplitudes

// Exclusive prefixes of the chunk sums into cs, by every workgroup, and the
// total; the first workgroup reports a zero total or a sum that wraps.
__device__ __forceinline__ uint64_t scan_chunks(const uint64_t *chunk, int64_t nchunk, uint64_t *cs, uint64_t *red,
                                                int tid, int32_t *flag)
{
    uint64_t T;
    int32_t over = 0;
    cs[tid] = block_scan_u64(tid < nchunk ? chunk[tid] : 0, red, tid, &T, over);
    if (blockIdx.x == 0) {
        if (over) flag[1] = 2;
        if (T == 0 && tid == 0) flag[0] = 1;
    }
    __syncthreads();
    return T;
}

// The basis state of stored index x; r1: word 1 of the shot's Philox output.
// Complement-symmetric layout (sym_n qubits): z -> y(z) (suffix XOR), or its
// complement.
__device__ __forceinline__ uint64_t shot_state(int64_t x, uint64_t r1, int sym_n)
{
    uint64_t xo = (uint64_t)x;
    if (sym_n) {
#pragma unroll
        for (int sh = 1; sh < 64; sh <<= 1) xo ^= xo >> sh;
        if (r1 >> 63) xo ^= (~0ull) >> (64 - sym_n);
    }
    return xo;
}

// Lanes that work on one shot together, and the shots that such a group draws
// one after the other: one, or kShotRounds from kManyShots on.
constexpr int kShotLanes = 16;
constexpr int64_t kManyShots = 1 << 19;
constexpr int kShotRounds = 16;

// Number of leading lanes of the shot's group for which yes holds.
__device__ __forceinline__ int group_count(bool yes)
{
    const uint64_t m = __ballot(yes) >> (threadIdx.x & 63 & ~(kShotLanes - 1));
    return __builtin_ctzll(~(m & ((1ull << kShotLanes) - 1ull)));
}

// Largest i in [0, len) with a[i] <= u (a nondecreasing, a[0] = 0 <= u, len a
// power of two), kShotLanes probes at a time.  The first probe of every step
// holds, whatever a is, so the result is in range also where sums wrapped.
__device__ __forceinline__ int64_t group_last_le(const uint64_t *a, int64_t len, uint64_t u, int g)
{
    int64_t base = 0;
    for (int64_t span = len; span > 1;) {
        const int64_t step = span > kShotLanes ? span / kShotLanes : 1;
        const bool in = g * step < span;
        const int c = group_count(in && a[in ? base + g * step : base] <= u);
        base += (int64_t)(c - 1) * step;
        span = step;
    }
    return base;
}

// A shot is a chain of dependent reads.  Sixteen lanes share it: four probes
// find the block of 8192 in a chunk, two the sub-block, and the 64 amplitudes
// are read at once and scanned across the lanes (one lane per shot took 20
// binary-search steps and a serial walk over the amplitudes: 24 us for 10,000
// shots at n = 27, 10 us now).  With shots enough to fill the chip the latency is
// hidden and the work per shot counts: a group then draws 16 shots in turn, so
// that the chunk scan is shared by 256 shots and a wave's lanes evaluate 64
// Philox outputs at once, or every lane draws a shot of its own (shot_lanes).
template <typename V>
__global__ void __launch_bounds__(kShotThreads) sample_shots_kernel(const V *psi, const uint64_t *sub,
                                                                    const uint64_t *blk, const uint64_t *chunk,
                                                                    int64_t nchunk, int64_t nblk, uint64_t seed,
                                                                    int64_t shots, int rounds, uint64_t *out,
                                                                    int32_t *flag, int sym_n)
{
    __shared__ uint64_t cs[kMaxChunks];
    __shared__ uint64_t red[kShotThreads / 64];
    constexpr int kGroups = 64 / kShotLanes;  // of a wave
    const int tid = threadIdx.x, lane = tid & 63, g = lane & (kShotLanes - 1);
    const uint64_t T = scan_chunks(chunk, nchunk, cs, red, tid, flag);
    // lane i evaluates the draw of the wave's shot i (i < kGroups * rounds <= 64)
    const int64_t s0 = ((int64_t)blockIdx.x * (kShotThreads / 64) + (tid >> 6)) * (kGroups * rounds);
    uint64_t w0, w1;
    philox_words01((uint64_t)(s0 + lane), seed, w0, w1);
    for (int i = 0; i < rounds; ++i) {
        const int at_lane = i * kGroups + lane / kShotLanes;
        const int64_t s = s0 + at_lane;
        const uint64_t r0 = __shfl(w0, at_lane, 64), r1 = __shfl(w1, at_lane, 64);
        if (s >= shots) return;  // a whole group, and its later shots
        uint64_t u = __umul64hi(r0, T);
        const int64_t c = group_last_le(cs, nchunk, u, g);
        u -= cs[c];
        const int64_t b0 = c * kBlkPerChunk;
        const int64_t blen = (nblk - b0) < kBlkPerChunk ? (nblk - b0) : kBlkPerChunk;
        const int64_t b = b0 + group_last_le(blk + b0, blen, u, g);
        u -= blk[b];
        const int64_t j = group_last_le(sub + b * kSubPerBlock, kSubPerBlock, u, g);
        u -= sub[b * kSubPerBlock + j];
        const int64_t x0 = (b << kBlockBits) + (j << kSubBits);
        const int64_t fb = swz_fold(b) << kSwzDst;
        constexpr int per = 64 / kShotLanes;  // consecutive amplitudes of a lane (the fold keeps runs of 16)
        const V *p = psi + ((x0 + g * per) ^ fb);
        uint64_t q[per], loc = 0;
#pragma unroll
        for (int t = 0; t < per; ++t) q[t] = qval_of(p[t], flag + 1);
#pragma unroll
        for (int t = 0; t < per; ++t) loc += q[t];
        uint64_t acc = loc;
#pragma unroll
        for (int off = 1; off < kShotLanes; off <<= 1) {
            const uint64_t t = __shfl_up(acc, off, kShotLanes);
            if (g >= off) acc += t;
        }
        // the first lane whose inclusive sum exceeds u holds the shot; none
        // (only if the state changed meanwhile): the last amplitude
        const int at = group_count(!(acc > u));
        if (g == (at < kShotLanes ? at : kShotLanes - 1)) {
            acc -= loc;
            int64_t x = x0 + 63;
            bool found = false;
#pragma unroll
            for (int t = 0; t < per; ++t) {
                acc += q[t];
                if (!found && acc > u) {
                    x = x0 + g * per + t;
                    found = true;
                }
            }
            out[s] = shot_state(x, r1, sym_n);
        }
    }
}

// Largest i in [0, len) with a[i] <= u (a nondecreasing, a[0] = 0 <= u).
__device__ __forceinline__ int64_t last_le(const uint64_t *a, int64_t len, uint64_t u)
{
    int64_t lo = 0, hi = len - 1;
    while (lo < hi) {
        const int64_t mid = lo + (hi - lo + 1) / 2;
        if (a[mid] <= u) lo = mid;
        else hi = mid - 1;
    }
    return lo;
}

// One lane per shot: a long chain (20 probes and a walk over the amplitudes),
// but few instructions, for many shots (shot_lanes).
template <typename V>
__global__ void __launch_bounds__(kShotThreads) sample_lanes_kernel(const V *psi, const uint64_t *sub,
                                                                    const uint64_t *blk, const uint64_t *chunk,
                                                                    int64_t nchunk, int64_t nblk, uint64_t seed,
                                                                    int64_t shots, uint64_t *out, int32_t *flag,
                                                                    int sym_n)
{
    __shared__ uint64_t cs[kMaxChunks];
    __shared__ uint64_t red[kShotThreads / 64];
    const int tid = threadIdx.x;
    const uint64_t T = scan_chunks(chunk, nchunk, cs, red, tid, flag);
    const int64_t s = (int64_t)blockIdx.x * kShotThreads + tid;
    if (s >= shots) return;
    uint64_t r0, r1;
    philox_words01((uint64_t)s, seed, r0, r1);
    uint64_t u = __umul64hi(r0, T);
    const int64_t c = last_le(cs, nchunk, u);
    u -= cs[c];
    const int64_t b0 = c * kBlkPerChunk;
    const int64_t blen = (nblk - b0) < kBlkPerChunk ? (nblk - b0) : kBlkPerChunk;
    const int64_t b = b0 + last_le(blk + b0, blen, u);
    u -= blk[b];
    const int64_t j = last_le(sub + b * kSubPerBlock, kSubPerBlock, u);
    u -= sub[b * kSubPerBlock + j];
    const int64_t x0 = (b << kBlockBits) + (j << kSubBits);
    const int64_t fb = swz_fold(b) << kSwzDst;
    uint64_t acc = 0;
    int64_t x = x0 + 63;
    for (int t = 0; t < 64; ++t) {
        acc += qval_of(psi[(x0 + t) ^ fb], flag + 1);
        if (acc > u) {
            x = x0 + t;
            break;
        }
    }
    out[s] = shot_state(x, r1, sym_n);
}

// n < 13: every workgroup builds the whole CDF in LDS and draws kSmallShots
// shots, one per thread; kSmallGroups workgroups at most (more shots than
// that: several rounds each), so that a launch stays far below the 2^32 threads
// that the runtime accepts.
constexpr int kSmallShots = 1024;
constexpr int64_t kSmallGroups = 1 << 16;
template <typename V>
__global__ void __launch_bounds__(kSmallShots) sample_small_kernel(const V *psi, int n, uint64_t seed, int64_t shots,
                                                                   uint64_t *out, int32_t *flag)
{
    constexpr int per = (1 << (kBlockBits - 1)) / kSmallShots;
    __shared__ uint64_t F[1 << (kBlockBits - 1)];
    __shared__ uint64_t red[kSmallShots / 64];
    const int tid = threadIdx.x, dim = 1 << n;
    uint64_t q[per], loc = 0, T;
    int32_t over = 0;
#pragma unroll
    for (int k = 0; k < per; ++k) {
        const int x = tid * per + k;
        q[k] = x < dim ? qval_of(psi[x], &over) : 0;
        loc += q[k];
        over |= loc < q[k];
    }
    uint64_t acc = block_scan_u64(loc, red, tid, &T, over);
#pragma unroll
    for (int k = 0; k < per; ++k) {
        acc += q[k];
        F[tid * per + k] = acc;
    }
    if (blockIdx.x == 0) {
        if (over) flag[1] = 2;
        if (T == 0 && tid == 0) flag[0] = 1;
    }
    __syncthreads();
    for (int64_t s = (int64_t)blockIdx.x * kSmallShots + tid; s < shots; s += (int64_t)gridDim.x * kSmallShots) {
        const uint64_t u = __umul64hi(philox_word0((uint64_t)s, seed), T);
        int lo = 0, hi = dim - 1;  // first x with F[x] > u
        while (lo < hi) {
            const int mid = (lo + hi) / 2;
            if (F[mid] > u) hi = mid;
            else lo = mid + 1;
        }
        out[s] = (uint64_t)lo;
    }
}

}  // namespace

void sample_sizes(int n, int64_t *nsub, int64_t *nblk, int64_t *nchunk)
{
    if (n < kBlockBits) {
        *nsub = *nblk = 0;
        *nchunk = 0;
        return;
    }
    *nsub = (int64_t)1 << (n - kSubBits);
    *nblk = (int64_t)1 << (n - kBlockBits);
    *nchunk = n > kChunkBits ? (int64_t)1 << (n - kChunkBits) : 1;
}

hipError_t launch_sample(int prec, const void *psi, int n, const SampleBufs &b, uint64_t seed, int64_t shots,
                         uint64_t *out, hipStream_t st, int sym_n)
{
    // (also without shots: a workgroup reports a state that cannot be sampled)
    const auto groups = [&](int64_t per) { return dim3((unsigned)std::max<int64_t>(1, (shots + per - 1) / per)); };
    if (n < kBlockBits) {
        const dim3 g((unsigned)std::min<int64_t>(kSmallGroups, groups(kSmallShots).x));
        if (prec == 0)
            hipLaunchKernelGGL(sample_small_kernel<float2>, g, dim3(kSmallShots), 0, st, (const float2 *)psi, n, seed,
                               shots, out, b.flag);
        else
            hipLaunchKernelGGL(sample_small_kernel<double2>, g, dim3(kSmallShots), 0, st, (const double2 *)psi, n,
                               seed, shots, out, b.flag);
        return hipGetLastError();
    }
    int64_t nsub, nblk, nchunk;
    sample_sizes(n, &nsub, &nblk, &nchunk);
    if (prec == 0)
        hipLaunchKernelGGL(sample_blocks_kernel<float2>, dim3((unsigned)nblk), dim3(256), 0, st,
                           (const float2 *)psi, b.sub, b.blk, b.flag);
    else
        hipLaunchKernelGGL(sample_blocks_kernel<double2>, dim3((unsigned)nblk), dim3(256), 0, st,
                           (const double2 *)psi, b.sub, b.blk, b.flag);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    if (nchunk > kMaxChunks) return hipErrorInvalidValue;
    hipLaunchKernelGGL(scan_blocks_kernel, dim3((unsigned)nchunk), dim3(kScanThreads), 0, st, b.blk, nblk, b.chunk,
                       b.flag);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    if (shot_lanes(prec, n, shots)) {
        const dim3 g = groups(kShotThreads);
        if (prec == 0)
            hipLaunchKernelGGL(sample_lanes_kernel<float2>, g, dim3(kShotThreads), 0, st, (const float2 *)psi,
                               (const uint64_t *)b.sub, (const uint64_t *)b.blk, (const uint64_t *)b.chunk, nchunk,
                               nblk, seed, shots, out, b.flag, sym_n);
        else
            hipLaunchKernelGGL(sample_lanes_kernel<double2>, g, dim3(kShotThreads), 0, st, (const double2 *)psi,
                               (const uint64_t *)b.sub, (const uint64_t *)b.blk, (const uint64_t *)b.chunk, nchunk,
                               nblk, seed, shots, out, b.flag, sym_n);
        return hipGetLastError();
    }
    const int rounds = shots < kManyShots ? 1 : kShotRounds;
    const dim3 g = groups((int64_t)(kShotThreads / kShotLanes) * rounds);
    if (prec == 0)
        hipLaunchKernelGGL(sample_shots_kernel<float2>, g, dim3(kShotThreads), 0, st, (const float2 *)psi,
                           (const uint64_t *)b.sub, (const uint64_t *)b.blk, (const uint64_t *)b.chunk, nchunk, nblk,
                           seed, shots, rounds, out, b.flag, sym_n);
    else
        hipLaunchKernelGGL(sample_shots_kernel<double2>, g, dim3(kShotThreads), 0, st, (const double2 *)psi,
                           (const uint64_t *)b.sub, (const uint64_t *)b.blk, (const uint64_t *)b.chunk, nchunk, nblk,
                           seed, shots, rounds, out, b.flag, sym_n);
    e = hipGetLastError();
    return e;
}

}  // namespace qs
