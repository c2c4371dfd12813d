// Noisy LR-QAOA trajectories (arXiv:2604.26423, Sec. II-C): a two-qubit
// depolarizing channel of rate eps after every RZZ gate, unravelled into
// Pauli insertions.  One workgroup runs one trajectory of an n <= 12 qubit
// circuit with the whole state in registers (2^RB amplitudes per thread) and
// LDS (exchanges, the cost diagonal, the phase table).
//
// Draw rule (trajectory t, layer k, edge e in lexicographic order):
//   (r0, r1, ..) = Philox4x64-10(counter (t, k, e, 1), key (seed, 0));
//   the gate errs iff (r0 >> 11) < thr = floor(eps 2^53); its Pauli is
//   code = r1 & 15, P_a = code & 3 on the edge's lower qubit, P_b = code >> 2
//   on the upper one (0 I, 1 X, 2 Y = i X Z, 3 Z).
//
// The cost layer stays one fused diagonal.  Errors are moved to the end of
// the layer: an X component on qubit v anticommutes with Z_v Z_u, so every
// later gate touching v changes the sign of its angle.  With F the set of
// gates whose sign flipped an odd number of times,
//   prod_g E_g U_g = E_tot exp(-i theta/2 [sum_g w_g z_a z_b - 2 sum_{g in F} w_g z_a z_b]),
// and E_tot = i^a X^ex Z^ez (product of the layer's Paulis in gate order).
// X components are not applied to the state: they commute with every RX, so
// the trajectory keeps a frame m with psi_true = i^phi X^m psi_stored, and the
// next cost diagonal is read at x ^ m.  Z components are applied as signs.
// Per amplitude the layer's phase is exp(-i theta K / 20) with
//   K = (W - 2 C(y)) - 2 (W_F - 2 C_F(y)),  y = x ^ m,
// C_F the cut of y over the flipped gates (a short list, empty without
// errors).  The mixer is unchanged.
//
// Nothing of this reaches HBM; the vector units bound it (about 640
// instructions per wave and layer at n = 12, 384 of them the RX updates), then
// LDS.  So the layer is kept short: a register's cut values stay in registers
// (a layout's are reloaded when a layer is about to start from it in another
// frame), a layer without errors takes its phase from one table entry per cut
// value, four qubits are updated across lanes instead of through a second
// exchange, the exchange has one barrier, and which layers of a chunk have
// errors is one word.  20,000 trajectories, p = 10, us, before (diagonal and
// two-level table in LDS, two exchanges of two barriers) and now:
//   n, precision     eps = 0.0005    0.003           0.05
//   12, complex64    1363 ->  790    1544 -> 1000    3118 -> 2506
//   12, complex128   2816 -> 1500                    6007 -> 3979
//   11, complex64                     672 ->  500    1258 -> 1197
//   10, complex64                     384 ->  275     633 ->  564
//    9, complex64     176 ->  135                     286 ->  274
// 200 trajectories leave most of the chip idle and are bound by one
// trajectory's chain: n = 12, eps = 0.003 64 -> 66.  Registers for three
// workgroups of n = 12 per CU instead of four: 8% slower.  The n = 11
// complex64 kernel spills 6 of its 128 registers, the others none.
#include "tiles.h"

namespace qs {

namespace {

// Philox4x64-10 (Salmon, Moraes, Dror, Shaw, SC'11), words 0 and 1 of the
// output for counter (c0, c1, c2, c3) and key (k0, 0).
__device__ __forceinline__ void philox_w01(uint64_t c0, uint64_t c1, uint64_t c2, uint64_t c3, uint64_t k0,
                                           uint64_t &w0, uint64_t &w1)
{
    const uint64_t M0 = 0xD2E7470EE14C6C93ULL, M1 = 0xCA5A826395121157ULL;
    const uint64_t W0 = 0x9E3779B97F4A7C15ULL, W1 = 0xBB67AE8584CAA73BULL;
    uint64_t x0 = c0, x1 = c1, x2 = c2, x3 = c3, ka = k0, kb = 0;
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

template <int N> struct NoiseCfg {
    // threads: 2^(n-4) from n = 10 (16 amplitudes each), one wave for n = 8, 9
    static constexpr int TB = N >= 10 ? N - 4 : (N >= 8 ? 6 : N - 2);
    static constexpr int RB = N - TB;
    static constexpr int NR = 1 << RB, NT = 1 << TB;
    static constexpr int WL = NT < 64 ? NT : 64;  // lanes of the bookkeeping wave
    static constexpr int NW = (N + RB - 1) / RB;  // groups of RB qubits, see mid
    static constexpr int G = N * (N - 1) / 2;     // gates per cost layer
    // Two layouts of the index bits.  The top layout holds bits [HI, N) in
    // registers, the low layout bits [0, RB); the M bits between them are
    // thread bits 0 .. M - 1 (lanes: M <= 4) in both, and the other window's
    // bits the thread bits above.  (n = 3: the windows share a bit, M = 0 and
    // the top layout's thread bit is bit 0.)
    static constexpr int HI = N - RB;
    static constexpr int M = N > 2 * RB ? N - 2 * RB : 0;
    static constexpr int XB = TB - M;             // thread bits of the other window
    // The i-th middle qubit of a layer: ascending, or in groups of RB from the
    // highest down and ascending within each (the groups begin at multiples of
    // RB, the last at HI): the order in which the state is rounded.
    static constexpr int mid(int i, bool asc)
    {
        if (asc) return RB + i;
        int at = 0;
        for (int j = NW - 2; j >= 1; --j) {
            const int lo = j * RB, hi = lo + RB < HI ? lo + RB : HI;
            for (int q = lo; q < hi; ++q, ++at)
                if (at == i) return q;
        }
        return RB;
    }
};

// Workgroup sum of two doubles into thread 0.  Fewer than 64 threads form
// one partial wave: shuffle only among its lanes.
template <int NT>
__device__ __forceinline__ void noise_sum(double (&x)[2], double *red, int tid)
{
    if constexpr (NT >= 64) {
        block_sum(x, red, tid, NT);
    } else {
#pragma unroll
        for (int k = 0; k < 2; ++k) {
#pragma unroll
            for (int off = NT / 2; off >= 1; off >>= 1) x[k] += __shfl_xor(x[k], off, 64);
        }
    }
}

// Index bits of register r in the low or the top layout, and the LDS slot
// through which it passes to the other one: the same slot, so that a thread
// writes exactly the slots that it has read last (one barrier per exchange).
// Rows of 2^TB + 2^M slots put the lanes of half a wave on distinct banks
// either way, at a constant distance from register to register.
template <int N, bool TOP>
__host__ __device__ __forceinline__ constexpr uint32_t noise_x(int r, int tid)
{
    using Cfg = NoiseCfg<N>;
    // (the middle bits are lane bits, see lane_index)
    const uint32_t l = (uint32_t)tid & ((1u << Cfg::M) - 1u), o = (uint32_t)tid >> Cfg::M;
    const uint32_t m = Cfg::M > 2 ? lane_index(l) : l;
    return TOP ? o | (m << Cfg::RB) | ((uint32_t)r << Cfg::HI) : (uint32_t)r | (m << Cfg::RB) | (o << (N - Cfg::XB));
}
template <int N> constexpr int kNoiseRow = (1 << NoiseCfg<N>::TB) + (1 << NoiseCfg<N>::M);
template <int N, bool TOP>
__host__ __device__ __forceinline__ constexpr int noise_slot(int r, int tid)
{
    using Cfg = NoiseCfg<N>;
    const int m = tid & ((1 << Cfg::M) - 1), o = tid >> Cfg::M;
    if (!TOP) return r * kNoiseRow<N> + tid;
    // the row is the low RB index bits, the place in it the high XB ones
    if (2 * Cfg::RB > N)  // (n = 3: the windows share a bit)
        return (o | ((r << Cfg::HI) & ((1 << Cfg::RB) - 1))) * kNoiseRow<N> + (r >> (Cfg::RB - Cfg::XB));
    return o * kNoiseRow<N> + (r << Cfg::M) + m;
}

// Cut values 0 .. W_t of a layer without sign flips: one table entry each, the
// product of the two levels, when they are at most kNoiseDirect (this many let
// four workgroups of n = 12 share a CU's LDS).
constexpr int kNoiseDirect = 528;
// The layer's table goes through LDS from n = 9 on; below, a trajectory's 2^n
// amplitudes read fewer entries than its 2^(n-2) threads would copy.  20,000
// trajectories, p = 10, us, through LDS / from global memory: n = 12, eps = 0.05
// 2556 / 3299; eps = 0.003, n = 10, W_t = 962 307 / 359; n = 8, W_t = 658 113 /
// 109; n = 6, W_t = 848 160 / 129; n = 4, W_t = 987 333 / 162.
template <int N> constexpr bool kNoiseStage = N >= 9;
static_assert(kNoiseDirect >= kTabMax, "the levels of a table take its place in LDS");

struct NoiseShared {
    int nf, wf, ph, cnt;
    uint32_t ex, ez;
    uint32_t drawn;  // bit i: layer i of the chunk has an error
};
static_assert(kNoiseChunk <= 32, "one bit per layer of a chunk");

// LV = 2: two-level phase table (3 W < 2^13, every graph with weights up to
// 10 tenths at n <= 12); LV = 0: levels read at run time.
template <typename V, int LV>
__device__ __forceinline__ V noise_phase(const V *tab, int levels, int u)
{
    if constexpr (LV == 2) return cmul(tab[u & 63], tab[64 + ((u >> 6) & 127)]);
    else return phase_factor(tab, levels, u);
}

// RX on one qubit: a register bit, or a lane bit (the partner's value through a
// lane permutation; the same fused operations for both ends of the pair).
template <int B, int MODE, typename V, int NR, typename R>
__device__ __forceinline__ void noise_rx_reg(V (&v)[NR], R a, R b)
{
    if constexpr (MODE == kModeTan) rxt_reg_bit<B>(v, a);
    else rx_reg_bit<B>(v, a, b);
}
template <int B, int MODE, typename V, int NR, typename R>
__device__ __forceinline__ void noise_rx_lane(V (&v)[NR], R a, R b)
{
#pragma unroll
    for (int r = 0; r < NR; ++r) {
        const V o = v[r], p = lane_xor_v<B>(o);
        if constexpr (MODE == kModeTan) v[r] = V{fma(a, p.y, o.x), fma(-a, p.x, o.y)};
        else v[r] = V{fma(a, o.x, b * p.y), fma(a, o.y, -(b * p.x))};
    }
}
template <int N, int MODE, bool ASC, int I = 0, typename V, int NR, typename R>
__device__ __forceinline__ void noise_mid(V (&v)[NR], R a, R b)
{
    using Cfg = NoiseCfg<N>;
    if constexpr (I < Cfg::M) {
        noise_rx_lane<Cfg::mid(I, ASC) - Cfg::RB, MODE>(v, a, b);
        noise_mid<N, MODE, ASC, I + 1>(v, a, b);
    }
}
// Register bits LO .. RB - 1.
template <int N, int MODE, int LO, typename V, int NR, typename R>
__device__ __forceinline__ void noise_regs(V (&v)[NR], R a, R b)
{
    if constexpr (LO < NoiseCfg<N>::RB) {
        noise_rx_reg<LO, MODE>(v, a, b);
        noise_regs<N, MODE, LO + 1>(v, a, b);
    }
}

// The thread index, hidden from the optimizer: what the rare paths derive from
// it is computed there and does not occupy registers through every layer.
__device__ __forceinline__ int noise_tid(int tid)
{
    asm volatile("" : "+v"(tid));
    return tid;
}

// Cut values of the thread's registers in the top or the low layout, and the
// frame that they are for.
template <int N, bool TOP, int NR>
__device__ __forceinline__ void noise_cuts(const int32_t *diag, uint32_t m, int tid, int32_t (&c)[NR], uint32_t &frame)
{
    tid = noise_tid(tid);
#pragma unroll
    for (int r = 0; r < NR; ++r) c[r] = diag[noise_x<N, TOP>(r, tid) ^ m];
    frame = m;
}

// Cost layer with its errors, then the mixer, for layer k.  Ascending layers
// take the state from the low layout to the top one, the others back.
template <typename V, int N, int MODE, int LV, bool ASC>
__device__ __forceinline__ void noise_layer(const NoiseProg &np, int k, V (&v)[NoiseCfg<N>::NR], V *lds,
                                            int32_t (&clo)[NoiseCfg<N>::NR], int32_t (&chi)[NoiseCfg<N>::NR],
                                            uint32_t &mlo, uint32_t &mhi, V *tab, uint8_t *codes, uint32_t &drawn, uint32_t *fm, int *fw,
                                            NoiseShared &sh, uint32_t &m, int &phi, int &nerr, double &fprev, int tid)
{
    using Cfg = NoiseCfg<N>;
    using R = typename Real<V>::T;
    constexpr int RB = Cfg::RB, NR = Cfg::NR, NT = Cfg::NT, G = Cfg::G, WL = Cfg::WL;
    const double *lay = np.layers + 4 * k;
    const int at = k % kNoiseChunk;

    // draws of the next chunk of layers (counter-based: any order gives the
    // same codes), and whether a layer has any error
    if (at == 0) {
        const int len = np.p - k < kNoiseChunk ? np.p - k : kNoiseChunk;
        __syncthreads();  // the previous chunk's codes are no longer read
        if (tid == 0) sh.drawn = 0;
        __syncthreads();
        for (int i = tid; i < len * G; i += NT) {
            uint8_t c = 0;
            if (np.thr != 0) {
                uint64_t r0, r1;
                philox_w01(np.traj0 + blockIdx.x, (uint64_t)(k + i / G), (uint64_t)(i % G), 1, np.seed, r0, r1);
                c = (r0 >> 11) < np.thr ? (uint8_t)(r1 & 15u) : (uint8_t)0;
            }
            codes[i] = c;
            if (c) atomicOr(&sh.drawn, 1u << (i / G));
        }
        __syncthreads();
        drawn = (uint32_t)__builtin_amdgcn_readfirstlane((int)sh.drawn);
    }
    const bool errs = (drawn >> at) & 1u;

    // Table of the layer (the same for every trajectory, built by
    // noise_table_kernel): an entry per cut value if nothing flips a sign, else,
    // and for more cut values than that, its levels.  The last reads of the
    // previous layer's table and flags lie before that layer's exchange.
    const bool flat = np.direct && !errs;
    const V *src = reinterpret_cast<const V *>(np.tabs) + (size_t)k * (kTabMax + kNoiseDirect) + (flat ? kTabMax : 0);
    if constexpr (kNoiseStage<N>) {
        const int len = flat ? (int)np.W + 1 : 64 * (np.levels - 1) + 128;
        for (int i = tid; i < len; i += NT) tab[i] = src[i];
        src = tab;
    }

    // the layer's errors, moved to its end (one wave, gates in order)
    if (errs && tid < WL) {
        const int lane = tid;
        const uint8_t *cl = codes + at * G;
        uint32_t carry = 0, ez = 0;
        int nf = 0, wf = 0, ph = 0, cnt = 0;
        for (int base = 0; base < G; base += WL) {
            const int e = base + lane;
            const bool valid = e < G;
            const int code = valid ? cl[e] : 0;
            const uint32_t ab = valid ? (uint32_t)np.edges[e] : 0u;
            const int a = ab & 15, b = (ab >> 4) & 15, wt = (int)(ab >> 8);
            const int pa = code & 3, pb = code >> 2;
            const uint32_t xm = ((uint32_t)(pa == 1 || pa == 2) << a) | ((uint32_t)(pb == 1 || pb == 2) << b);
            const uint32_t zm = ((uint32_t)(pa >= 2) << a) | ((uint32_t)(pb >= 2) << b);
            // prefix XOR of the X components over the gates before e
            uint32_t incl = xm;
#pragma unroll
            for (int d = 1; d < WL; d <<= 1) {
                const uint32_t t = __shfl_up(incl, d, 64);
                if (lane >= d) incl ^= t;
            }
            const uint32_t before = incl ^ xm ^ carry;
            const uint32_t emask = (1u << a) | (1u << b);
            const bool flip = valid && (__popc(before & emask) & 1);
            const uint64_t bal = __ballot(flip);
            if (flip) {
                const int to = nf + __popcll(bal & ((1ull << lane) - 1ull));
                fm[to] = emask;
                fw[to] = wt;
            }
            nf += __popcll(bal);
            int sw = flip ? wt : 0;
            // E_e (i^y X^xm Z^zm) multiplied onto the product of the earlier errors
            int sp = (pa == 2) + (pb == 2) + 2 * (__popc(zm & before) & 1);
            int sc = code != 0;
            uint32_t sz = zm;
#pragma unroll
            for (int off = WL / 2; off >= 1; off >>= 1) {
                sw += __shfl_xor(sw, off, 64);
                sp += __shfl_xor(sp, off, 64);
                sc += __shfl_xor(sc, off, 64);
                sz ^= __shfl_xor(sz, off, 64);
            }
            wf += sw;
            ph += sp;
            cnt += sc;
            ez ^= sz;
            carry ^= __shfl(incl, WL - 1, 64);
        }
        if (lane == 0) {
            sh.nf = nf;
            sh.wf = wf;
            sh.ph = ph & 3;
            sh.cnt = cnt;
            sh.ex = carry;
            sh.ez = ez;
        }
    }
    __syncthreads();

    // The frame moves at the end of the layer, and with it the cut values of the
    // layout that the next one starts from (the other's when a layer starts from
    // it); their loads go ahead of this layer's arithmetic.
    const uint32_t next = errs ? m ^ (uint32_t)__builtin_amdgcn_readfirstlane((int)sh.ex) : m;
    if constexpr (ASC) {
        if (mhi != next) noise_cuts<N, true>(np.diag, next, tid, chi, mhi);
    } else {
        if (mlo != next) noise_cuts<N, false>(np.diag, next, tid, clo, mlo);
    }

    // cost phase, in the layout that the layer starts from
    const auto c = [&](int r) {
        if constexpr (ASC) return clo[r];
        else return chi[r];
    };
    const int nf = errs ? __builtin_amdgcn_readfirstlane(sh.nf) : 0;
    V f[NR];
    if (flat) {
#pragma unroll
        for (int r = 0; r < NR; ++r) f[r] = src[c(r)];
    } else {
        int cf[NR];
        const int tf = noise_tid(tid);
#pragma unroll
        for (int r = 0; r < NR; ++r) cf[r] = 0;
        for (int i = 0; i < nf; ++i) {
            const uint32_t mk = fm[i];
            const int wk = fw[i];
#pragma unroll
            for (int r = 0; r < NR; ++r)
                cf[r] += (__popc((noise_x<N, !ASC>(r, tf) ^ m) & mk) & 1) ? wk : 0;
        }
        const int u0 = 2 * (int)np.W - (nf ? __builtin_amdgcn_readfirstlane(sh.wf) : 0);
#pragma unroll
        for (int r = 0; r < NR; ++r) f[r] = noise_phase<V, LV>(src, np.levels, u0 - c(r) + 2 * cf[r]);
    }
    if (errs) {
        const uint32_t ez = (uint32_t)__builtin_amdgcn_readfirstlane((int)sh.ez);
        if (ez != 0) {  // Z components of the layer's errors: signs
            const int tz = noise_tid(tid);
#pragma unroll
            for (int r = 0; r < NR; ++r)
                if (__popc(noise_x<N, !ASC>(r, tz) & ez) & 1) f[r] = V{-f[r].x, -f[r].y};
        }
        phi = (phi + sh.ph + 2 * (__popc(ez & m) & 1)) & 3;
        nerr += sh.cnt;
    }
#pragma unroll
    for (int r = 0; r < NR; ++r) v[r] = cmul(v[r], f[r]);

    // mixer: RX on every qubit; the registers' qubits of the starting layout,
    // the middle ones, and after the exchange the other window's
    const R a = (R)lay[1], b = (R)lay[2];
    noise_regs<N, MODE, 0>(v, a, b);
    noise_mid<N, MODE, ASC>(v, a, b);
    if constexpr (Cfg::TB > 0) {
#pragma unroll
        for (int r = 0; r < NR; ++r) lds[noise_slot<N, !ASC>(r, tid)] = v[r];
        __syncthreads();
#pragma unroll
        for (int r = 0; r < NR; ++r) v[r] = lds[noise_slot<N, ASC>(r, tid)];
        // (n = 3: the windows share a qubit, already done)
        if constexpr (ASC) noise_regs<N, MODE, (2 * RB > N ? 2 * RB - N : 0)>(v, a, b);
        else if constexpr (2 * RB > N) noise_rx_reg<0, MODE>(v, a, b);
        else noise_regs<N, MODE, 0>(v, a, b);
    }
    m = next;
    fprev = lay[3];
}

// Norm, sum |a|^2 C and the final state: psi_true[x ^ m] = i^phi fs psi_stored[x].
template <typename V, int N, bool TOP, int NR, typename R>
__device__ __forceinline__ void noise_readout(const NoiseProg &np, const V (&v)[NR], const int32_t (&c)[NR], uint32_t m,
                                              int phi, R fs, double (&acc)[2], int tid)
{
    V *out = np.states ? reinterpret_cast<V *>(np.states) + ((int64_t)blockIdx.x << N) : nullptr;
#pragma unroll
    for (int r = 0; r < NR; ++r) {
        V a = V{fs * v[r].x, fs * v[r].y};
        const double pr = (double)a.x * (double)a.x + (double)a.y * (double)a.y;
        acc[0] += pr;
        acc[1] += pr * (double)c[r];
        if (out) {
            V t = a;
            if (phi & 1) t = V{-a.y, a.x};
            if (phi & 2) t = V{-t.x, -t.y};
            out[noise_x<N, TOP>(r, tid) ^ m] = t;
        }
    }
}

// Registers for as many workgroups of n >= 11 (complex128: 10) as share a CU's
// LDS; bounded like that the n = 10 complex64 kernel lost 4%.
template <typename V, int N, int MODE, int LV>
__global__ void __launch_bounds__(NoiseCfg<N>::NT, (N < (sizeof(V) == 8 ? 11 : 10) ? 1 : sizeof(V) == 8 ? 4 : 2)) noise_kernel(NoiseProg np)
{
    using Cfg = NoiseCfg<N>;
    using R = typename Real<V>::T;
    constexpr int NR = Cfg::NR, NT = Cfg::NT, G = Cfg::G;
    __shared__ V lds[kNoiseRow<N> << Cfg::RB];
    __shared__ V tab[kNoiseStage<N> ? kNoiseDirect : 1];
    __shared__ uint8_t codes[kNoiseChunk * G];
    __shared__ uint32_t fm[G];
    __shared__ int fw[G];
    __shared__ NoiseShared sh;
    __shared__ double red[2 * (NT < 64 ? 1 : NT / 64)];
    const int tid = threadIdx.x;

    V v[NR];
    int32_t clo[NR], chi[NR];
    uint32_t mlo, mhi, drawn = 0;
    noise_cuts<N, false>(np.diag, 0u, tid, clo, mlo);
    noise_cuts<N, true>(np.diag, 0u, tid, chi, mhi);
#pragma unroll
    for (int r = 0; r < NR; ++r) v[r] = V{(R)np.amp0, (R)0};
    uint32_t m = 0;
    int phi = 0, nerr = 0;
    double fprev = 1.0;

    int k = 0;
    for (; k + 1 < np.p; k += 2) {
        noise_layer<V, N, MODE, LV, true>(np, k, v, lds, clo, chi, mlo, mhi, tab, codes, drawn, fm, fw, sh, m, phi,
                                          nerr, fprev, tid);
        noise_layer<V, N, MODE, LV, false>(np, k + 1, v, lds, clo, chi, mlo, mhi, tab, codes, drawn, fm, fw, sh, m,
                                           phi, nerr, fprev, tid);
    }
    const bool top = k < np.p;
    if (top)
        noise_layer<V, N, MODE, LV, true>(np, k, v, lds, clo, chi, mlo, mhi, tab, codes, drawn, fm, fw, sh, m, phi,
                                          nerr, fprev, tid);

    double acc[2] = {0.0, 0.0};
    if (top) noise_readout<V, N, true>(np, v, chi, m, phi, (R)fprev, acc, tid);
    else noise_readout<V, N, false>(np, v, clo, m, phi, (R)fprev, acc, tid);
    noise_sum<NT>(acc, red, tid);
    if (tid == 0) {
        np.exp_c[blockIdx.x] = acc[1] / acc[0] / 10.0;
        if (np.norm) np.norm[blockIdx.x] = acc[0];
        if (np.nerr) np.nerr[blockIdx.x] = nerr;
    }
}

// Phase table of every layer k: entry(u) = f_(k-1) exp(-i theta_zz,k (2u - 3W) / 20),
// f_(k-1) the tangent-form factor of the previous layer's mixer (1 for k = 0);
// then, for cut value C of a layer without flips, the factor of u = 2W - C, as
// the two levels give it.
template <typename V>
__global__ void __launch_bounds__(256) noise_table_kernel(NoiseProg np)
{
    const int k = blockIdx.x;
    const double f = k == 0 ? 1.0 : np.layers[4 * (k - 1) + 3];
    V *tab = reinterpret_cast<V *>(np.tabs) + (size_t)k * (kTabMax + kNoiseDirect);
    build_phase_table(tab, np.levels, -np.layers[4 * k], 3 * np.W, f, threadIdx.x, 256);
    if (!np.direct) return;
    __syncthreads();
    for (int C = threadIdx.x; C <= (int)np.W; C += 256)
        tab[kTabMax + C] = noise_phase<V, 2>(tab, np.levels, 2 * (int)np.W - C);
}

template <typename V, int MODE, int LV>
hipError_t launch_noise_v(const NoiseProg &np, int64_t ntraj, hipStream_t st)
{
    hipLaunchKernelGGL(noise_table_kernel<V>, dim3(np.p), dim3(256), 0, st, np);
    const dim3 g((unsigned)ntraj);
    switch (np.n) {
#define QS_NOISE_CASE(NN)                                                                                       \
    case NN: hipLaunchKernelGGL((noise_kernel<V, NN, MODE, LV>), g, dim3(NoiseCfg<NN>::NT), 0, st, np); break;
        QS_NOISE_CASE(2)
        QS_NOISE_CASE(3)
        QS_NOISE_CASE(4)
        QS_NOISE_CASE(5)
        QS_NOISE_CASE(6)
        QS_NOISE_CASE(7)
        QS_NOISE_CASE(8)
        QS_NOISE_CASE(9)
        QS_NOISE_CASE(10)
        QS_NOISE_CASE(11)
        QS_NOISE_CASE(12)
#undef QS_NOISE_CASE
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

}  // namespace

int noise_table_entries() { return kTabMax + kNoiseDirect; }

int noise_direct(int64_t W, int levels) { return levels == 2 && W < kNoiseDirect ? 1 : 0; }

int noise_threads(int n)
{
    return n >= 10 ? 1 << (n - 4) : (n >= 8 ? 64 : 1 << (n - 2));
}

hipError_t launch_noise(int prec, int tangent, const NoiseProg &np, int64_t ntraj, hipStream_t st)
{
    if (np.n < 2 || np.n > kNoiseMaxQubits || ntraj < 1 || ntraj > 0x7fffffff) return hipErrorInvalidValue;
    // np.levels is 2 whenever 3 W < 2^13 (the host raises 1 to 2); larger graphs take the
    // run-time-levels kernel with the direct-form mixer
    if (np.levels == 2) {
        if (prec == 0)
            return tangent ? launch_noise_v<float2, kModeTan, 2>(np, ntraj, st)
                           : launch_noise_v<float2, kModeGeneral, 2>(np, ntraj, st);
        return tangent ? launch_noise_v<double2, kModeTan, 2>(np, ntraj, st)
                       : launch_noise_v<double2, kModeGeneral, 2>(np, ntraj, st);
    }
    return prec == 0 ? launch_noise_v<float2, kModeGeneral, 0>(np, ntraj, st)
                     : launch_noise_v<double2, kModeGeneral, 0>(np, ntraj, st);
}

}  // namespace qs
