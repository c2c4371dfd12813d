// Single-workgroup kernels for states that fit in one workgroup's registers
// (n <= 13 for complex64, n <= 12 for complex128): the whole state (and, for
// the adjoint, the adjoint vector) stays in registers for a chunk of up to
// kSmallMaxLayers layers.
//
// Layer k (arXiv:2604.26423, Sec. II-B): cost phase of eq. (2) on every
// amplitude, exp(-i theta_zz (W - 2C)/20) with an FP64 argument, then RX on
// each qubit in turn (eq. 3).  The adjoint walks the chunk backwards,
// accumulating dE/dtheta_x = Im <lam| sum_q X_q |psi> and
// dE/dtheta_zz = -2 Im <lam| C |psi> before undoing each layer on both vectors.
//
// These kernels are a chain of dependent steps on one CU, bound by latency:
// the fewer barriers and the fewer serial steps, the faster.  Index bits 0..5
// are the lanes of a wave, whose butterflies take the partner's value by a
// lane permutation (no LDS, no barrier); the other bits are shared out
// between registers and waves in two layouts, so that two LDS exchanges per
// layer bring every bit into registers (none up to n = 8, one wave).  Eight
// waves at most: with sixteen each exchange costs more than its halved
// register work saves.  The phase factors are a table over the cut values
// 0..W_t, evaluated once per layer, instead of a sine and cosine per
// amplitude and layer, where that is fewer (small_table_entries).  The factors, the order of the qubits (0 to n - 1
// forward, back in reverse) and each operation's rounding are those of a plain
// loop over the qubits.  Measured against that loop in LDS (1024 threads, one
// barrier per qubit): see launch_small_forward.
#include <type_traits>

#include "device.h"

namespace qs {

namespace {

// N: index bits (6 stands for 1..6).  LB lane bits, RB register bits, WB wave
// bits; RB >= WB, so that two layouts put every bit into registers once:
//   layout 1: x = lane | wave << 6 | reg << (6 + WB)
//   layout 2: x = lane | reg << 6 | wave << (6 + RB)
template <int N> struct SmallCfg {
    static constexpr int REST = N - 6;
    static constexpr int WB = REST <= 2 ? 0 : REST / 2;
    static constexpr int RB = REST - WB;
    static constexpr int NR = 1 << RB, NT = 64 << WB;
};

// Phase-table entries in LDS: as many layers as fit are evaluated at once.
template <typename V> constexpr int kSmallTab = small_table_room(sizeof(V) == 8 ? 0 : 1);

// One half of an RX pair, a' = c a - i s b (b: the other amplitude).  Of the
// two products of a part one is rounded and the other goes into the fused
// multiply-add.  Which one is part of the result in complex64 (its last bit,
// and through the sums over a long circuit the gradient's sixth digit), so it
// is fixed here: c a in the fused operation, except for the upper amplitude's
// (bit set, HI) real part forward and its imaginary part in reverse (REV).
// (complex128, where no digit that anyone reads depends on it, has one form.)
template <bool HI, bool REV, typename V, typename R>
__device__ __forceinline__ V rx_half(V a, V b, R c, R s)
{
    V t{fma(c, a.x, s * b.y), fma(c, a.y, -(s * b.x))};
    if constexpr (sizeof(R) == 4 && HI && !REV) t.x = fma(s, b.y, c * a.x);
    if constexpr (sizeof(R) == 4 && HI && REV) t.y = fma(-s, b.x, c * a.y);
    return t;
}

template <typename V>
__device__ __forceinline__ V cmul_fma(V a, V b)
{
    return V{fma(a.x, b.x, -(a.y * b.y)), fma(a.x, b.y, a.y * b.x)};
}

// RX on lane bit B: a lane is the lower or the upper amplitude by its own bit.
template <int B, bool REV, typename V, int NR, typename R>
__device__ __forceinline__ void rx_lane(V (&v)[NR], R c, R s)
{
    const bool hi = (lane_index(threadIdx.x) >> B) & 1;
    const R sr = REV ? -s : s;
    const R fused = hi ? sr : c, plain = hi ? c : sr;
#pragma unroll
    for (int r = 0; r < NR; ++r) {
        const V a = v[r], b = lane_xor_v<B>(a);
        if constexpr (sizeof(R) == 8) {
            v[r] = rx_half<false, REV>(a, b, c, s);
        } else if constexpr (REV) {
            v[r].x = fma(c, a.x, s * b.y);
            v[r].y = fma(fused, hi ? b.x : a.y, plain * (hi ? a.y : b.x));
        } else {
            v[r].x = fma(fused, hi ? b.y : a.x, plain * (hi ? a.x : b.y));
            v[r].y = fma(c, a.y, -(s * b.x));
        }
    }
}

template <int B, bool REV, typename V, int NR, typename R>
__device__ __forceinline__ void rx_reg(V (&v)[NR], R c, R s)
{
#pragma unroll
    for (int r = 0; r < NR; ++r)
        if (!(r & (1 << B))) {
            const V a = v[r], b = v[r | (1 << B)];
            v[r] = rx_half<false, REV>(a, b, c, s);
            v[r | (1 << B)] = rx_half<true, REV>(b, a, c, s);
        }
}

// RX on the lane bits below n, in ascending or descending order.
template <bool DESC, int B = 0, typename V, int NR, typename R>
__device__ __forceinline__ void rx_lanes(V (&v)[NR], int n, R c, R s)
{
    if constexpr (B < 6) {
        constexpr int b = DESC ? 5 - B : B;
        if (b < n) rx_lane<b, DESC>(v, c, s);
        rx_lanes<DESC, B + 1>(v, n, c, s);
    }
}

// RX on register bits LO .. HI - 1, ascending or descending.
template <int LO, int HI, bool DESC, int B = LO, typename V, int NR, typename R>
__device__ __forceinline__ void rx_regs(V (&v)[NR], R c, R s)
{
    if constexpr (B < HI) {
        rx_reg<DESC ? LO + HI - 1 - B : B, DESC>(v, c, s);
        rx_regs<LO, HI, DESC, B + 1>(v, c, s);
    }
}

// Im of conj(l) p, FP64 (the products of complex64 parts are exact).
template <typename V>
__device__ __forceinline__ double im_dot(V l, V p)
{
    return (double)l.x * (double)p.y - (double)l.y * (double)p.x;
}

// sum_q Im <lam| X_q |psi> = sum_x Im conj(l_x) sum_q p_(x ^ bit q): the
// partners of each amplitude are added up first, in FP64, so that a bit costs
// two conversions and two additions per amplitude; eight registers at a time.
// Lane bits below n (0: none) and register bits LO .. HI - 1.
template <int AT, int CH, int B = 0, typename V, int NR>
__device__ __forceinline__ void sum_lanes(double2 (&s)[CH], V (&p)[NR], int n)
{
    if constexpr (B < 6) {
        if (B < n) {
#pragma unroll
            for (int i = 0; i < CH; ++i) {
                const V t = lane_xor_v<B>(p[AT + i]);
                s[i].x += (double)t.x;
                s[i].y += (double)t.y;
            }
            pin_regs(p);
        }
        sum_lanes<AT, CH, B + 1>(s, p, n);
    }
}
template <int LO, int HI, int AT = 0, typename V, int NR>
__device__ __forceinline__ double im_sums(V (&l)[NR], V (&p)[NR], int n)
{
    constexpr int CH = NR < 8 ? NR : 8;
    double2 s[CH] = {};
    sum_lanes<AT, CH>(s, p, n);
#pragma unroll
    for (int b = LO; b < HI; ++b) {
#pragma unroll
        for (int i = 0; i < CH; ++i) {
            s[i].x += (double)p[(AT + i) ^ (1 << b)].x;
            s[i].y += (double)p[(AT + i) ^ (1 << b)].y;
        }
    }
    double g = 0.0;
#pragma unroll
    for (int i = 0; i < CH; ++i) g += (double)l[AT + i].x * s[i].y - (double)l[AT + i].y * s[i].x;
    if constexpr (AT + CH < NR) {
        pin_regs(p);
        pin_regs(l);
        g += im_sums<LO, HI, AT + CH>(l, p, n);
    }
    return g;
}

// Index of register r in layout 1 or 2 (see SmallCfg).
template <int N, int LAYOUT>
__device__ __forceinline__ int small_x(int r, int tid)
{
    using Cfg = SmallCfg<N>;
    const int lane = (int)lane_index(tid & 63), wave = tid >> 6;
    return LAYOUT == 1 ? lane | (wave << 6) | (r << (6 + Cfg::WB)) : lane | (r << 6) | (wave << (6 + Cfg::RB));
}

// Move the thread's amplitudes from one layout to the other.  Consecutive
// lanes hold consecutive elements in both: no bank conflicts.
template <int N, int FROM, typename V, int NR>
__device__ __forceinline__ void small_put(const V (&v)[NR], V *lds, int tid)
{
#pragma unroll
    for (int r = 0; r < NR; ++r) lds[small_x<N, FROM>(r, tid)] = v[r];
}
template <int N, int TO, typename V, int NR>
__device__ __forceinline__ void small_get(V (&v)[NR], const V *lds, int tid)
{
#pragma unroll
    for (int r = 0; r < NR; ++r) v[r] = lds[small_x<N, TO>(r, tid)];
}

// Phase factors of the thread's amplitudes: from the layer's table, or
// evaluated here where the table does not hold C (a diagonal outside 0..W_t,
// or a W_t for which there is no table): one pass of the loop per such
// register, so that the sine and cosine are in the code once.
template <typename V, int NR>
__device__ __forceinline__ void small_factors(V (&f)[NR], const V *tab, int entries, const int32_t (&C)[NR],
                                              double theta, int64_t W)
{
    uint32_t slow = 0;
#pragma unroll
    for (int r = 0; r < NR; ++r) {
        const bool in = (uint32_t)C[r] < (uint32_t)entries;
        slow |= (in ? 0u : 1u) << r;
        f[r] = tab[in ? C[r] : 0];
    }
    while (__ballot(slow != 0)) {
        const int at = slow ? __builtin_ctz(slow) : 0;
        int32_t c = C[0];
#pragma unroll
        for (int r = 1; r < NR; ++r) c = at == r ? C[r] : c;
        const V e = expi<V>(theta * (double)(2 * (int64_t)c - W) / 20.0);
#pragma unroll
        for (int r = 0; r < NR; ++r)
            if (slow != 0 && at == r) f[r] = e;
        slow &= slow - 1;
    }
}

template <typename V, typename R>
struct SmallLds {
    V tab[kSmallTab<V>];
    R c[kSmallMaxLayers], s[kSmallMaxLayers];
    double red[2 * 8];
};

// Entries of one layer's table (0: none) and the layers held at once.
template <typename V, int N>
__device__ __forceinline__ void small_tab_geom(int64_t W, int &entries, int &group)
{
    entries = small_table_entries(sizeof(V) == 8 ? 0 : 1, N, W);
    group = entries ? kSmallTab<V> / entries : kSmallMaxLayers;
}

// Tables of layers [lo, hi).  The factors of C and W - C have opposite angles
// and so are conjugates, bit for bit: one sine and cosine for both.
template <typename V>
__device__ __forceinline__ void small_tables(V *tab, int entries, const SmallProg &sp, int lo, int hi, int tid,
                                             int nt)
{
    const int half = (entries + 1) / 2;
    for (int i = tid; i < (hi - lo) * half; i += nt) {
        const int L = i / half, C = i % half;
        const V f = expi<V>(sp.tzz[lo + L] * (double)(2 * (int64_t)C - sp.W) / 20.0);
        tab[L * entries + C] = f;
        tab[L * entries + (entries - 1 - C)] = C == entries - 1 - C ? f : V{f.x, -f.y};
    }
}

template <typename V, int N>
__global__ void __launch_bounds__(SmallCfg<N>::NT) small_forward(SmallProg sp)
{
    using R = typename Real<V>::T;
    using Cfg = SmallCfg<N>;
    constexpr int NR = Cfg::NR, NT = Cfg::NT, RB = Cfg::RB, WB = Cfg::WB;
    __shared__ SmallLds<V, R> sh;
    __shared__ V xb[WB ? 1 << N : 1];
    const int tid = threadIdx.x, n = N > 6 ? N : sp.n;
    const bool on = N > 6 || (tid >> n) == 0;
    V *psi = reinterpret_cast<V *>(sp.psi);

    V v[NR];
    int32_t C[NR];
#pragma unroll
    for (int r = 0; r < NR; ++r) {
        const int x = small_x<N, 1>(r, tid);
        C[r] = on && sp.diag ? sp.diag[x] : 0;
        v[r] = V{(R)(sp.init && on ? sp.amp0 : 0.0), (R)0};
        if (!sp.init && on) v[r] = psi[x];
    }
    if (tid < sp.nlayers) {
        sh.c[tid] = (R)cos(0.5 * sp.tx[tid]);
        sh.s[tid] = (R)sin(0.5 * sp.tx[tid]);
    }
    int entries, group, base = 0;
    small_tab_geom<V, N>(sp.W, entries, group);
    if (!sp.diag) group = kSmallMaxLayers;
    for (int L = 0; L < sp.nlayers; ++L) {
        if (L % group == 0) {
            __syncthreads();
            base = L;
            if (sp.diag && entries)
                small_tables(sh.tab, entries, sp, L, min(L + group, sp.nlayers), tid, NT);
            __syncthreads();
        }
        if (sp.do_phase[L]) {
            V f[NR];
            small_factors(f, sh.tab + (L - base) * entries, entries, C, sp.tzz[L], sp.W);
#pragma unroll
            for (int r = 0; r < NR; ++r) v[r] = cmul_fma(v[r], f[r]);
        }
        if (sp.do_mixer[L]) {
            const R c = sh.c[L], s = sh.s[L];
            rx_lanes<false>(v, n, c, s);
            if constexpr (WB) {
                // one barrier per exchange: each time a thread writes the slots
                // that it read last (or none has read yet)
                small_put<N, 1>(v, xb, tid);
                __syncthreads();
                small_get<N, 2>(v, xb, tid);
                rx_regs<0, RB, false>(v, c, s);
                small_put<N, 2>(v, xb, tid);
                __syncthreads();
                small_get<N, 1>(v, xb, tid);
                rx_regs<RB - WB, RB, false>(v, c, s);
            } else {
                rx_regs<0, RB, false>(v, c, s);
            }
        }
    }
    if (sp.readout) {
        double acc[2] = {0.0, 0.0};
#pragma unroll
        for (int r = 0; r < NR; ++r) {
            const double pr = (double)v[r].x * (double)v[r].x + (double)v[r].y * (double)v[r].y;
            acc[0] += pr;
            acc[1] += pr * (double)C[r];
        }
        block_sum(acc, sh.red, tid, NT);
        if (tid == 0) {
            sp.out[0] = acc[0];
            sp.out[1] = acc[1];
        }
    }
#pragma unroll
    for (int r = 0; r < NR; ++r)
        if (on) psi[small_x<N, 1>(r, tid)] = v[r];
}

// Accumulator layout in sp.out: [0] norm, [1] sum |a|^2 C_t, [2 + k] dE/dtheta_zz[k],
// [2 + ptotal + k] dE/dtheta_x[k].  The layer's sums are left by each wave in
// LDS and added up, wave by wave, once at the end.
template <typename V, int N>
__global__ void __launch_bounds__(SmallCfg<N>::NT) small_adjoint(SmallProg sp)
{
    using R = typename Real<V>::T;
    using Cfg = SmallCfg<N>;
    constexpr int NR = Cfg::NR, NT = Cfg::NT, RB = Cfg::RB, WB = Cfg::WB, NW = 1 << WB;
    __shared__ SmallLds<V, R> sh;
    __shared__ V xp[WB ? 1 << N : 1], xl[WB ? 1 << N : 1];
    __shared__ double gsum[2 * kSmallMaxLayers * NW];  // [layer][zz, x][wave]
    const int tid = threadIdx.x, n = N > 6 ? N : sp.n, wave = tid >> 6, lane = tid & 63;
    const bool on = N > 6 || (tid >> n) == 0;
    const int ptotal = sp.ptotal;
    V *psi = reinterpret_cast<V *>(sp.psi);
    V *lam = reinterpret_cast<V *>(sp.lam);

    V p[NR], l[NR];
    int32_t C[NR];
#pragma unroll
    for (int r = 0; r < NR; ++r) {
        const int x = small_x<N, 2>(r, tid);
        C[r] = on ? sp.diag[x] : 0;
        p[r] = on ? psi[x] : V{(R)0, (R)0};
        l[r] = V{(R)0, (R)0};
        if (on && !sp.turnaround) l[r] = lam[x];
    }
    if (tid < sp.nlayers) {
        sh.c[tid] = (R)cos(0.5 * sp.tx[tid]);
        sh.s[tid] = (R)-sin(0.5 * sp.tx[tid]);
    }
    if (sp.turnaround) {
        double acc[2] = {0.0, 0.0};
#pragma unroll
        for (int r = 0; r < NR; ++r) {
            const double pr = (double)p[r].x * (double)p[r].x + (double)p[r].y * (double)p[r].y;
            acc[0] += pr;
            acc[1] += pr * (double)C[r];
            const R cu = (R)(((double)C[r] - sp.lam_shift) * 0.1);
            l[r] = V{cu * p[r].x, cu * p[r].y};
        }
        block_sum(acc, sh.red, tid, NT);
        if (tid == 0) {
            sp.out[0] = acc[0];
            sp.out[1] = acc[1];
        }
    }
    int entries, group, base = sp.nlayers;
    small_tab_geom<V, N>(sp.W, entries, group);
    for (int L = sp.nlayers - 1; L >= 0; --L) {
        if (L < base) {
            __syncthreads();
            base = max(0, L + 1 - group);
            if (entries) small_tables(sh.tab, entries, sp, base, L + 1, tid, NT);
            __syncthreads();
        }
        double gx = 0.0, gz = 0.0;
        if (sp.do_mixer[L]) {
            // every qubit's term on the vectors before any RX of the layer is undone
            const R c = sh.c[L], s = sh.s[L];
            gx = im_sums<0, RB>(l, p, n);
            if constexpr (WB) {
                small_put<N, 2>(p, xp, tid);
                small_put<N, 2>(l, xl, tid);
                __syncthreads();
                small_get<N, 1>(p, xp, tid);
                small_get<N, 1>(l, xl, tid);
                gx += im_sums<RB - WB, RB>(l, p, 0);
                rx_regs<RB - WB, RB, true>(p, c, s);
                rx_regs<RB - WB, RB, true>(l, c, s);
                // (a thread writes the slots that it has just read: no barrier in between)
                small_put<N, 1>(p, xp, tid);
                small_put<N, 1>(l, xl, tid);
                __syncthreads();
                small_get<N, 2>(p, xp, tid);
                small_get<N, 2>(l, xl, tid);
            }
            rx_regs<0, RB, true>(p, c, s);
            rx_regs<0, RB, true>(l, c, s);
            rx_lanes<true>(p, n, c, s);
            pin_regs(p);
            pin_regs(l);
            rx_lanes<true>(l, n, c, s);
            pin_regs(p);
            pin_regs(l);
        }
        if (sp.do_phase[L]) {
#pragma unroll
            for (int r = 0; r < NR; ++r) gz += -0.2 * ((double)C[r] - sp.lam_shift) * im_dot(l[r], p[r]);
            V f[NR];
            small_factors(f, sh.tab + (L - base) * entries, entries, C, sp.tzz[L], sp.W);
#pragma unroll
            for (int r = 0; r < NR; ++r) {
                const V g{f[r].x, -f[r].y};
                p[r] = cmul_fma(p[r], g);
                l[r] = cmul_fma(l[r], g);
            }
        }
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) {
            gx += __shfl_xor(gx, off, 64);
            gz += __shfl_xor(gz, off, 64);
        }
        if (lane == 0) {
            gsum[2 * L * NW + wave] = gz;
            gsum[(2 * L + 1) * NW + wave] = gx;
        }
    }
    __syncthreads();
    if (tid < 2 * sp.nlayers) {
        double s = 0.0;
        for (int w = 0; w < NW; ++w) s += gsum[tid * NW + w];
        sp.out[2 + (tid & 1 ? ptotal : 0) + sp.layer0 + (tid >> 1)] = s;
    }
    if (sp.store) {
#pragma unroll
        for (int r = 0; r < NR; ++r) {
            const int x = small_x<N, 2>(r, tid);
            if (on) {
                psi[x] = p[r];
                lam[x] = l[r];
            }
        }
    }
}

template <typename V, typename F>
hipError_t small_dispatch(int n, F &&launch)
{
    switch (n) {
    case 1: case 2: case 3: case 4: case 5: case 6: launch(std::integral_constant<int, 6>{}); break;
    case 7: launch(std::integral_constant<int, 7>{}); break;
    case 8: launch(std::integral_constant<int, 8>{}); break;
    case 9: launch(std::integral_constant<int, 9>{}); break;
    case 10: launch(std::integral_constant<int, 10>{}); break;
    case 11: launch(std::integral_constant<int, 11>{}); break;
    case 12: launch(std::integral_constant<int, 12>{}); break;
    case 13:
        if constexpr (sizeof(V) == sizeof(float2)) {
            launch(std::integral_constant<int, 13>{});
            break;
        }
        return hipErrorInvalidValue;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

}  // namespace

// Whole calls of Simulator.forward / adjoint (us; p = 10 layers), before: one
// 1024-thread workgroup, the state in LDS, a barrier per qubit, a sine and
// cosine per amplitude and layer; about 15 us of each are launch and
// synchronisation:
//   n, precision     forward          forward + adjoint
//    9, complex128    57 ->  33        132 ->  73
//   10, complex64     61 ->  30        148 ->  65
//   12, complex64    119 ->  48        343 -> 132
//   12, complex128   144 ->  59        419 -> 168
//   13, complex64    197 ->  74        614 -> 242
// What is left is the issue rate of one CU's vector units (about 2100
// instructions per wave and reverse layer at n = 12, 8 waves).  The complex64
// reverse kernel of n = 13 spills 35 of its 256 registers, the others none.
hipError_t launch_small_forward(int prec, const SmallProg &sp, hipStream_t st)
{
    if (prec == 0)
        return small_dispatch<float2>(sp.n, [&](auto k) {
            hipLaunchKernelGGL((small_forward<float2, k.value>), dim3(1), dim3(SmallCfg<k.value>::NT), 0, st, sp);
        });
    return small_dispatch<double2>(sp.n, [&](auto k) {
        hipLaunchKernelGGL((small_forward<double2, k.value>), dim3(1), dim3(SmallCfg<k.value>::NT), 0, st, sp);
    });
}

hipError_t launch_small_adjoint(int prec, const SmallProg &sp, hipStream_t st)
{
    if (prec == 0)
        return small_dispatch<float2>(sp.n, [&](auto k) {
            hipLaunchKernelGGL((small_adjoint<float2, k.value>), dim3(1), dim3(SmallCfg<k.value>::NT), 0, st, sp);
        });
    return small_dispatch<double2>(sp.n, [&](auto k) {
        hipLaunchKernelGGL((small_adjoint<double2, k.value>), dim3(1), dim3(SmallCfg<k.value>::NT), 0, st, sp);
    });
}

}  // namespace qs
