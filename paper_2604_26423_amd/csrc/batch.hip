// Batched forward + adjoint gradient of many circuits.  Each circuit runs the
// same pass sequence as a single circuit: forward passes, the turnaround,
// reverse passes.  Launch r runs step r of every circuit that has one: its
// workgroups are the items (a tile, or a few tiles of a large state) of all
// those steps, whatever their shape.  The kernel boundary is the only
// synchronisation.  (One persistent launch with a ticket queue and completion
// counters, agent-scope release and acquire fences around every item, took
// 20.6 ms instead of 13.3 for 128 circuits of 14 to 22 qubits, 79 instead of 49
// for 512, 4.6 instead of 0.8 for 64 circuits of 14 to 17: each fence writes
// back or drops a whole L2, and halving the items' size doubled the time.)
#include "tiles.h"

namespace qs {

namespace {

// Kernel shapes.  FAST: the steps whose stages are in tangent form; each pass
// runs code fixed for its shape (see pass_shape), psi and lambda are exchanged
// one after the other through a one-tile buffer, and two workgroups share a
// CU: 512 threads within 128 registers in complex64 (127, no spill), 256 threads
// within 256 in complex128 (252; with 512 the single circuits' junction
// spills).  One workgroup's loads and barriers then overlap the other's
// arithmetic.  (Complex64 with the 256 threads
// and 5-bit windows of the single circuits' reverse kernels has not been
// tried.)  The other steps (a mixer angle with |cos(theta / 2)| < 1/2) run
// runtime-shape code, 512 threads, one workgroup per CU with a two-tile buffer.
// A round that has steps of both kinds launches both kernels over all its
// items, and a workgroup leaves when its item's step is the other's; other
// rounds do not look, since that read ahead of the step's others cost 0.5-1% (60
// rounds of one circuit of 14 qubits 1955 us, without it 1941).  The general
// kernel for all 512 circuits takes 58.2 ms when one of them has such an angle,
// this 40.4, and 39.6 without the angle; where rounds are short the second
// launches cost more than that saves (64 circuits of 14 to 17: 688 and 718 us),
// but a circuit's results do not depend on the others.
template <typename V, bool FAST> constexpr int batch_tb = FAST && sizeof(V) == 16 ? 8 : 9;

// Tiles [t0, t1) of one step, general stage code.
template <typename V, int T>
__device__ __forceinline__ void run_item(const BatchStep &st, int64_t t0, int64_t t1, V *lds, const V *tab,
                                         double (&acc)[kSlots], int tid)
{
    constexpr int TB = batch_tb<V, false>, NR = TileCfg<V, T, TB>::NR;
    const PassProg &pp = st.pp;
    if (st.kind == 0) {
        double fa[2] = {0.0, 0.0};
        for (int64_t t = t0; t < t1; ++t) fwd_tile<V, T, TB, kModeGeneral>(pp, t, lds, tab, fa, tid);
        acc[0] = fa[0];
        acc[1] = fa[1];
    } else if (st.kind == 1) {
        for (int64_t t = t0; t < t1; ++t) turn_tile<V, T, TB, kModeGeneral>(pp, t, lds, acc, tid);
    } else {
        for (int64_t t = t0; t < t1; ++t) {
            V p[NR], l[NR];
            int32_t dg[NR];
            if (pp.has_phase) rev_load_diag<V, T, TB>(pp, t, dg, tid);
            rev_load_vectors<V, T, TB>(pp, t, p, l, tid);
            rev_tile<V, T, TB, kModeGeneral>(pp, t, p, l, dg, lds, tab, acc, tid);
        }
    }
}

// The same in tangent form, with code fixed for each shape.
template <typename V, int T, int TB, int SH>
__device__ __forceinline__ void fwd_tiles(const PassProg &pp, int64_t t0, int64_t t1, V *lds, const V *tab, int tid)
{
    double fa[2] = {0.0, 0.0};  // no readout: the turnaround takes the last pass
    for (int64_t t = t0; t < t1; ++t) fwd_tile<V, T, TB, kModeTan, SH>(pp, t, lds, tab, fa, tid);
}

template <typename V, int T, int TB, int SH>
__device__ __forceinline__ void rev_tiles(const PassProg &pp, int64_t t0, int64_t t1, V *lds, const V *tab,
                                          double (&acc)[kSlots], int tid)
{
    constexpr int NR = TileCfg<V, T, TB>::NR;
    constexpr bool LATE = SH == (kShPre | kShPhase | kShPost);  // within the registers (see adjoint_kernel)
    for (int64_t t = t0; t < t1; ++t) {
        V p[NR], l[NR];
        int32_t dg[NR];
        if (!LATE && (SH & kShPhase)) rev_load_diag<V, T, TB>(pp, t, dg, tid);
        rev_load_vectors<V, T, TB>(pp, t, p, l, tid);
        rev_tile<V, T, TB, kModeTan, SH, false, LATE>(pp, t, p, l, dg, lds, tab, acc, tid);
    }
}

template <typename V, int T>
__device__ __forceinline__ void run_item_fast(const BatchStep &st, int64_t t0, int64_t t1, V *lds, const V *tab,
                                              double (&acc)[kSlots], int tid)
{
    constexpr int TB = batch_tb<V, true>, NR = TileCfg<V, T, TB>::NR;
    constexpr int kFirst = kShInit | kShPhase | kShPost, kJunc = kShPre | kShPhase | kShPost;
    const PassProg &pp = st.pp;
    const int sh = __builtin_amdgcn_readfirstlane(pass_shape(pp));
    if (st.kind == 0) {
        if (sh == kFirst) fwd_tiles<V, T, TB, kFirst>(pp, t0, t1, lds, tab, tid);
        else if (sh == kJunc) fwd_tiles<V, T, TB, kJunc>(pp, t0, t1, lds, tab, tid);
        else fwd_tiles<V, T, TB, kShPost>(pp, t0, t1, lds, tab, tid);
    } else if (st.kind == 1) {
        for (int64_t t = t0; t < t1; ++t) {
            V p[NR];
            int32_t dg[NR];
            turn_load_diag<V, T, TB>(pp, t, dg, tid);
            turn_load<V, T, TB>(pp, t, p, tid);
            turn_compute<V, T, TB, kModeTan, false>(pp, t, p, dg, lds, acc, tid);
        }
    } else {
        if (sh == kFirst) rev_tiles<V, T, TB, kFirst>(pp, t0, t1, lds, tab, acc, tid);
        else if (sh == kJunc) rev_tiles<V, T, TB, kJunc>(pp, t0, t1, lds, tab, acc, tid);
        else rev_tiles<V, T, TB, kShPost>(pp, t0, t1, lds, tab, acc, tid);
    }
}

// Workgroup b of launch `round` takes item i of the first nitems.  Workgroups
// go to XCDs round-robin; runs of kBatchRun consecutive items go to one XCD, so
// that neighbouring tiles, whose 64-byte runs share 128-byte lines, share an
// L2, while each XCD still gets items of every circuit (the circuits of a
// launch may be at passes of very different cost).
constexpr int kBatchRun = 16;

template <typename V, int T, bool FAST>
__global__ void __launch_bounds__((1 << batch_tb<V, FAST>), (!FAST ? 1 : batch_tb<V, FAST> == 9 ? 4 : 2))
    batch_kernel(BatchArgs a, int round, int64_t nitems, int mixed)
{
    constexpr int NT = 1 << batch_tb<V, FAST>;
    __shared__ V lds[(FAST ? 1 : 2) << T];
    __shared__ V tab[kTabMax];
    __shared__ double red[kSlots * (NT / 64)];
    const int tid = threadIdx.x;
    const int64_t k = blockIdx.x >> 3;
    const int64_t item = ((k / kBatchRun) * 8 + (blockIdx.x & 7)) * kBatchRun + k % kBatchRun;
    if (item >= nitems) return;
    const BatchItem it = a.items[item];
    const BatchStep &st = a.steps[__builtin_amdgcn_readfirstlane(it.step0) + round];
    if (mixed && (st.fast != 0) != FAST) return;
    const PassProg &pp = st.pp;
    const int64_t t0 = (int64_t)__builtin_amdgcn_readfirstlane(it.chunk) * st.tiles_per_chunk;
    const int64_t t1 = t0 + st.tiles_per_chunk < pp.ntiles ? t0 + st.tiles_per_chunk : pp.ntiles;
    if (pp.has_phase) {
        load_phase_table(tab, reinterpret_cast<const V *>(a.tabs) + st.tab_off, pp.phase_levels, tid, NT);
        __syncthreads();
    }
    double acc[kSlots] = {0.0, 0.0, 0.0, 0.0};
    if constexpr (FAST) run_item_fast<V, T>(st, t0, t1, lds, tab, acc, tid);
    else run_item<V, T>(st, t0, t1, lds, tab, acc, tid);
    if (st.kind == 0) return;
    block_sum(acc, red, tid, NT);
    if (tid == 0) {
        double *row = a.partials + (st.row0 + it.chunk) * kSlots;
#pragma unroll
        for (int j = 0; j < kSlots; ++j) row[j] = acc[j];
    }
}

// One workgroup per step: that step's phase table.  Forward passes, and
// reverse passes in tangent form that undo a phase, carry the tangent-form
// factor of their stages (see rev_tile); the others use the plain phase.
template <typename V>
__global__ void __launch_bounds__(256) batch_table_kernel(const BatchStep *steps, V *tabs)
{
    const BatchStep &st = steps[blockIdx.x];
    if (!st.pp.has_phase || st.tab_off < 0) return;
    const bool fold = st.kind == 2 && st.mode == kModeTan && !st.pp.init;  // (the fast kernel's)
    const double f = st.kind == 0 || fold ? st.pp.factor : 1.0;
    build_phase_table(tabs + st.tab_off, st.pp.phase_levels, st.pp.theta_zz, st.pp.W, f, threadIdx.x, 256);
}

// One workgroup per step that writes sums: they go to sums[kSlots * its number
// among those steps], added up in a fixed order.
__global__ void __launch_bounds__(256) batch_reduce_kernel(const BatchStep *steps, const int *summed,
                                                           const double *partials, double *sums)
{
    __shared__ double red[kSlots * 4];
    const BatchStep &st = steps[summed[blockIdx.x]];
    double acc[kSlots] = {0.0, 0.0, 0.0, 0.0};
    for (int64_t i = threadIdx.x; i < st.chunks; i += 256) {
#pragma unroll
        for (int k = 0; k < kSlots; ++k) acc[k] += partials[(st.row0 + i) * kSlots + k];
    }
    block_sum(acc, red, threadIdx.x, 256);
    if (threadIdx.x == 0) {
#pragma unroll
        for (int k = 0; k < kSlots; ++k) sums[(int64_t)blockIdx.x * kSlots + k] = acc[k];
    }
}

}  // namespace

int batch_table_entries() { return kTabMax; }

namespace {
// f(kernel, threads) for the batch kernel of a precision and shape.
template <typename F>
auto with_batch_kernel(int prec, bool fast, F &&f)
{
    if (prec == 0)
        return fast ? f(batch_kernel<float2, kTileBitsC64, true>, 1 << batch_tb<float2, true>)
                    : f(batch_kernel<float2, kTileBitsC64, false>, 1 << batch_tb<float2, false>);
    return fast ? f(batch_kernel<double2, kTileBitsC128, true>, 1 << batch_tb<double2, true>)
                : f(batch_kernel<double2, kTileBitsC128, false>, 1 << batch_tb<double2, false>);
}
}  // namespace

int batch_thread_bits(int prec, bool fast)
{
    if (prec == 0) return fast ? batch_tb<float2, true> : batch_tb<float2, false>;
    return fast ? batch_tb<double2, true> : batch_tb<double2, false>;
}

bool batch_step_fast(const BatchStep &s)
{
    const int sh = pass_shape(s.pp);
    return s.mode == kModeTan &&
           (sh == kShPost || sh == (kShInit | kShPhase | kShPost) || sh == (kShPre | kShPhase | kShPost));
}

hipError_t launch_batch_tables(int prec, const BatchStep *steps, int nsteps, void *tabs, hipStream_t st)
{
    if (prec == 0)
        hipLaunchKernelGGL(batch_table_kernel<float2>, dim3(nsteps), dim3(256), 0, st, steps, (float2 *)tabs);
    else
        hipLaunchKernelGGL(batch_table_kernel<double2>, dim3(nsteps), dim3(256), 0, st, steps, (double2 *)tabs);
    return hipGetLastError();
}

hipError_t launch_batch_round(int prec, bool fast, bool mixed, const BatchArgs &a, int round, int64_t nitems,
                              hipStream_t st)
{
    const int64_t per = 8 * kBatchRun, grid = (nitems + per - 1) / per * per;
    return with_batch_kernel(prec, fast, [&](auto kern, int threads) {
        hipLaunchKernelGGL(kern, dim3((unsigned)grid), dim3(threads), 0, st, a, round, nitems, mixed ? 1 : 0);
        return hipGetLastError();
    });
}

hipError_t launch_batch_reduce(const BatchStep *steps, const int *summed, int count, const double *partials,
                               double *sums, hipStream_t st)
{
    hipLaunchKernelGGL(batch_reduce_kernel, dim3((unsigned)count), dim3(256), 0, st, steps, summed, partials, sums);
    return hipGetLastError();
}

}  // namespace qs
