// Batched circuits: one graph launch runs thousands of independent circuits
// of different widths.
//
// A circuit whose state fits in one LDS tile (up to 2^13 complex64 / 2^12
// complex128 amplitudes) starts from |0...0> directly in LDS, runs all its
// gates there and reduces its Z-string expectation without touching HBM: a
// persistent kernel's workgroups pop such circuits from a device queue (an
// atomic counter) in the host's longest-first order until it is empty.
// Wider circuits keep their states in HBM and advance together, one launch
// per pass index over the tiles of all of them; the first pass synthesises
// |0...0> instead of loading it, and the last writes one expectation partial
// per tile, which a final kernel adds up in tile order.
//
// With a wide circuit walked by one workgroup the batch took as long as its
// widest circuit alone, whatever the other compute units did: 1024 circuits
// of 10 to 18 qubits took 11.9 ms on the device, with one launch per pass
// 5.4 ms; 4096 circuits of 10 to 20 qubits 106 and 85 ms; one 20-qubit
// circuit alone 43 and 0.32 ms.
//
// A wide circuit starts on one amplitude and each pass spreads it over the
// qubits of its tiles.  The host knows from the gates which qubits the
// passes before this one have moved (BatchPass::live), so tiles that still
// hold only zeros are not listed: the first pass, which holds most of a
// ladder's gates, runs one tile of each circuit instead of 2 to 32 (0.36
// instead of 2.47 ms on the 1024 circuits; their whole run takes 2.55 ms
// with the later changes to the sweeps).  Listed and left at once by their
// workgroups they saved nothing: the tiles that remained were every 2nd to
// 32nd workgroup, which the dispatcher had dealt to the same XCD and compute
// units.
#include "sv_internal.hpp"
#include "tile_sweep.hpp"

#include <algorithm>
#include <type_traits>

namespace sv {

constexpr int kBatchThreads = 512;

__device__ __forceinline__ double bwave_sum(double x) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) x += __shfl_xor(x, off, 64);
    return x;
}

template <typename T>
__device__ __forceinline__ double zterm(cpx<T> a, uint64_t x, uint64_t zmask) {
    const double p = (double)a.re * a.re + (double)a.im * a.im;
    return (__popcll(x & zmask) & 1) ? -p : p;
}

// One pass of a circuit over one tile.  As in the gate tile pass, the first
// sweep takes its register groups straight from the source and the last
// hands them straight to the sink, so the tile crosses LDS only between
// sweeps: the source is |0...0> synthesised in registers on the circuit's
// first pass, else the state; the sink accumulates the Z-string terms on
// the last pass and stores the state unless that pass is the last and the
// states are not kept.  A thread owns at most one group per sweep
// (2^(m-W) <= kBatchThreads).  'dead' holds the qubits no earlier pass has
// moved: amplitudes with such a bit set are zero and are not read.
template <typename T, int W, bool TWOQ>
__device__ void batch_tile(cpx<T> *state, char *lds, int m, uint64_t base,
                           const TileSweep *__restrict__ sweeps, int n_sweeps, const char *__restrict__ recs,
                           bool synth, bool last_pass, bool store, uint64_t dead, uint64_t zmask,
                           double &zacc) {
    constexpr int D = 1 << W;
    const uint32_t n_groups = (1u << m) >> W;
    const uint32_t wave_first = __builtin_amdgcn_readfirstlane(threadIdx.x & ~63u);
    for (int si = 0; si < n_sweeps; ++si) {
        const TileSweep &S = sweeps[si];
        const bool first = si == 0, last = si == n_sweeps - 1;
        for (uint32_t g = threadIdx.x; g < n_groups; g += blockDim.x) {
            cpx<T> v[D];
            if (first) {
                const uint64_t row = base | group_columns(S.at_lane, g);
#pragma unroll
                for (int j = 0; j < D; ++j) {
                    const uint64_t x = row | register_columns<W>(S.at_reg, j);
                    if (synth) v[j] = cpx<T>{x == 0 ? T(1) : T(0), T(0)};
                    else v[j] = x & dead ? cpx<T>{T(0), T(0)} : state[x];
                }
            } else {
                lds_load_group<T, W>(lds, group_columns(S.in_lane, g), S.in_reg, v);
            }
            PhaseAcc<T, W> acc;
            acc.init();
            run_records<T, W, TWOQ>(v, acc, g, recs + S.rec_off, S.n_gates, base);
            // results that go to other groups' places wait until every group
            // of this sweep has been read
            if (S.perm && first == last) __syncthreads();
            if (last) {
                const uint64_t to = to_constant(S, recs, base) ^ group_columns(S.to_lane, g);
                if (last_pass) {
#pragma unroll
                    for (int j = 0; j < D; ++j)
                        zacc += zterm(v[j], base | (to ^ register_columns<W>(S.to_reg, j)), zmask);
                }
                if (store) {
#pragma unroll
                    for (int j = 0; j < D; ++j) state[base | (to ^ register_columns<W>(S.to_reg, j))] = v[j];
                }
            } else {
                lds_store_group<T, W>(lds, out_constant(S, recs, base) ^ group_columns(S.out_lane, g), S.out_reg, v);
            }
        }
        // waves without groups take part in the barrier above
        if (S.perm && first == last && wave_first >= n_groups) __syncthreads();
        __syncthreads();
    }
}

// Sum over the workgroup in a fixed order, in thread 0.
__device__ __forceinline__ double batch_sum(double x, double *s_red) {
    x = bwave_sum(x);
    if ((threadIdx.x & 63) == 0) s_red[threadIdx.x >> 6] = x;
    __syncthreads();
    double t = 0.0;
    if (threadIdx.x == 0)
        for (int w = 0; w < kBatchThreads / 64; ++w) t += s_red[w];
    __syncthreads();
    return t;
}

// The program's arrays are kernel arguments of their own, const and without
// aliases: the records are then read with scalar loads, as in the gate tile
// pass.  Read through the argument struct they came by vector loads and a
// readfirstlane per word.
#define SV_BATCH_PROGRAM                                                                           \
    const BatchCircuit *__restrict__ circuits, const BatchPass *__restrict__ passes,               \
        const TileSweep *__restrict__ sweeps, const char *__restrict__ recs

// LDS-resident circuits: one pass over one tile each.
template <typename T, int W, bool TWOQ>
__global__ __launch_bounds__(kBatchThreads) void k_batch(BatchArgs a, SV_BATCH_PROGRAM,
                                                         const int32_t *__restrict__ order) {
    extern __shared__ char lds[];
    __shared__ int s_idx;
    __shared__ double s_red[kBatchThreads / 64];
    for (;;) {
        if (threadIdx.x == 0) s_idx = (int)atomicAdd(a.counter, 1u);
        __syncthreads();
        // uniform, and known to be: the record walk stays on the scalar unit
        const int qi = __builtin_amdgcn_readfirstlane(s_idx);
        if (qi >= a.n_small) break; // uniform: every wave leaves together
        const int ci = order[qi];
        const BatchCircuit &c = circuits[ci];
        const BatchPass &p = passes[c.pass_off];
        warm_records(sweeps + p.sweep_off, p.n_sweeps * (uint32_t)sizeof(TileSweep));
        warm_records(recs + p.gate_off, p.rec_bytes);
        cpx<T> *state = reinterpret_cast<cpx<T> *>(reinterpret_cast<char *>(a.states) + c.state_off);
        double zacc = 0.0;
        batch_tile<T, W, TWOQ>(state, lds, c.w, 0, sweeps + p.sweep_off, p.n_sweeps, recs + p.gate_off,
                               true, true, c.keep, 0, a.zmask, zacc);
        zacc = batch_sum(zacc, s_red);
        if (threadIdx.x == 0) a.out[ci] = zacc;
        // Also keeps this store and the next pop apart: as neighbouring
        // blocks of thread 0 they were merged into a loop of their own, in
        // which the other threads went round again before the pop.
        __syncthreads();
    }
}

// Pass 'level' of every wide circuit that has one.
template <typename T, int W, bool TWOQ>
__global__ __launch_bounds__(kBatchThreads) void k_batch_wide(BatchArgs a, SV_BATCH_PROGRAM,
                                                              const int32_t *__restrict__ wide,
                                                              const BatchGroup *__restrict__ all_groups,
                                                              BatchLevel lv, int level) {
    extern __shared__ char lds[];
    __shared__ double s_red[kBatchThreads / 64];
    const BatchGroup *groups = all_groups + lv.group_off;
    for (int64_t item = blockIdx.x; item < lv.items; item += gridDim.x) {
        int g = 0;
        while (g + 1 < lv.n_groups && item >= groups[g + 1].first) ++g;
        const int64_t local = item - groups[g].first;
        const int tl = groups[g].tiles_log;
        const int ci = wide[groups[g].list_off + (int)(local >> tl)];
        const BatchCircuit &c = circuits[ci];
        const BatchPass &p = passes[c.pass_off + level];
        // bit i of the tile's number in the list is the i-th bit of p.tiles
        uint32_t tile = 0, rest = (uint32_t)local & ((1u << tl) - 1u);
        for (uint32_t b = p.tiles; b; b &= b - 1u, rest >>= 1)
            if (rest & 1u) tile |= b & (0u - b);
        if ((local & ((1ll << tl) - 1)) < 8) { // the first tiles, one on each XCD
            warm_records(sweeps + p.sweep_off, p.n_sweeps * (uint32_t)sizeof(TileSweep));
            warm_records(recs + p.gate_off, p.rec_bytes);
        }
        cpx<T> *state = reinterpret_cast<cpx<T> *>(reinterpret_cast<char *>(a.states) + c.state_off);
        uint64_t base = (uint64_t)tile << p.sp.L;
        for (int i = 0; i < p.sp.K; ++i) base = insert_zero(base, p.sp.high[i]);
        const bool last = level == c.n_passes - 1;
        const int m = p.sp.L + p.sp.K;
        const uint64_t dead = ~p.live;
        if (base & dead) { // a tile of zeros: no pass reads it before one has written it
            if (last && c.keep)
                for (uint32_t l = threadIdx.x; l < (1u << m); l += kBatchThreads)
                    state[base | tile_offset(p.sp, l)] = cpx<T>{T(0), T(0)};
            if (last && threadIdx.x == 0) a.parts[c.part_off + (int64_t)tile] = 0.0;
            continue;
        }
        double zacc = 0.0;
        batch_tile<T, W, TWOQ>(state, lds, m, base, sweeps + p.sweep_off, p.n_sweeps,
                               recs + p.gate_off, level == 0, last, !last || c.keep, dead, a.zmask, zacc);
        if (last) {
            zacc = batch_sum(zacc, s_red);
            if (threadIdx.x == 0) a.parts[c.part_off + (int64_t)tile] = zacc;
        }
    }
}

// Expectation of a wide circuit: its tiles' partials, in a fixed order.
__global__ __launch_bounds__(64) void k_batch_sum(BatchArgs a, int tile_m) {
    const int ci = a.wide[blockIdx.x];
    const BatchCircuit &c = a.circuits[ci];
    const int64_t n = 1ll << (c.w - tile_m);
    double x = 0.0;
    for (int64_t i = threadIdx.x; i < n; i += 64) x += a.parts[c.part_off + i];
    x = bwave_sum(x);
    if (threadIdx.x == 0) a.out[ci] = x;
}

__global__ void k_batch_reset(unsigned int *counter) { *counter = 0u; }

// A launch's threads must number fewer than 2^32.
constexpr int64_t kMaxWideGrid = 1 << 22;

template <typename T, int W, bool TWOQ>
static void launch_batch_t(const BatchArgs &args, const BatchLevel *levels, int n_levels, int tile_m, int grid,
                           size_t lds, hipStream_t s) {
    if (args.n_small) {
        (void)hipFuncSetAttribute((const void *)k_batch<T, W, TWOQ>, hipFuncAttributeMaxDynamicSharedMemorySize,
                                  (int)lds);
        k_batch_reset<<<1, 1, 0, s>>>(args.counter);
        k_batch<T, W, TWOQ><<<grid, kBatchThreads, lds, s>>>(args, args.circuits, args.passes, args.sweeps, args.recs,
                                                            args.order);
    }
    if (!args.n_wide) return;
    (void)hipFuncSetAttribute((const void *)k_batch_wide<T, W, TWOQ>, hipFuncAttributeMaxDynamicSharedMemorySize,
                              (int)lds);
    for (int l = 0; l < n_levels; ++l)
        k_batch_wide<T, W, TWOQ><<<(unsigned)std::min(levels[l].items, kMaxWideGrid), kBatchThreads, lds, s>>>(
            args, args.circuits, args.passes, args.sweeps, args.recs, args.wide, args.groups, levels[l], l);
    k_batch_sum<<<args.n_wide, 64, 0, s>>>(args, tile_m);
}

hipError_t launch_batch(const BatchArgs &args, const BatchLevel *levels, int n_levels, int dtype, int sweep_w,
                        int tile_m, int grid, bool two_qubit, hipStream_t s) {
    const size_t lds = (size_t)(1u << tile_m) * (dtype == SV_C64 ? 8 : 16);
#define SV_BATCH_CASE(TT, WW, Q)                                                                   \
    if ((dtype == SV_C64) == std::is_same<TT, float>::value && sweep_w == WW && two_qubit == Q) {  \
        launch_batch_t<TT, WW, Q>(args, levels, n_levels, tile_m, grid, lds, s);                   \
        return hipGetLastError();                                                                  \
    }
    SV_BATCH_CASE(float, 4, false)
    SV_BATCH_CASE(float, 3, false)
    SV_BATCH_CASE(double, 3, false)
    SV_BATCH_CASE(double, 4, false)
    SV_BATCH_CASE(float, 4, true)
    SV_BATCH_CASE(float, 3, true)
    SV_BATCH_CASE(double, 3, true)
    SV_BATCH_CASE(double, 4, true)
#undef SV_BATCH_CASE
    return hipErrorInvalidValue;
}

} // namespace sv
