// Measurement in the computational basis (Sec. 1.3.3, Sec. 2.4): outcome
// probabilities of a few qubits, projection onto an outcome with
// renormalisation, and full-register sampling by the inverse cumulative
// distribution.  All sums are FP64 and run in a fixed order, so results are
// deterministic.
#include "sv_internal.hpp"
#include "tile_sweep.hpp"

#include <algorithm>

namespace sv {

constexpr int kMeasThreads = 256;

__device__ __forceinline__ double meas_wave_sum(double x) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) x += __shfl_xor(x, off, 64);
    return x;
}

template <typename T>
__device__ __forceinline__ double pr(const cpx<T> &a) {
    return (double)a.re * a.re + (double)a.im * a.im;
}

template <typename T>
__device__ __forceinline__ cpx<T> amp_of(const typename Amp16<T>::type &w, int i) {
    if constexpr (sizeof(T) == 4) return i == 0 ? cpx<T>{w.x, w.y} : cpx<T>{w.z, w.w};
    else return cpx<T>{w.x, w.y};
}

// Outcome index of x: bit i = bit pos[i] of x.
__device__ __forceinline__ uint32_t outcome_bits(uint64_t x, const MeasurePos &mp) {
    uint32_t o = 0;
#pragma unroll
    for (int i = 0; i < kMaxMeasureQubits; ++i)
        if (i < mp.k) o |= (uint32_t)((x >> mp.pos[i]) & 1ull) << i;
    return o;
}

// ------------------------------------------------------------- marginals
// Every thread keeps its own 2^k FP64 bins in LDS (bin b of thread t at
// b * kMeasThreads + t: consecutive lanes, consecutive banks), the
// workgroup then sums each bin over its threads in order.  Bound by the read
// of the state: kMeasUnroll nontemporal loads in flight per thread, and the
// outcome of a vector is a part of the thread's own bits, set once, and a
// part that the workgroup shares, on the scalar unit.  27 qubits complex128,
// 4 qubits measured: 354 us, 400 with one load per round.
constexpr int kMeasUnroll = 8;
constexpr int kMeasThreadBits = 8;
static_assert(kMeasThreads == 1 << kMeasThreadBits, "index bits");
template <typename T>
__global__ __launch_bounds__(kMeasThreads) void k_marginals(const typename Amp16<T>::type *__restrict__ v,
                                                            uint64_t n_vec, MeasurePos mp, double *partials) {
    extern __shared__ double bins[];
    constexpr int vb = Amp16<T>::bits;
    const int nb = 1 << mp.k;
    for (int b = 0; b < nb; ++b) bins[b * kMeasThreads + threadIdx.x] = 0.0;
    uint32_t own[1 << vb];
#pragma unroll
    for (int i = 0; i < (1 << vb); ++i) own[i] = outcome_bits(((uint64_t)threadIdx.x << vb) + i, mp);
    constexpr uint64_t per = (uint64_t)kMeasUnroll * kMeasThreads;
    for (uint64_t base = (uint64_t)blockIdx.x * per; base < n_vec; base += (uint64_t)gridDim.x * per) {
        typename Amp16<T>::type w[kMeasUnroll];
#pragma unroll
        for (int u = 0; u < kMeasUnroll; ++u) {
            const uint64_t e = base + (uint64_t)u * kMeasThreads + threadIdx.x;
            w[u] = e < n_vec ? ld_nt(&v[e]) : typename Amp16<T>::type{};
        }
#pragma unroll
        for (int u = 0; u < kMeasUnroll; ++u) {
            const uint32_t shared = outcome_bits((base + (uint64_t)u * kMeasThreads) << vb, mp);
#pragma unroll
            for (int i = 0; i < (1 << vb); ++i)
                bins[(shared | own[i]) * kMeasThreads + threadIdx.x] += pr(amp_of<T>(w[u], i));
        }
    }
    __syncthreads();
    for (int b = threadIdx.x; b < nb; b += kMeasThreads) {
        double s = 0.0;
        for (int t = 0; t < kMeasThreads; ++t) s += bins[b * kMeasThreads + t];
        partials[(size_t)b * gridDim.x + blockIdx.x] = s;
    }
}

// ------------------------------------------------- masked probability
template <typename T>
__global__ __launch_bounds__(kMeasThreads) void k_masked_prob(const typename Amp16<T>::type *__restrict__ v,
                                                              uint64_t n_vec, uint64_t mask, uint64_t want,
                                                              double *partials) {
    __shared__ double sh[kMeasThreads / 64];
    double acc = 0.0;
    const uint64_t stride = (uint64_t)gridDim.x * kMeasThreads;
    for (uint64_t e = (uint64_t)blockIdx.x * kMeasThreads + threadIdx.x; e < n_vec; e += stride) {
        const typename Amp16<T>::type w = v[e];
#pragma unroll
        for (int i = 0; i < (sizeof(T) == 4 ? 2 : 1); ++i) {
            const uint64_t x = (e << Amp16<T>::bits) + i;
            if ((x & mask) == want) acc += pr(amp_of<T>(w, i));
        }
    }
    acc = meas_wave_sum(acc);
    if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = acc;
    __syncthreads();
    if (threadIdx.x == 0) {
        double s = 0.0;
        for (int i = 0; i < kMeasThreads / 64; ++i) s += sh[i];
        partials[blockIdx.x] = s;
    }
}

// --------------------------------------------------------------- collapse
// psi_x * scale on the outcome, zero elsewhere.  Only vectors that hold an
// amplitude of the outcome are read: the write of the state bounds this (4
// of 27 qubits complex128: 400 us, 778 reading all of it).
constexpr int kCollapseUnroll = 4;
template <typename T>
__global__ __launch_bounds__(kMeasThreads) void k_collapse(typename Amp16<T>::type *__restrict__ v, uint64_t n_vec,
                                                           uint64_t mask, uint64_t want, T scale) {
    constexpr int vb = Amp16<T>::bits;
    constexpr uint64_t vmask = (1ull << vb) - 1ull; // index bits within a vector
    constexpr uint64_t per = (uint64_t)kCollapseUnroll * kMeasThreads;
    for (uint64_t base = (uint64_t)blockIdx.x * per; base < n_vec; base += (uint64_t)gridDim.x * per) {
        typename Amp16<T>::type w[kCollapseUnroll];
#pragma unroll
        for (int u = 0; u < kCollapseUnroll; ++u) {
            const uint64_t e = base + (uint64_t)u * kMeasThreads + threadIdx.x;
            const bool some = e < n_vec && (((e << vb) ^ want) & mask & ~vmask) == 0;
            w[u] = some ? ld_nt(&v[e]) : typename Amp16<T>::type{};
        }
#pragma unroll
        for (int u = 0; u < kCollapseUnroll; ++u) {
            const uint64_t e = base + (uint64_t)u * kMeasThreads + threadIdx.x;
            if (e >= n_vec) continue;
            const uint64_t x = e << vb;
            const bool in0 = (x & mask) == want;
            if constexpr (vb == 1) {
                const bool in1 = ((x + 1) & mask) == want;
                w[u] = float4{in0 ? w[u].x * scale : 0.f, in0 ? w[u].y * scale : 0.f, in1 ? w[u].z * scale : 0.f,
                              in1 ? w[u].w * scale : 0.f};
            } else {
                w[u] = double2{in0 ? w[u].x * scale : 0.0, in0 ? w[u].y * scale : 0.0};
            }
            v[e] = w[u];
        }
    }
}

// --------------------------------------------------------------- sampling
// Sum of each contiguous block of 2^block_log amplitudes (one workgroup per
// block).  27 qubits complex128: 310 us, 405 with one load in flight per
// thread.
template <typename T>
__global__ __launch_bounds__(kMeasThreads) void k_block_sums(const typename Amp16<T>::type *__restrict__ v,
                                                             int block_log, uint64_t n_blocks, double *sums) {
    __shared__ double sh[kMeasThreads / 64];
    constexpr int vb = Amp16<T>::bits;
    const uint64_t n_vec = (1ull << block_log) >> vb;
    for (uint64_t b = blockIdx.x; b < n_blocks; b += gridDim.x) {
        const typename Amp16<T>::type *p = v + b * n_vec;
        double acc = 0.0;
        for (uint64_t i0 = 0; i0 < n_vec; i0 += (uint64_t)kMeasUnroll * kMeasThreads) {
            typename Amp16<T>::type w[kMeasUnroll];
#pragma unroll
            for (int u = 0; u < kMeasUnroll; ++u) {
                const uint64_t i = i0 + (uint64_t)u * kMeasThreads + threadIdx.x;
                w[u] = i < n_vec ? ld_nt(&p[i]) : typename Amp16<T>::type{};
            }
#pragma unroll
            for (int u = 0; u < kMeasUnroll; ++u)
#pragma unroll
                for (int k = 0; k < (1 << vb); ++k) acc += pr(amp_of<T>(w[u], k));
        }
        acc = meas_wave_sum(acc);
        if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = acc;
        __syncthreads();
        if (threadIdx.x == 0) {
            double s = 0.0;
            for (int i = 0; i < kMeasThreads / 64; ++i) s += sh[i];
            sums[b] = s;
        }
        __syncthreads();
    }
}

// Cumulative sums of the blocks in two steps: a thread adds one run of
// kRunBlocks blocks (a line of sums), then one workgroup forms pre[r], the
// mass before run r, and pre[n_runs], the total.  There a thread adds its
// runs in order, one thread the threads' sums in order, and each thread
// writes its prefixes from the same operands, so that they never decrease
// and a run without mass has pre[r] == pre[r + 1]: no target falls into it.
// On the host, with the copy of 2^16 sums and a second round trip for the
// targets, this took 420 us; in one workgroup, whose threads read a run of 64
// sums each, 111; here 25.
constexpr int kRunBlocks = 16, kPrefixThreads = 1024, kPrefixRuns = 4;
__global__ __launch_bounds__(64) void k_run_sums(const double *__restrict__ sums, int per, int n_runs,
                                                 double *__restrict__ runs) {
    const int r = blockIdx.x * 64 + threadIdx.x;
    if (r >= n_runs) return;
    double s = 0.0;
#pragma unroll
    for (int k = 0; k < kRunBlocks; ++k)
        if (k < per) s += sums[r * per + k];
    runs[r] = s;
}

__global__ __launch_bounds__(kPrefixThreads) void k_run_prefix(const double *__restrict__ runs, int n_runs,
                                                               double *__restrict__ pre) {
    __shared__ double run[kPrefixThreads + 1];
    const int t = threadIdx.x;
    double x[kPrefixRuns], s = 0.0;
#pragma unroll
    for (int k = 0; k < kPrefixRuns; ++k) {
        x[k] = t * kPrefixRuns + k < n_runs ? runs[t * kPrefixRuns + k] : 0.0;
        s += x[k];
    }
    run[t + 1] = s;
    __syncthreads();
    if (t == 0) {
        double c = 0.0;
        run[0] = 0.0;
#pragma unroll 32
        for (int i = 1; i <= (n_runs + kPrefixRuns - 1) / kPrefixRuns; ++i) { // the threads that hold runs
            c += run[i];
            run[i] = c;
        }
        pre[n_runs] = c;
    }
    __syncthreads();
    const double from = run[t];
    double part = 0.0;
#pragma unroll
    for (int k = 0; k < kPrefixRuns; ++k) {
        if (t * kPrefixRuns + k < n_runs) pre[t * kPrefixRuns + k] = from + part;
        part += x[k];
    }
}

// One wave per sample.  Its target is u times the total; its run of blocks
// is the first whose cumulative end exceeds the target (64 ends per step of
// the search), or the last one with mass if rounding leaves none, its block
// is found in the run likewise, and it then scans the block 64 amplitudes at
// a time
// (FP64 inclusive prefix across the wave plus the running sum) and take the
// first amplitude whose cumulative sum exceeds the sample's target; if
// rounding leaves none, the block's last amplitude with p > 0.
template <typename T>
__global__ __launch_bounds__(kMeasThreads) void k_sample_scan(const cpx<T> *__restrict__ v, int block_log,
                                                              int n_samples, int per, int n_runs,
                                                              const double *__restrict__ sums,
                                                              const double *__restrict__ pre,
                                                              const double *__restrict__ uniforms,
                                                              uint64_t *__restrict__ out) {
    const int lane = threadIdx.x & 63;
    const int s = (int)((blockIdx.x * kMeasThreads + threadIdx.x) >> 6);
    if (s >= n_samples) return; // whole waves leave together
    const uint64_t bsize = 1ull << block_log;
    const double total = pre[n_runs];
    if (!(total > 0.0)) return; // reported by the host
    const double goal = uniforms[s] * total;
    const bool beyond = !(total > goal);
    int r = 0;
    for (int len = n_runs; len > 1;) {
        const int step = len > 64 ? len >> 6 : 1;
        const bool in = (lane + 1) * step <= len;
        const double end = in ? pre[r + (lane + 1) * step] : 0.0;
        const uint64_t hit = __ballot(in && (beyond ? end >= total : end > goal));
        r += (hit ? __builtin_ctzll(hit) : 0) * step;
        len = step;
    }
    const double mass = lane < per ? sums[r * per + lane] : 0.0;
    const double from = pre[r];
    double part = 0.0, before = 0.0;
    int blk = -1, last_mass = 0;
    for (int k = 0; k < per && blk < 0; ++k) {
        const double x = __shfl(mass, k, 64);
        if (x > 0.0) {
            last_mass = k;
            before = part;
        }
        part += x;
        if (from + part > goal) blk = k;
    }
    if (blk < 0) blk = last_mass;
    const uint64_t base = (uint64_t)(r * per + blk) << block_log;
    const double t = goal - (from + before);
    double run = 0.0;
    int64_t last = -1;
    int64_t found = -1;
    for (uint64_t c = 0; c < bsize; c += 64) {
        const uint64_t i = c + lane;
        const double p = i < bsize ? pr(v[base + i]) : 0.0;
        double inc = p;
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
            const double y = __shfl_up(inc, off, 64);
            if (lane >= off) inc += y;
        }
        const uint64_t hit = __ballot(run + inc > t);
        if (hit) {
            found = (int64_t)(c + __builtin_ctzll(hit));
            break;
        }
        const uint64_t nz = __ballot(p > 0.0);
        if (nz) last = (int64_t)(c + 63 - __builtin_clzll(nz));
        run += __shfl(inc, 63, 64);
    }
    if (lane == 0) out[s] = base + (uint64_t)(found >= 0 ? found : (last >= 0 ? last : 0));
}

// ---------------------------------------------------------------- launchers
static unsigned stream_grid(uint64_t n_vec) {
    return (unsigned)std::max<uint64_t>(1, std::min<uint64_t>((n_vec + kMeasThreads - 1) / kMeasThreads, 1024));
}

int marginal_blocks(int n, int dtype) {
    const uint64_t n_vec = (1ull << n) >> (dtype == SV_C64 ? 1 : 0);
    return (int)stream_grid(std::max<uint64_t>(n_vec, 1));
}

hipError_t launch_marginals(const void *amps, int n, int dtype, const MeasurePos &mp, double *partials,
                            hipStream_t s) {
    if (mp.k < 1 || mp.k > kMaxMeasureQubits) return hipErrorInvalidValue;
    const int vb = dtype == SV_C64 ? 1 : 0;
    if (n < vb) return hipErrorInvalidValue;
    const uint64_t n_vec = (1ull << n) >> vb;
    const unsigned grid = stream_grid(n_vec);
    const size_t lds = (size_t)(1u << mp.k) * kMeasThreads * sizeof(double);
    if (dtype == SV_C64) {
        (void)hipFuncSetAttribute((const void *)k_marginals<float>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        k_marginals<float><<<grid, kMeasThreads, lds, s>>>((const float4 *)amps, n_vec, mp, partials);
    } else {
        (void)hipFuncSetAttribute((const void *)k_marginals<double>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        k_marginals<double><<<grid, kMeasThreads, lds, s>>>((const double2 *)amps, n_vec, mp, partials);
    }
    return hipGetLastError();
}

hipError_t launch_masked_prob(const void *amps, int n, int dtype, uint64_t mask, uint64_t want,
                              double *partials, hipStream_t s) {
    const int vb = dtype == SV_C64 ? 1 : 0;
    if (n < vb) return hipErrorInvalidValue;
    const uint64_t n_vec = (1ull << n) >> vb;
    const unsigned grid = stream_grid(n_vec);
    if (dtype == SV_C64)
        k_masked_prob<float><<<grid, kMeasThreads, 0, s>>>((const float4 *)amps, n_vec, mask, want, partials);
    else
        k_masked_prob<double><<<grid, kMeasThreads, 0, s>>>((const double2 *)amps, n_vec, mask, want, partials);
    return hipGetLastError();
}

hipError_t launch_collapse(void *amps, int n, int dtype, uint64_t mask, uint64_t want, double scale,
                           hipStream_t s) {
    const int vb = dtype == SV_C64 ? 1 : 0;
    if (n < vb) return hipErrorInvalidValue;
    const uint64_t n_vec = (1ull << n) >> vb;
    const uint64_t per = (uint64_t)kCollapseUnroll * kMeasThreads;
    const unsigned grid = (unsigned)std::min<uint64_t>((n_vec + per - 1) / per, 1u << 20);
    if (dtype == SV_C64)
        k_collapse<float><<<grid, kMeasThreads, 0, s>>>((float4 *)amps, n_vec, mask, want, (float)scale);
    else
        k_collapse<double><<<grid, kMeasThreads, 0, s>>>((double2 *)amps, n_vec, mask, want, scale);
    return hipGetLastError();
}

int sample_block_log(int n) { return std::max(std::min(n, 8), n - 16); }

hipError_t launch_block_sums(const void *amps, int n, int dtype, int block_log, double *sums, hipStream_t s) {
    if (block_log > n || block_log < (dtype == SV_C64 ? 1 : 0)) return hipErrorInvalidValue;
    const uint64_t nbk = 1ull << (n - block_log);
    const unsigned grid = (unsigned)std::min<uint64_t>(nbk, 1u << 16);
    if (dtype == SV_C64)
        k_block_sums<float><<<grid, kMeasThreads, 0, s>>>((const float4 *)amps, block_log, nbk, sums);
    else
        k_block_sums<double><<<grid, kMeasThreads, 0, s>>>((const double2 *)amps, block_log, nbk, sums);
    return hipGetLastError();
}

static int sample_per(int n_blocks) { return std::min(n_blocks, kRunBlocks); }
int sample_runs(int n_blocks) { return n_blocks / sample_per(n_blocks); }

hipError_t launch_run_prefix(const double *sums, int n_blocks, double *runs, double *pre, hipStream_t s) {
    if (n_blocks < 1 || (n_blocks & (n_blocks - 1))) return hipErrorInvalidValue;
    const int n_runs = sample_runs(n_blocks);
    if (n_runs > kPrefixThreads * kPrefixRuns) return hipErrorInvalidValue;
    k_run_sums<<<(n_runs + 63) / 64, 64, 0, s>>>(sums, sample_per(n_blocks), n_runs, runs);
    k_run_prefix<<<1, kPrefixThreads, 0, s>>>(runs, n_runs, pre);
    return hipGetLastError();
}

hipError_t launch_sample_scan(const void *amps, int dtype, int block_log, int n_samples, int n_blocks,
                              const double *sums, const double *pre, const double *uniforms, uint64_t *out,
                              hipStream_t s) {
    if (n_samples <= 0) return hipSuccess;
    const unsigned grid = (unsigned)(((uint64_t)n_samples * 64 + kMeasThreads - 1) / kMeasThreads);
    const int per = sample_per(n_blocks), n_runs = sample_runs(n_blocks);
    if (dtype == SV_C64)
        k_sample_scan<float><<<grid, kMeasThreads, 0, s>>>((const cpx<float> *)amps, block_log, n_samples, per, n_runs,
                                                           sums, pre, uniforms, out);
    else
        k_sample_scan<double><<<grid, kMeasThreads, 0, s>>>((const cpx<double> *)amps, block_log, n_samples, per,
                                                            n_runs, sums, pre, uniforms, out);
    return hipGetLastError();
}

} // namespace sv
