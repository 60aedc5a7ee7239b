// Reductions over the state: measurement probabilities (Sec. 2.4) with the
// FP64 total, and Z-string expectation values accumulated in FP64.
//
// Both kernels stream the state once with 16-byte loads, keep one FP64
// partial sum per lane, reduce a wavefront with cross-lane shuffles and a
// workgroup through LDS, and write one partial per workgroup; a one-block
// kernel adds the partials in a fixed order, so results are deterministic.
#include "sv_internal.hpp"

#include <algorithm>
#include <cmath>
#include <mutex>

namespace sv {

constexpr int kRedThreads = 256;

__device__ __forceinline__ double wave_sum(double x) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) x += __shfl_xor(x, off, 64);
    return x;
}

__device__ __forceinline__ double block_sum(double x, double *sh) {
    x = wave_sum(x);
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    if (lane == 0) sh[wid] = x;
    __syncthreads();
    double r = 0.0;
    if (threadIdx.x == 0)
        for (int w = 0; w < (int)(blockDim.x >> 6); ++w) r += sh[w];
    __syncthreads();
    return r;
}

__global__ __launch_bounds__(kRedThreads) void k_sum_partials(const double *partials, int n,
                                                              double *total) {
    __shared__ double sh[kRedThreads / 64];
    double acc = 0.0;
    for (int i = threadIdx.x; i < n; i += kRedThreads) acc += partials[i];
    acc = block_sum(acc, sh);
    if (threadIdx.x == 0) *total = acc;
}

// Every thread keeps kRedUnroll 16-byte nontemporal loads in flight per
// round (rounds stride over the grid): measured 7.0 TB/s for a read-only
// stream of a 32 GiB state with 8192 workgroups, against 5.5 TB/s with one
// load per round.
constexpr int kRedUnroll = 8;

// complex64: one float4 = amplitudes 2e, 2e+1 -> probabilities as float2.
__global__ __launch_bounds__(kRedThreads) void k_probs_c64(const float4 *__restrict__ v,
                                                           uint64_t n_vec, float2 *__restrict__ out,
                                                           double *partials) {
    __shared__ double sh[kRedThreads / 64];
    double acc = 0.0;
    const uint64_t per = (uint64_t)kRedUnroll * kRedThreads;
    for (uint64_t base = (uint64_t)blockIdx.x * per; base < n_vec; base += (uint64_t)gridDim.x * per) {
        float4 w[kRedUnroll];
#pragma unroll
        for (int u = 0; u < kRedUnroll; ++u) {
            const uint64_t e = base + (uint64_t)u * kRedThreads + threadIdx.x;
            w[u] = e < n_vec ? ld_nt(&v[e]) : float4{0.f, 0.f, 0.f, 0.f};
        }
#pragma unroll
        for (int u = 0; u < kRedUnroll; ++u) {
            const uint64_t e = base + (uint64_t)u * kRedThreads + threadIdx.x;
            const float p0 = fmaf(w[u].x, w[u].x, w[u].y * w[u].y), p1 = fmaf(w[u].z, w[u].z, w[u].w * w[u].w);
            if (out && e < n_vec) {
                typedef float f32x2_nt __attribute__((ext_vector_type(2)));
                const f32x2_nt pv = {p0, p1};
                __builtin_nontemporal_store(pv, reinterpret_cast<f32x2_nt *>(&out[e]));
            }
            acc += (double)w[u].x * w[u].x + (double)w[u].y * w[u].y + (double)w[u].z * w[u].z +
                   (double)w[u].w * w[u].w;
        }
    }
    acc = block_sum(acc, sh);
    if (threadIdx.x == 0) partials[blockIdx.x] = acc;
}

__global__ __launch_bounds__(kRedThreads) void k_probs_c128(const double2 *__restrict__ v,
                                                            uint64_t n, double *__restrict__ out,
                                                            double *partials) {
    __shared__ double sh[kRedThreads / 64];
    double acc = 0.0;
    const uint64_t per = (uint64_t)kRedUnroll * kRedThreads;
    for (uint64_t base = (uint64_t)blockIdx.x * per; base < n; base += (uint64_t)gridDim.x * per) {
        double2 w[kRedUnroll];
#pragma unroll
        for (int u = 0; u < kRedUnroll; ++u) {
            const uint64_t e = base + (uint64_t)u * kRedThreads + threadIdx.x;
            w[u] = e < n ? ld_nt(&v[e]) : double2{0.0, 0.0};
        }
#pragma unroll
        for (int u = 0; u < kRedUnroll; ++u) {
            const uint64_t e = base + (uint64_t)u * kRedThreads + threadIdx.x;
            const double p = fma(w[u].x, w[u].x, w[u].y * w[u].y);
            if (out && e < n) __builtin_nontemporal_store(p, &out[e]);
            acc += p;
        }
    }
    acc = block_sum(acc, sh);
    if (threadIdx.x == 0) partials[blockIdx.x] = acc;
}

static unsigned red_grid(uint64_t work, int n_partials) {
    const uint64_t per = (uint64_t)kRedUnroll * kRedThreads;
    uint64_t b = (work + per - 1) / per;
    return (unsigned)std::max<uint64_t>(1, std::min<uint64_t>(b, (uint64_t)n_partials));
}

hipError_t launch_probabilities(const void *amps, int n, int dtype, void *dev_out,
                                double *dev_partials, int n_partials, double *dev_total,
                                hipStream_t s) {
    const uint64_t N = 1ull << n;
    unsigned grid;
    if (dtype == SV_C64) {
        grid = red_grid(N / 2, n_partials);
        k_probs_c64<<<dim3(grid), dim3(kRedThreads), 0, s>>>((const float4 *)amps, N / 2, (float2 *)dev_out, dev_partials);
    } else {
        grid = red_grid(N, n_partials);
        k_probs_c128<<<dim3(grid), dim3(kRedThreads), 0, s>>>((const double2 *)amps, N, (double *)dev_out, dev_partials);
    }
    k_sum_partials<<<dim3(1), dim3(kRedThreads), 0, s>>>(dev_partials, (int)grid, dev_total);
    return hipGetLastError();
}

// ----------------------------------------------------------- expectation
// Terms of the observable, split by where a mask's bits meet the reduction's
// index: amplitude x = (base + u * kRedThreads + thread) * A + k for round
// base, unrolled vector u and amplitude k of the A in a vector.  'reg' is the
// mask on the register index (u, k), 'lane' on the thread, 'base' on the
// rest (uniform over the workgroup).  Terms are sorted by reg: those with
// mask r are [start[r], start[r + 1]).
constexpr int kRedUnrollBits = 3, kRedThreadBits = 8;
static_assert(kRedUnroll == 1 << kRedUnrollBits && kRedThreads == 1 << kRedThreadBits, "index bits");
constexpr int kMaxRegBits = kRedUnrollBits + 1; // complex64: two amplitudes per vector
struct Terms {
    int n;
    int one_reg;   // the terms' reg mask if all share it, else -1
    int direct;    // a coefficient is not finite: evaluate h(x) per amplitude
    int start[(1 << kMaxRegBits) + 1];
    uint32_t lane[kMaxTerms];
    uint64_t base[kMaxTerms];
    uint64_t mask[kMaxTerms];
    double coeff[kMaxTerms];
};

__device__ __forceinline__ double zsum(const Terms &t, uint64_t x) {
    double h = 0.0;
    for (int j = 0; j < t.n; ++j) {
        const double c = t.coeff[j];
        h += (__popcll(x & t.mask[j]) & 1) ? -c : c;
    }
    return h;
}

template <typename T>
struct RedVec;
template <>
struct RedVec<float> {
    using type = float4;
    static constexpr int bits = 1;
    __device__ static void probs(const float4 &w, double *p) {
        p[0] = (double)w.x * w.x + (double)w.y * w.y;
        p[1] = (double)w.z * w.z + (double)w.w * w.w;
    }
};
template <>
struct RedVec<double> {
    using type = double2;
    static constexpr int bits = 0;
    __device__ static void probs(const double2 &w, double *p) { p[0] = fma(w.x, w.x, w.y * w.y); }
};

// sum_x p_x h(x) over the whole state, h(x) = sum_j c_j (-1)^popcount(x & m_j).
// Per round a thread holds D = 8 or 16 probabilities that differ in the
// register index only.  With W_r = sum_i p_i (-1)^popcount(i & r) their
// Walsh-Hadamard transform (D log2 D additions), every term is one sign
// flip and one addition to its W_r's coefficient, so the work per amplitude
// no longer grows with the number of terms: 28 terms (a ZZ ring) on 2^29
// complex64 amplitudes took 5.4 ms with h(x) evaluated per amplitude (bound
// by the vector ALUs) and take 0.7 ms as a transform (HBM: 6 TB/s).  ONE:
// all terms share one register mask (a lone Z string does), so only that
// W_r is formed, by multiplying with D uniform signs.
// A probability that is not finite makes differences of W undefined where
// the sum itself is not: such a round is evaluated amplitude by amplitude.
template <typename T, bool ONE>
__global__ __launch_bounds__(kRedThreads) void k_expect(const typename RedVec<T>::type *__restrict__ v,
                                                        uint64_t n_vec, Terms t, double *partials) {
    using V = RedVec<T>;
    constexpr int D = kRedUnroll << V::bits, A = 1 << V::bits;
    __shared__ double sh[kRedThreads / 64];
    const uint64_t per = (uint64_t)kRedUnroll * kRedThreads;
    uint64_t flip_lane = 0; // bit j: the thread's share of term j's sign
    for (int j = 0; j < t.n; ++j)
        flip_lane |= (uint64_t)(__popc(threadIdx.x & t.lane[j]) & 1) << j;
    double sg[ONE ? D : 1];
    if constexpr (ONE) {
#pragma unroll
        for (int i = 0; i < D; ++i) sg[i] = (__builtin_popcount(i & t.one_reg) & 1) ? -1.0 : 1.0;
    }
    double acc = 0.0;
    for (uint64_t base = (uint64_t)blockIdx.x * per; base < n_vec; base += (uint64_t)gridDim.x * per) {
        typename V::type w[kRedUnroll];
#pragma unroll
        for (int u = 0; u < kRedUnroll; ++u) {
            const uint64_t e = base + (uint64_t)u * kRedThreads + threadIdx.x;
            w[u] = e < n_vec ? ld_nt(&v[e]) : typename V::type{};
        }
        uint64_t flip = 0;
        for (int j = 0; j < t.n; ++j) flip |= (uint64_t)(__popcll(base & t.base[j]) & 1) << j;
        flip ^= flip_lane;
        // +-c_j summed over the terms of one register mask
        auto coeff = [&](int j0, int j1) {
            double h = 0.0;
            for (int j = j0; j < j1; ++j)
                h += __longlong_as_double(__double_as_longlong(t.coeff[j]) ^ (long long)((flip >> j) << 63));
            return h;
        };
        double p[D];
#pragma unroll
        for (int u = 0; u < kRedUnroll; ++u) V::probs(w[u], p + A * u);
        double total = 0.0, part = 0.0;
        if constexpr (ONE) {
#pragma unroll
            for (int i = 0; i < D; ++i) {
                total += p[i];
                part = fma(p[i], sg[i], part);
            }
            part *= coeff(0, t.n);
        } else {
#pragma unroll
            for (int b = 1; b < D; b <<= 1)
#pragma unroll
                for (int i = 0; i < D; ++i)
                    if (!(i & b)) {
                        const double x = p[i], y = p[i | b];
                        p[i] = x + y;
                        p[i | b] = x - y;
                    }
            total = p[0];
#pragma unroll
            for (int r = 0; r < D; ++r)
                if (t.start[r] < t.start[r + 1]) part = fma(p[r], coeff(t.start[r], t.start[r + 1]), part);
        }
        if (t.direct || !(total < __builtin_inf())) {
            part = 0.0;
            for (int u = 0; u < kRedUnroll; ++u) {
                const uint64_t e = base + (uint64_t)u * kRedThreads + threadIdx.x;
                if (e >= n_vec) continue;
                double q[A];
                V::probs(v[e], q);
                for (int k = 0; k < A; ++k) part += q[k] * zsum(t, (e << V::bits) | (uint64_t)k);
            }
        }
        acc += part;
    }
    acc = block_sum(acc, sh);
    if (threadIdx.x == 0) partials[blockIdx.x] = acc;
}

// Split and sort the terms for vectors of 2^vb amplitudes.
static Terms make_terms(int n_terms, const uint64_t *masks, const double *coeffs, int vb) {
    Terms t{};
    t.n = n_terms;
    const uint64_t amp = (1ull << vb) - 1ull, unroll = (uint64_t)kRedUnroll - 1ull;
    auto reg = [&](uint64_t m) {
        return (int)((m & amp) | (((m >> (vb + kRedThreadBits)) & unroll) << vb));
    };
    int at = 0;
    for (int r = 0; r < (1 << kMaxRegBits); ++r) {
        t.start[r] = at;
        for (int j = 0; j < n_terms; ++j) {
            if (reg(masks[j]) != r) continue;
            t.lane[at] = (uint32_t)(masks[j] >> vb) & (uint32_t)(kRedThreads - 1);
            t.base[at] = (masks[j] >> (vb + kRedThreadBits + kRedUnrollBits)) << (kRedThreadBits + kRedUnrollBits);
            t.mask[at] = masks[j];
            t.coeff[at] = coeffs[j];
            if (!std::isfinite(coeffs[j])) t.direct = 1;
            ++at;
        }
    }
    t.start[1 << kMaxRegBits] = at;
    t.one_reg = reg(masks[0]);
    for (int j = 1; j < n_terms; ++j)
        if (reg(masks[j]) != t.one_reg) t.one_reg = -1;
    return t;
}

template <typename T>
static void launch_expect_t(const void *amps, uint64_t n_vec, const Terms &t, unsigned grid, double *partials,
                            hipStream_t s) {
    const auto *v = (const typename RedVec<T>::type *)amps;
    if (t.one_reg >= 0) k_expect<T, true><<<dim3(grid), dim3(kRedThreads), 0, s>>>(v, n_vec, t, partials);
    else k_expect<T, false><<<dim3(grid), dim3(kRedThreads), 0, s>>>(v, n_vec, t, partials);
}

hipError_t launch_expectation(const void *amps, int n, int dtype, int n_terms,
                              const uint64_t *masks, const double *coeffs, double *dev_partials,
                              int n_partials, double *dev_total, hipStream_t s) {
    if (n_terms < 1 || n_terms > kMaxTerms) return hipErrorInvalidValue;
    const int vb = dtype == SV_C64 ? 1 : 0;
    const Terms t = make_terms(n_terms, masks, coeffs, vb);
    const uint64_t n_vec = (1ull << n) >> vb;
    const unsigned grid = red_grid(n_vec, n_partials);
    if (dtype == SV_C64) launch_expect_t<float>(amps, n_vec, t, grid, dev_partials, s);
    else launch_expect_t<double>(amps, n_vec, t, grid, dev_partials, s);
    k_sum_partials<<<dim3(1), dim3(kRedThreads), 0, s>>>(dev_partials, (int)grid, dev_total);
    return hipGetLastError();
}

// ------------------------------------------- reduction without allocation
// Partial sums of sv_expectation_noalloc: one FP64 per reduction workgroup
// (kReduceBlocks of them, 64 KiB).  Every device the library runs on holds its
// own copy until the process ends.  In host code the array's name only
// stands for the symbol: its device address, which differs per device, is
// taken once per device with hipGetSymbolAddress and used for every kernel
// argument.  Calls on one device share the array, so calls that overlap on
// one device (two streams) race; calls ordered on one stream do not.  Every
// launch writes each partial it later reads, so nothing needs clearing.
static __device__ __align__(256) double scratch[kReduceBlocks];

constexpr int kMaxScratchDevices = 64;
static std::mutex g_scratch_mu;
static double *g_scratch_addr[kMaxScratchDevices] = {};

static hipError_t scratch_address(double **out) {
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= kMaxScratchDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (!g_scratch_addr[dev]) {
        void *p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        g_scratch_addr[dev] = static_cast<double *>(p);
    }
    *out = g_scratch_addr[dev];
    return hipSuccess;
}

hipError_t launch_expectation_static(const void *amps, int n, int dtype, int n_terms,
                                     const uint64_t *masks, const double *coeffs, double *dev_total,
                                     hipStream_t s) {
    double *partials = nullptr;
    const hipError_t e = scratch_address(&partials);
    if (e != hipSuccess) return e;
    // red_grid never exceeds the partial count it is given: the array's size
    static_assert(sizeof(scratch) == kReduceBlocks * sizeof(double), "one partial per workgroup");
    return launch_expectation(amps, n, dtype, n_terms, masks, coeffs, partials, kReduceBlocks, dev_total, s);
}

} // namespace sv
