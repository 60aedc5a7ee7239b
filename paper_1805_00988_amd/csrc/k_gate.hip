// Gate kernels: streamed pair/quad updates for gates on high qubits, a
// subspace-scaling kernel for phase-type diagonal gates, and the on-chip tile
// pass that applies a run of gates to tiles staged in LDS.
//
// Memory access: the state is read and written as 16-byte vectors (float4 =
// two complex64 amplitudes, double2 = one complex128 amplitude).  Consecutive
// lanes take consecutive vectors of the same half of the pair space, so every
// wavefront load is a contiguous run as long as the target qubit is above the
// vector width.
#include "sv_internal.hpp"
#include "tile_sweep.hpp"

#include <algorithm>
#include <cfloat>
#include <cmath>

namespace sv {

template <typename T>
struct Vec;
template <>
struct Vec<float> {
    using type = float4;
    static constexpr int amps = 2;
    static constexpr int bits = 1;
    __device__ static cpx<float> get(const float4 &v, int k) {
        return k == 0 ? cpx<float>{v.x, v.y} : cpx<float>{v.z, v.w};
    }
    __device__ static void put(float4 &v, int k, cpx<float> c) {
        if (k == 0) { v.x = c.re; v.y = c.im; } else { v.z = c.re; v.w = c.im; }
    }
};
template <>
struct Vec<double> {
    using type = double2;
    static constexpr int amps = 1;
    static constexpr int bits = 0;
    __device__ static cpx<double> get(const double2 &v, int) { return {v.x, v.y}; }
    __device__ static void put(double2 &v, int, cpx<double> c) { v.x = c.re; v.y = c.im; }
};

constexpr int kStreamThreads = 256;

// 16-byte access, nontemporal when NT.  Launchers pick NT only when every
// wavefront access is a run of at least 128 contiguous bytes: nontemporal
// accesses to interleaved shorter runs (a gate on the lowest qubits) were
// measured much slower.
template <bool NT, typename V>
__device__ __forceinline__ V ld16(const V *p) {
    if constexpr (NT) return ld_nt(p);
    else return *p;
}
template <bool NT, typename V>
__device__ __forceinline__ void st16(V *p, V v) {
    if constexpr (NT) st_nt(p, v);
    else *p = v;
}
constexpr int kMinNtRunBits = 3; // 2^3 16-byte vectors = 128 bytes

// Zero runs.  A register starts as a basis state, so until most qubits have
// been rotated nearly all of it is zero, and a gate maps zeros to zeros: a
// wave whose amplitudes are all zero leaves them as they are.  The accesses
// are what bounds these kernels, and the stores are half of them (a layer of
// 27 gates and 3 two-qubit unitaries on |0> at 29 qubits complex64: 52.2 ms
// storing everything, 22.5 ms).  The test covers whole waves, not lanes:
// lines written in part would be read back by the memory.  'skip' is off
// when a matrix entry is not finite in the state's precision (0 * inf).
static bool finite_as(int dtype, const double *U, int n) {
    for (int i = 0; i < n; ++i)
        if (!(std::fabs(U[i]) <= (dtype == SV_C64 ? (double)FLT_MAX : DBL_MAX))) return false;
    return true;
}

static inline uint64_t grid_for(uint64_t work_items, uint64_t per_block, uint64_t cap) {
    uint64_t b = (work_items + per_block - 1) / per_block;
    return std::max<uint64_t>(1, std::min<uint64_t>(b, cap));
}

// ---------------------------------------------------------------- init
// UNROLL vectors per thread and round; a grid of up to 2^20 workgroups
// covers a 32 GiB state in one round (measured faster than fewer
// workgroups looping).
template <typename T, int UNROLL>
__global__ __launch_bounds__(kStreamThreads) void k_init_basis(typename Vec<T>::type *v,
                                                               uint64_t n_vec, uint64_t x) {
    using V = Vec<T>;
    const uint64_t per_block = (uint64_t)UNROLL * kStreamThreads;
    for (uint64_t base = (uint64_t)blockIdx.x * per_block; base < n_vec;
         base += (uint64_t)gridDim.x * per_block) {
#pragma unroll
        for (int u = 0; u < UNROLL; ++u) {
            const uint64_t e = base + (uint64_t)u * kStreamThreads + threadIdx.x;
            if (e >= n_vec) break;
            typename V::type z;
            for (int k = 0; k < V::amps; ++k)
                V::put(z, k, cpx<T>{(((e << V::bits) | k) == x) ? T(1) : T(0), T(0)});
            v[e] = z;
        }
    }
}

hipError_t launch_init_basis(void *amps, int n, int dtype, uint64_t x, hipStream_t s) {
    const uint64_t N = 1ull << n;
    constexpr int U = 4;
    const uint64_t nv = dtype == SV_C64 ? N / 2 : N;
    const dim3 grid((unsigned)grid_for(nv, (uint64_t)U * kStreamThreads, 1ull << 20));
    if (dtype == SV_C64)
        k_init_basis<float, U><<<grid, dim3(kStreamThreads), 0, s>>>((float4 *)amps, nv, x);
    else
        k_init_basis<double, U><<<grid, dim3(kStreamThreads), 0, s>>>((double2 *)amps, nv, x);
    return hipGetLastError();
}

// ------------------------------------------------------- streamed 1q gate
// Element-pair j -> element a (bit te clear, control bits set) and a | 2^te.
// lane_ctrl holds control bits below the vector width (amplitude bits inside
// one 16-byte element): only amplitudes with all of them set are updated.
template <typename T, int UNROLL, bool NT>
__global__ __launch_bounds__(kStreamThreads) void k_gate1(typename Vec<T>::type *v, Enum e, int te,
                                                          uint64_t count, Mat2<T> g,
                                                          uint32_t lane_ctrl, bool skip) {
    using V = Vec<T>;
    const uint64_t per_block = (uint64_t)UNROLL * kStreamThreads;
    const uint64_t bstep = 1ull << te;
    for (uint64_t base = (uint64_t)blockIdx.x * per_block; base < count;
         base += (uint64_t)gridDim.x * per_block) {
        typename V::type va[UNROLL], vb[UNROLL];
        uint64_t ia[UNROLL];
        bool ok[UNROLL];
#pragma unroll
        for (int u = 0; u < UNROLL; ++u) {
            const uint64_t j = base + (uint64_t)u * kStreamThreads + threadIdx.x;
            const uint64_t a = expand(e, j < count ? j : 0);
            ok[u] = (j < count) && ((a & e.check) == e.check);
            ia[u] = a;
            if (ok[u]) {
                va[u] = ld16<NT>(&v[a]);
                vb[u] = ld16<NT>(&v[a + bstep]);
            }
        }
#pragma unroll
        for (int u = 0; u < UNROLL; ++u) {
            if (!ok[u]) continue;
            if (skip && wave_zero(magnitude_bits(va[u]) | magnitude_bits(vb[u]))) continue;
            typename V::type oa = va[u], ob = vb[u];
#pragma unroll
            for (int k = 0; k < V::amps; ++k) {
                if (((uint32_t)k & lane_ctrl) != lane_ctrl) continue;
                const cpx<T> x0 = V::get(va[u], k), x1 = V::get(vb[u], k);
                V::put(oa, k, cfma(g.m[0], x0, cmul(g.m[1], x1)));
                V::put(ob, k, cfma(g.m[2], x0, cmul(g.m[3], x1)));
            }
            st16<NT>(&v[ia[u]], oa);
            st16<NT>(&v[ia[u] + bstep], ob);
        }
    }
}

// complex64 gate on qubit 0: both amplitudes of a pair sit in one float4.
template <int UNROLL, bool NT>
__global__ __launch_bounds__(kStreamThreads) void k_gate1_q0(float4 *v, Enum e, uint64_t count,
                                                             Mat2<float> g, bool skip) {
    const uint64_t per_block = (uint64_t)UNROLL * kStreamThreads;
    for (uint64_t base = (uint64_t)blockIdx.x * per_block; base < count;
         base += (uint64_t)gridDim.x * per_block) {
        float4 w[UNROLL];
        uint64_t ia[UNROLL];
        bool ok[UNROLL];
#pragma unroll
        for (int u = 0; u < UNROLL; ++u) {
            const uint64_t j = base + (uint64_t)u * kStreamThreads + threadIdx.x;
            const uint64_t a = expand(e, j < count ? j : 0);
            ok[u] = (j < count) && ((a & e.check) == e.check);
            ia[u] = a;
            if (ok[u]) w[u] = ld16<NT>(&v[a]);
        }
#pragma unroll
        for (int u = 0; u < UNROLL; ++u) {
            if (!ok[u]) continue;
            if (skip && wave_zero(magnitude_bits(w[u]))) continue;
            const cpx<float> x0{w[u].x, w[u].y}, x1{w[u].z, w[u].w};
            const cpx<float> y0 = cfma(g.m[0], x0, cmul(g.m[1], x1));
            const cpx<float> y1 = cfma(g.m[2], x0, cmul(g.m[3], x1));
            st16<NT>(&v[ia[u]], float4{y0.re, y0.im, y1.re, y1.im});
        }
    }
}

// Build the element-level enumeration for a set of zero positions (element
// bit indices) plus control bits; controls beyond the insert capacity are
// checked instead of enumerated.
static Enum make_enum(int vbits, const int *zero_pos, int n_zero, uint64_t ctrl,
                      uint32_t *lane_ctrl, int *n_enumerated) {
    Enum e{};
    int pos[64];
    int np = 0;
    for (int i = 0; i < n_zero; ++i) pos[np++] = zero_pos[i];
    const uint64_t lane_mask = (1ull << vbits) - 1ull;
    *lane_ctrl = (uint32_t)(ctrl & lane_mask);
    uint64_t ec = ctrl >> vbits;
    e.set = 0;
    e.check = 0;
    while (ec) {
        const int b = __builtin_ctzll(ec);
        ec &= ec - 1;
        if (np < kMaxInsert) {
            pos[np++] = b;
            e.set |= 1ull << b;
        } else {
            e.check |= 1ull << b;
        }
    }
    std::sort(pos, pos + np);
    e.n_pos = np;
    for (int i = 0; i < np; ++i) e.pos[i] = pos[i];
    *n_enumerated = np;
    return e;
}

// Every enumerated element index lies in a run of 2^pos[0] consecutive
// vectors (the lowest inserted bit), and checked controls thin the runs out.
static bool nt_ok(const Enum &e) {
    return e.check == 0 && (e.n_pos == 0 || e.pos[0] >= kMinNtRunBits);
}

template <typename T>
static Mat2<T> to_mat2(const double *U) {
    Mat2<T> g;
    for (int i = 0; i < 4; ++i) g.m[i] = cpx<T>{(T)U[2 * i], (T)U[2 * i + 1]};
    return g;
}

constexpr int kUnroll = 4;
constexpr uint64_t kGridCap = 1ull << 20;
// The streamed one-qubit gate on pairs of 16-byte elements: one pair per
// thread and a grid covering the state in one round measured 5.5-6.0 TB/s
// on a 32 GiB state against 4.9-5.6 TB/s with four pairs per thread, except
// for element strides near 2^20 (5.44 against 5.59 TB/s).  The grid stops
// at 2^23 workgroups (a launch's threads must number fewer than 2^32): one
// round up to 33 qubits complex64 / 32 complex128, grid-stride beyond.
constexpr int kPairUnroll = 1;
constexpr uint64_t kPairGridCap = 1ull << 23;

hipError_t launch_gate1(void *amps, int n, int dtype, int t, uint64_t ctrl, const double *U,
                        hipStream_t s) {
    const int vbits = dtype == SV_C64 ? 1 : 0;
    const uint64_t n_el = (1ull << n) >> vbits;
    uint32_t lane_ctrl = 0;
    int np = 0;
    const bool skip = finite_as(dtype, U, 8);
    if (t < vbits) {
        // complex64, target qubit 0: enumerate elements restricted by controls
        Enum e = make_enum(vbits, nullptr, 0, ctrl, &lane_ctrl, &np);
        const uint64_t count = n_el >> np;
        const uint64_t per = (uint64_t)kUnroll * kStreamThreads;
        const dim3 grid((unsigned)grid_for(count, per, kGridCap));
        if (nt_ok(e))
            k_gate1_q0<kUnroll, true><<<grid, dim3(kStreamThreads), 0, s>>>((float4 *)amps, e, count, to_mat2<float>(U), skip);
        else
            k_gate1_q0<kUnroll, false><<<grid, dim3(kStreamThreads), 0, s>>>((float4 *)amps, e, count, to_mat2<float>(U), skip);
        return hipGetLastError();
    }
    const int te = t - vbits;
    Enum e = make_enum(vbits, &te, 1, ctrl, &lane_ctrl, &np);
    const uint64_t count = n_el >> np;
    const uint64_t per = (uint64_t)kPairUnroll * kStreamThreads;
    const dim3 grid((unsigned)grid_for(count, per, kPairGridCap));
    const bool nt = nt_ok(e);
    constexpr int PU = kPairUnroll;
    if (dtype == SV_C64 && nt)
        k_gate1<float, PU, true><<<grid, dim3(kStreamThreads), 0, s>>>((float4 *)amps, e, te, count, to_mat2<float>(U), lane_ctrl, skip);
    else if (dtype == SV_C64)
        k_gate1<float, PU, false><<<grid, dim3(kStreamThreads), 0, s>>>((float4 *)amps, e, te, count, to_mat2<float>(U), lane_ctrl, skip);
    else if (nt)
        k_gate1<double, PU, true><<<grid, dim3(kStreamThreads), 0, s>>>((double2 *)amps, e, te, count, to_mat2<double>(U), lane_ctrl, skip);
    else
        k_gate1<double, PU, false><<<grid, dim3(kStreamThreads), 0, s>>>((double2 *)amps, e, te, count, to_mat2<double>(U), lane_ctrl, skip);
    return hipGetLastError();
}

// ------------------------------------------------------- streamed 2q gate
// Quad index q = b0 + 2 b1 (bit j of q = value of targets[j]); both targets
// at or above the vector width.
template <typename T, int UNROLL, bool NT>
__global__ __launch_bounds__(kStreamThreads) void k_gate2(typename Vec<T>::type *v, Enum e, int te0,
                                                          int te1, uint64_t count, Mat4<T> g,
                                                          uint32_t lane_ctrl, bool skip) {
    using V = Vec<T>;
    const uint64_t per_block = (uint64_t)UNROLL * kStreamThreads;
    const uint64_t s0 = 1ull << te0, s1 = 1ull << te1;
    for (uint64_t base = (uint64_t)blockIdx.x * per_block; base < count;
         base += (uint64_t)gridDim.x * per_block) {
        typename V::type w[UNROLL][4];
        uint64_t ia[UNROLL];
        bool ok[UNROLL];
#pragma unroll
        for (int u = 0; u < UNROLL; ++u) {
            const uint64_t j = base + (uint64_t)u * kStreamThreads + threadIdx.x;
            const uint64_t a = expand(e, j < count ? j : 0);
            ok[u] = (j < count) && ((a & e.check) == e.check);
            ia[u] = a;
            if (ok[u]) {
                w[u][0] = ld16<NT>(&v[a]);
                w[u][1] = ld16<NT>(&v[a + s0]);
                w[u][2] = ld16<NT>(&v[a + s1]);
                w[u][3] = ld16<NT>(&v[a + s0 + s1]);
            }
        }
#pragma unroll
        for (int u = 0; u < UNROLL; ++u) {
            if (!ok[u]) continue;
            if (skip && wave_zero(magnitude_bits(w[u][0]) | magnitude_bits(w[u][1]) | magnitude_bits(w[u][2]) |
                                  magnitude_bits(w[u][3])))
                continue;
            typename V::type o[4] = {w[u][0], w[u][1], w[u][2], w[u][3]};
#pragma unroll
            for (int k = 0; k < V::amps; ++k) {
                if (((uint32_t)k & lane_ctrl) != lane_ctrl) continue;
                cpx<T> x[4];
#pragma unroll
                for (int q = 0; q < 4; ++q) x[q] = V::get(w[u][q], k);
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    cpx<T> acc = cmul(g.m[4 * r], x[0]);
#pragma unroll
                    for (int c = 1; c < 4; ++c) acc = cfma(g.m[4 * r + c], x[c], acc);
                    V::put(o[r], k, acc);
                }
            }
            st16<NT>(&v[ia[u]], o[0]);
            st16<NT>(&v[ia[u] + s0], o[1]);
            st16<NT>(&v[ia[u] + s1], o[2]);
            st16<NT>(&v[ia[u] + s0 + s1], o[3]);
        }
    }
}

template <typename T>
static Mat4<T> to_mat4(const double *U) {
    Mat4<T> g;
    for (int i = 0; i < 16; ++i) g.m[i] = cpx<T>{(T)U[2 * i], (T)U[2 * i + 1]};
    return g;
}

hipError_t launch_gate2(void *amps, int n, int dtype, int t0, int t1, uint64_t ctrl,
                        const double *U, hipStream_t s) {
    const int vbits = dtype == SV_C64 ? 1 : 0;
    if (t0 < vbits || t1 < vbits) return hipErrorInvalidValue; // routed to the tile pass
    const uint64_t n_el = (1ull << n) >> vbits;
    const int te[2] = {t0 - vbits, t1 - vbits};
    uint32_t lane_ctrl = 0;
    int np = 0;
    Enum e = make_enum(vbits, te, 2, ctrl, &lane_ctrl, &np);
    const uint64_t count = n_el >> np;
    constexpr int U2 = 2;
    const uint64_t per = (uint64_t)U2 * kStreamThreads;
    const dim3 grid((unsigned)grid_for(count, per, kGridCap));
    const bool nt = nt_ok(e), skip = finite_as(dtype, U, 32);
    if (dtype == SV_C64 && nt)
        k_gate2<float, U2, true><<<grid, dim3(kStreamThreads), 0, s>>>((float4 *)amps, e, te[0], te[1], count, to_mat4<float>(U), lane_ctrl, skip);
    else if (dtype == SV_C64)
        k_gate2<float, U2, false><<<grid, dim3(kStreamThreads), 0, s>>>((float4 *)amps, e, te[0], te[1], count, to_mat4<float>(U), lane_ctrl, skip);
    else if (nt)
        k_gate2<double, U2, true><<<grid, dim3(kStreamThreads), 0, s>>>((double2 *)amps, e, te[0], te[1], count, to_mat4<double>(U), lane_ctrl, skip);
    else
        k_gate2<double, U2, false><<<grid, dim3(kStreamThreads), 0, s>>>((double2 *)amps, e, te[0], te[1], count, to_mat4<double>(U), lane_ctrl, skip);
    return hipGetLastError();
}

// ------------------------------------------------- subspace scaling
// Multiply every amplitude x with (x & mask) == mask by a complex factor:
// a phase-type diagonal gate (diag(1, f), optionally controlled) only changes
// the amplitudes whose target and control bits are all 1.
template <typename T, int UNROLL, bool NT>
__global__ __launch_bounds__(kStreamThreads) void k_scale(typename Vec<T>::type *v, Enum e,
                                                          uint64_t count, cpx<T> f,
                                                          uint32_t lane_set, bool skip) {
    using V = Vec<T>;
    const uint64_t per_block = (uint64_t)UNROLL * kStreamThreads;
    for (uint64_t base = (uint64_t)blockIdx.x * per_block; base < count;
         base += (uint64_t)gridDim.x * per_block) {
        typename V::type w[UNROLL];
        uint64_t ia[UNROLL];
        bool ok[UNROLL];
#pragma unroll
        for (int u = 0; u < UNROLL; ++u) {
            const uint64_t j = base + (uint64_t)u * kStreamThreads + threadIdx.x;
            const uint64_t a = expand(e, j < count ? j : 0);
            ok[u] = (j < count) && ((a & e.check) == e.check);
            ia[u] = a;
            if (ok[u]) w[u] = ld16<NT>(&v[a]);
        }
#pragma unroll
        for (int u = 0; u < UNROLL; ++u) {
            if (!ok[u]) continue;
            if (skip && wave_zero(magnitude_bits(w[u]))) continue;
#pragma unroll
            for (int k = 0; k < V::amps; ++k) {
                if (((uint32_t)k & lane_set) != lane_set) continue;
                V::put(w[u], k, cmul(f, V::get(w[u], k)));
            }
            st16<NT>(&v[ia[u]], w[u]);
        }
    }
}

hipError_t launch_scale(void *amps, int n, int dtype, uint64_t set_mask, const double *factor,
                        hipStream_t s) {
    const int vbits = dtype == SV_C64 ? 1 : 0;
    const uint64_t n_el = (1ull << n) >> vbits;
    uint32_t lane_set = 0;
    int np = 0;
    Enum e = make_enum(vbits, nullptr, 0, set_mask, &lane_set, &np);
    const uint64_t count = n_el >> np;
    const uint64_t per = (uint64_t)kUnroll * kStreamThreads;
    const dim3 grid((unsigned)grid_for(count, per, kGridCap));
    const cpx<float> f32{(float)factor[0], (float)factor[1]};
    const cpx<double> f64{factor[0], factor[1]};
    const bool nt = nt_ok(e), skip = finite_as(dtype, factor, 2);
    if (dtype == SV_C64 && nt)
        k_scale<float, kUnroll, true><<<grid, dim3(kStreamThreads), 0, s>>>((float4 *)amps, e, count, f32, lane_set, skip);
    else if (dtype == SV_C64)
        k_scale<float, kUnroll, false><<<grid, dim3(kStreamThreads), 0, s>>>((float4 *)amps, e, count, f32, lane_set, skip);
    else if (nt)
        k_scale<double, kUnroll, true><<<grid, dim3(kStreamThreads), 0, s>>>((double2 *)amps, e, count, f64, lane_set, skip);
    else
        k_scale<double, kUnroll, false><<<grid, dim3(kStreamThreads), 0, s>>>((double2 *)amps, e, count, f64, lane_set, skip);
    return hipGetLastError();
}

// ------------------------------------------------------------ tile pass
// A workgroup holds one tile of 2^m amplitudes in registers and exchanges it
// through LDS: the low qubits 0..L-1 (contiguous runs of 2^L amplitudes in
// HBM) plus K further qubits.  The pass's gates, grouped into register sweeps
// by the host, are applied to the tile (tile_sweep.hpp); controls outside the
// tile are constant over a tile and tested once on its base index.
// one register group of 16 amplitudes per thread
template <typename T>
constexpr int kTileThreads = std::is_same<T, float>::value ? 1024 : 512;

// Tiles of 16384 complex64 or 8192 complex128 amplitudes, of which the sweeps
// exchange one component at a time: 64 KiB of LDS, two workgroups of 1024
// and 512 threads per CU, which fill the eight (complex64) and four
// (complex128) waves per SIMD that their registers allow.  A larger tile
// takes more gates per trip of the state: depth 20 at 29 qubits complex64
// takes 44.3, 39.9 and 36.1 ms with tiles of 2^12, 2^13 and 2^14, at 28
// qubits complex128 40.0, 35.6 and 38.7 (of 2^14 a CU holds one workgroup,
// and nothing runs while it loads or stores).  The order is the same for
// random circuits and QFTs from 13 to 27 qubits.  The batch kernel keeps
// 8192-amplitude complex64 tiles (whole circuits of up to 13 qubits in one
// workgroup).
static_assert(1 << (tile_max_qubits(SV_C64) - kSweepW) == kTileThreads<float> &&
                  1 << (tile_max_qubits(SV_C128) - kSweepW) == kTileThreads<double>,
              "one group per thread");

// Register qubits per sweep of the batch and adjoint kernels, which hold 8
// complex128 amplitudes per group.  The tile pass holds 16 (kSweepW) in both
// precisions.  For complex128 that doubled what a CU has in flight at its
// four waves per SIMD: with whole amplitudes crossing LDS, 512 threads with a
// group of 8 each took 64 KiB, of which two workgroups fit; now the two
// components cross one after the other, with two more barriers, and the same
// 64 KiB serve a tile of 512 groups of 16.  Half the records per amplitude and
// fewer sweeps come with it: depth 20 at 28 qubits 49.6 -> 40.1 ms, on tiles of
// 2^12, of which four workgroups of 256 threads fit (present tiles: see
// kTileThreads).  The same exchange took complex64 tiles of 2^12 from five to
// seven waves per SIMD (29 qubits 48.3 -> 44.7 ms); those of 2^14 run eight.
int sweep_width(int dtype) { return dtype == SV_C64 ? 4 : 3; }

// Waves per SIMD the register allocation aims at.
template <typename T>
constexpr int kTileWaves = std::is_same<T, double>::value ? 4 : 8;

// One pass: the first sweep reads its groups straight from the state and
// the last writes them straight back, so the tile crosses LDS only between
// sweeps (a pass of one sweep never touches it).  One workgroup per tile and
// one register group per thread.
//
// ZSKIP: a tile of zeros is left as it is (see launch_tile).  Each wave
// reports whether its groups hold anything, and the waves look at all reports
// after the first barrier of the first exchange, where they meet anyway; a
// wave of zeros walks no records until then.
template <typename T, int W, bool TWOQ, bool LPH, bool ZSKIP>
__global__ __launch_bounds__(kTileThreads<T>, kTileWaves<T>) void k_tile(typename Vec<T>::type *vec, TileSpec sp,
                                                                      const TileSweep *__restrict__ sweeps,
                                                                      int n_sweeps, const char *__restrict__ recs,
                                                                      uint32_t bytes) {
    constexpr int D = 1 << W;
    extern __shared__ char lds[];
    // the workgroups that start together (see warm_records); sweeps and
    // records lie one after the other
    if (blockIdx.x < kWarmGroups) warm_records(sweeps, bytes);
    uint64_t base = (uint64_t)blockIdx.x << sp.L;
    for (int i = 0; i < sp.K; ++i) base = insert_zero(base, sp.high[i]);
    cpx<T> *tile = reinterpret_cast<cpx<T> *>(vec) + base;
    const uint32_t g = threadIdx.x;
    cpx<T> v[D];
    {
        const TileSweep &S = sweeps[0];
        const cpx<T> *row = tile + group_columns(S.at_lane, g);
#pragma unroll
        for (int j = 0; j < D; ++j) v[j] = row[register_columns<W>(S.at_reg, j)];
    }
    bool zero = false;
    // ZSKIP: a word per wave behind the tile, whether its groups hold anything
    uint32_t *seen = reinterpret_cast<uint32_t *>(lds + blockDim.x * D * (uint32_t)sizeof(T));
    if constexpr (ZSKIP) {
        // the first amplitudes settle it for a register that is not sparse
        zero = wave_zero(magnitude_bits(v[0].re) | magnitude_bits(v[0].im));
        if (zero) {
            uint32_t bits = 0;
#pragma unroll
            for (int j = 1; j < D; ++j) bits |= magnitude_bits(v[j].re) | magnitude_bits(v[j].im);
            zero = wave_zero(bits);
        }
        if ((threadIdx.x & 63u) == 0u) seen[threadIdx.x >> 6] = zero ? 0u : 1u;
    }
    // behind a barrier: no wave of the tile's has seen anything (their number
    // is a power of two; a branch on the lane in the loop below would have the
    // compiler copy the groups, and an address formed before it a register)
    auto tile_zero = [&]() {
        uint32_t t = g;
        asm volatile("" : "+v"(t));
        return wave_zero(seen[t & ((blockDim.x >> 6) - 1u)]);
    };
    for (int si = 0;; ++si) {
        const TileSweep &S = sweeps[si];
        PhaseAcc<T, W> acc;
        acc.init();
        run_records<T, W, TWOQ, LPH>(v, acc, g, recs + S.rec_off, ZSKIP && si == 0 && zero ? 0 : S.n_gates, base);
        if (si == n_sweeps - 1) break;
        const TileSweep &N = sweeps[si + 1];
        uint32_t pg = out_constant(S, recs, base) ^ group_columns(S.out_lane, g);
        const uint32_t pn = group_columns(N.in_lane, g);
        // the real parts, then the imaginary parts
        lds_store_part<T, W, 0>(lds, pg, S.out_reg, v);
        __syncthreads();
        if constexpr (ZSKIP) {
            if (si == 0 && tile_zero()) return;
            // the imaginary parts' addresses are formed anew: kept across the
            // exit they spill (complex64)
            asm volatile("" : "+v"(pg));
        }
        lds_load_part<T, W, 0>(lds, pn, N.in_reg, v);
        __syncthreads();
        lds_store_part<T, W, 1>(lds, pg, S.out_reg, v);
        __syncthreads();
        lds_load_part<T, W, 1>(lds, pn, N.in_reg, v);
        // every group is read before the next exchange writes; the last
        // sweep's results go to the state
        if (si + 2 < n_sweeps) __syncthreads();
    }
    const TileSweep &S = sweeps[n_sweeps - 1];
    if (S.perm) {
        // other groups' places, once every group has been read
        if (n_sweeps == 1) {
            __syncthreads();
            if constexpr (ZSKIP) {
                if (tile_zero()) return;
            }
        }
        const uint64_t to = to_constant(S, recs, base) ^ group_columns(S.to_lane, g);
#pragma unroll
        for (int j = 0; j < D; ++j) tile[to ^ register_columns<W>(S.to_reg, j)] = v[j];
    } else {
        if (ZSKIP && n_sweeps == 1 && zero) return; // a group's results go where it was read
        cpx<T> *row = tile + group_columns(S.to_lane, g);
#pragma unroll
        for (int j = 0; j < D; ++j) row[register_columns<W>(S.to_reg, j)] = v[j];
    }
}

template <typename T, int W, bool TWOQ, bool LPH = std::is_same<T, double>::value>
static void launch_tile_t(typename Vec<T>::type *v, const TileSpec &spec, int m, const TileSweep *sw,
                          int n_sweeps, const char *g, uint32_t bytes, uint64_t n_tiles, bool skip_zero, size_t lds,
                          hipStream_t s) {
    // one workgroup per tile (measured faster than a capped grid looping
    // over tiles), and one thread per register group
    const unsigned threads = 1u << (m - W);
    auto launch = [&](auto kernel) {
        (void)hipFuncSetAttribute((const void *)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        kernel<<<(unsigned)n_tiles, threads, lds, s>>>(v, spec, sw, n_sweeps, g, bytes);
    };
    // tiles of less than a wave are states of one tile
    constexpr bool FULL = W == kSweepW;
    if constexpr (FULL) {
        if (skip_zero && threads >= 64) {
            lds += threads / 64 * sizeof(uint32_t);
            launch(k_tile<T, W, TWOQ, LPH, true>);
            return;
        }
    }
    launch(k_tile<T, W, TWOQ, LPH, false>);
}

// skip_zero: the pass may leave a tile that holds only zeros as it is.  A
// register starts as a basis state and spreads over the qubits of one tile
// after the other: until every qubit has been acted on, most tiles hold
// zeros, and zeros stay zeros under any gate.  Such a tile costs its read.
// On |x> at 30 qubits complex128 the QFT's first pass (phases conditioned on
// 18 outside qubits) takes 4.6 ms instead of 18.4, its second and third
// 2.7 and 3.2 instead of 7.0 and 7.2 (the whole circuit 43.1 -> 21.0 ms, on
// tiles of 2^12; on tiles of 2^13 18.9, and 18.1 since the test has no barrier
// of its own).  On a dense register, which a caller may have written after it
// was set to a basis state, the test costs nothing: ten rotations on 2^26
// complex128 amplitudes take 0.417 ms with it and 0.420 without.  With a
// barrier before the first sweep's updates, where every wave waited for the
// last one's reads, they took 0.468 (layers of gates 1 to 5 % more, up to 16 %
// on tiles of 2^12).  The host sets the flag only while some qubit outside the
// tile has not been acted on since the register was set to a basis state
// (sv_state::moved): later, a tile of zeros is no longer likely.
hipError_t launch_tile(void *amps, int n, int dtype, const TileSpec &spec, const TileSweep *dev_sweeps,
                       int n_sweeps, const char *dev_gates, size_t bytes, bool two_qubit, bool lane_phases, bool skip_zero,
                       hipStream_t s) {
    const int m = spec.L + spec.K;
    const int vbits = dtype == SV_C64 ? 1 : 0;
    if (m > n || m > tile_max_qubits(dtype) || spec.L < vbits || spec.K > kMaxTileHigh || m < 1 ||
        n - m > 30 || n_sweeps < 1)
        return hipErrorInvalidValue;
    const uint64_t n_tiles = 1ull << (n - m);
    const size_t lds = (size_t)(1u << m) * (dtype == SV_C64 ? 4 : 8); // one component
    const int W = std::min(m, kSweepW);
    if ((1 << (m - W)) > (dtype == SV_C64 ? kTileThreads<float> : kTileThreads<double>)) return hipErrorInvalidValue; // one group per thread
    // complex64 lane-bit phase lists: only the full-width instances hold
    // them (the complex128 instances always do)
    if (lane_phases && dtype == SV_C64) {
        if (W != kSweepW) return hipErrorInvalidValue;
        if (two_qubit)
            launch_tile_t<float, 4, true, true>((float4 *)amps, spec, m, dev_sweeps, n_sweeps, dev_gates, bytes, n_tiles,
                                                skip_zero, lds, s);
        else
            launch_tile_t<float, 4, false, true>((float4 *)amps, spec, m, dev_sweeps, n_sweeps, dev_gates,
                                                 bytes, n_tiles, skip_zero, lds, s);
        return hipGetLastError();
    }
#define SV_TILE_CASE(WW, Q)                                                                        \
    if (W == WW && two_qubit == Q) {                                                               \
        if (dtype == SV_C64)                                                                       \
            launch_tile_t<float, WW, Q>((float4 *)amps, spec, m, dev_sweeps, n_sweeps, dev_gates,  \
                                        bytes, n_tiles, skip_zero, lds, s);                                  \
        else                                                                                       \
            launch_tile_t<double, WW, Q>((double2 *)amps, spec, m, dev_sweeps, n_sweeps,           \
                                         dev_gates, bytes, n_tiles, skip_zero, lds, s);                      \
        return hipGetLastError();                                                                  \
    }
    SV_TILE_CASE(4, false)
    SV_TILE_CASE(3, false)
    SV_TILE_CASE(2, false)
    SV_TILE_CASE(1, false)
    SV_TILE_CASE(4, true)
    SV_TILE_CASE(3, true)
    SV_TILE_CASE(2, true)
    SV_TILE_CASE(1, true)
#undef SV_TILE_CASE
    return hipErrorInvalidValue;
}

} // namespace sv
