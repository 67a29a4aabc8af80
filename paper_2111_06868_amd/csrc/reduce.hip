// FP64 reductions over a state: norm, inner product, Pauli-sum expectation,
// the Pauli-sum matvec used by the adjoint method, and Tr(rho H) of a density
// matrix held as a state of 2n qubits.
//
// Every reduction is a fixed-shape two-stage tree (kRedBlocks x kRedThreads
// first stage with a fixed grid-stride assignment, LDS tree inside a block,
// then one block summing the partials in a fixed order), so results are
// bitwise reproducible run to run.  Amplitudes are widened to FP64 before any
// product.
//
// Pauli strings: P = i^{#Y} X^x Z^z (per qubit Y = i X Z), hence
//   (P psi)[i] = i^{#Y} (-1)^{popcount((i ^ x) & z)} psi[i ^ x].
// Terms are grouped by their x mask on the host so that each partner
// amplitude psi[i ^ x] is loaded once per group.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>

#include "device.h"
#include "kernels.h"

namespace sv {
namespace dev {

namespace {

template <int C>
struct Acc {
    double v[C];
};

template <int C>
__device__ __forceinline__ void block_reduce_store(Acc<C> a, double *__restrict__ out)
{
    __shared__ double sh[C][kRedThreads];
    const int t = threadIdx.x;
#pragma unroll
    for (int c = 0; c < C; ++c) sh[c][t] = a.v[c];
    __syncthreads();
    for (int s = kRedThreads / 2; s > 0; s >>= 1) {
        if (t < s) {
#pragma unroll
            for (int c = 0; c < C; ++c) sh[c][t] += sh[c][t + s];
        }
        __syncthreads();
    }
    if (t == 0) {
#pragma unroll
        for (int c = 0; c < C; ++c) out[c] = sh[c][0];
    }
}

__device__ __forceinline__ void ld(const float *p, uint64_t i, double &re, double &im)
{
    const float2 v = reinterpret_cast<const float2 *>(p)[i];
    re = v.x;
    im = v.y;
}
__device__ __forceinline__ void ld(const double *p, uint64_t i, double &re, double &im)
{
    const double2 v = reinterpret_cast<const double2 *>(p)[i];
    re = v.x;
    im = v.y;
}

template <typename T>
__global__ void __launch_bounds__(kRedThreads) k_norm(const T *__restrict__ psi, uint64_t N, double *partials)
{
    Acc<1> a{{0.0}};
    for (uint64_t i = uint64_t(blockIdx.x) * kRedThreads + threadIdx.x; i < N; i += uint64_t(kRedBlocks) * kRedThreads) {
        double r, m;
        ld(psi, i, r, m);
        a.v[0] = fma(r, r, fma(m, m, a.v[0]));
    }
    block_reduce_store<1>(a, partials + blockIdx.x);
}

// complex64 norm: each thread takes 4 consecutive 16-byte pairs of
// amplitudes per step (4 loads in flight), in a fixed assignment
__global__ void __launch_bounds__(kRedThreads) k_norm_c64(const float4 *__restrict__ psi, uint64_t N4,
                                                          double *partials)
{
    Acc<1> a{{0.0}};
    constexpr uint64_t kStep = uint64_t(kRedBlocks) * kRedThreads * 4;
    for (uint64_t i0 = (uint64_t(blockIdx.x) * kRedThreads + threadIdx.x) * 4; i0 < N4; i0 += kStep) {
        float4 v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) v[u] = i0 + u < N4 ? psi[i0 + u] : make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            a.v[0] = fma(double(v[u].x), double(v[u].x), a.v[0]);
            a.v[0] = fma(double(v[u].y), double(v[u].y), a.v[0]);
            a.v[0] = fma(double(v[u].z), double(v[u].z), a.v[0]);
            a.v[0] = fma(double(v[u].w), double(v[u].w), a.v[0]);
        }
    }
    block_reduce_store<1>(a, partials + blockIdx.x);
}

template <typename A, typename B>
__global__ void __launch_bounds__(kRedThreads) k_inner(const A *__restrict__ a, const B *__restrict__ b, uint64_t N,
                                                      double *partials)
{
    Acc<2> s{{0.0, 0.0}};
    for (uint64_t i = uint64_t(blockIdx.x) * kRedThreads + threadIdx.x; i < N; i += uint64_t(kRedBlocks) * kRedThreads) {
        double ar, ai, br, bi;
        ld(a, i, ar, ai);
        ld(b, i, br, bi);
        // conj(a) * b
        s.v[0] = fma(ar, br, fma(ai, bi, s.v[0]));
        s.v[1] = fma(ar, bi, fma(-ai, br, s.v[1]));
    }
    block_reduce_store<2>(s, partials + 2 * blockIdx.x);
}

// weight of group g at partner index j: sum_t c_t (-1)^{popcount(j & z_t)}
// (times i for a group with kPauliImag set)
__device__ __forceinline__ double group_weight(const PauliDev &H, int g, uint64_t j)
{
    double w = 0.0;
    for (int t = H.goff[g]; t < H.goff[g + 1]; ++t) {
        const double c = H.tc[t];
        w += __popcll(j & H.tz[t]) & 1 ? -c : c;
    }
    return w;
}

// (re, im) times w, or times i w for an imaginary group
__device__ __forceinline__ void add_weighted(uint64_t gx, double w, double pr, double pi, double &sr, double &si)
{
    if (gx & kPauliImag) {
        sr = fma(-w, pi, sr);
        si = fma(w, pr, si);
    } else {
        sr = fma(w, pr, sr);
        si = fma(w, pi, si);
    }
}

template <typename T>
__global__ void __launch_bounds__(kRedThreads) k_pauli_expect(const T *__restrict__ psi, uint64_t N, const PauliDev H,
                                                             double *partials)
{
    Acc<1> a{{0.0}};
    for (uint64_t i = uint64_t(blockIdx.x) * kRedThreads + threadIdx.x; i < N; i += uint64_t(gridDim.x) * kRedThreads) {
        double cr, ci;
        ld(psi, i, cr, ci);
        double sr = 0.0, si = 0.0;
        for (int g = 0; g < H.n_groups; ++g) {
            const uint64_t j = i ^ (H.gx[g] & ~kPauliImag);
            double pr, pi;
            ld(psi, j, pr, pi);
            add_weighted(H.gx[g], group_weight(H, g, j), pr, pi, sr, si);
        }
        // Re(conj(psi_i) * s)
        a.v[0] = fma(cr, sr, fma(ci, si, a.v[0]));
    }
    block_reduce_store<1>(a, partials + blockIdx.x);
}

// Tr(rho H) for rho held row-major in a state of 2n qubits (rho[r][c] at
// r 2^n + c).  With P|a> = omega(a)|a ^ x>, Tr(rho P) = sum_a omega(a)
// rho[a][a ^ x]; omega(a) is the group weight at a (group_weight), and only
// the real part is summed (H is Hermitian).
template <typename T>
__global__ void __launch_bounds__(kRedThreads) k_dm_expect(const T *__restrict__ rho, int n, const PauliDev H,
                                                          double *partials)
{
    Acc<1> acc{{0.0}};
    const uint64_t N = uint64_t(1) << n;
    for (uint64_t a = uint64_t(blockIdx.x) * kRedThreads + threadIdx.x; a < N; a += uint64_t(kRedBlocks) * kRedThreads) {
        for (int g = 0; g < H.n_groups; ++g) {
            double rr, ri;
            ld(rho, (a << n) | (a ^ (H.gx[g] & ~kPauliImag)), rr, ri);
            const double w = group_weight(H, g, a);
            acc.v[0] = H.gx[g] & kPauliImag ? fma(-ri, w, acc.v[0]) : fma(rr, w, acc.v[0]);
        }
    }
    block_reduce_store<1>(acc, partials + blockIdx.x);
}

// Outcome weights of a Kraus channel on k sorted positions: p_i = ||K_i psi||^2
// (paper, Simulations with noise section: channels sampled on pure states).
// Each thread gathers the 2^k amplitudes of U groups (local bit j on the j-th
// lowest position; all loads issued before any arithmetic, so that U groups
// are in flight per thread), forms K_i x for every operator and adds
// |K_i x|^2, all in FP64.  The per-thread order of the groups is fixed, so the
// result is reproducible.
template <typename T, int K>
__global__ void __launch_bounds__(kRedThreads) k_kraus_probs(const T *__restrict__ psi, int n, const KrausDev Kd,
                                                            double *partials)
{
    constexpr int D = 1 << K;
    constexpr int U = K == 3 ? 2 : 4;
    Acc<kMaxKraus> acc;
#pragma unroll
    for (int i = 0; i < kMaxKraus; ++i) acc.v[i] = 0.0;
    const uint64_t groups = uint64_t(1) << (n - K);
    const uint64_t stride = uint64_t(kRedBlocks) * kRedThreads;
    for (uint64_t g0 = uint64_t(blockIdx.x) * kRedThreads + threadIdx.x; g0 < groups; g0 += U * stride) {
        double xr[U][D], xi[U][D];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const uint64_t g = g0 + u * stride;
            uint64_t base = g < groups ? g : 0;
#pragma unroll
            for (int j = 0; j < K; ++j) {  // insert a zero bit at each position, lowest first
                const uint64_t low = base & ((uint64_t(1) << Kd.pos[j]) - 1);
                base = ((base - low) << 1) | low;
            }
#pragma unroll
            for (int m = 0; m < D; ++m) {
                uint64_t idx = base;
#pragma unroll
                for (int j = 0; j < K; ++j)
                    if ((m >> j) & 1) idx |= uint64_t(1) << Kd.pos[j];
                ld(psi, idx, xr[u][m], xi[u][m]);
            }
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (g0 + u * stride >= groups) continue;
#pragma unroll
            for (int i = 0; i < kMaxKraus; ++i) {
                if (i >= Kd.n_ops) continue;  // uniform
                const double *M = Kd.m + size_t(2) * D * D * i;
                double s = 0.0;
#pragma unroll
                for (int r = 0; r < D; ++r) {
                    double yr = 0.0, yi = 0.0;
#pragma unroll
                    for (int c = 0; c < D; ++c) {
                        const double mr = M[2 * (r * D + c)], mi = M[2 * (r * D + c) + 1];
                        yr = fma(mr, xr[u][c], fma(-mi, xi[u][c], yr));
                        yi = fma(mr, xi[u][c], fma(mi, xr[u][c], yi));
                    }
                    s = fma(yr, yr, fma(yi, yi, s));
                }
                acc.v[i] += s;
            }
        }
    }
    block_reduce_store<kMaxKraus>(acc, partials + size_t(blockIdx.x) * kMaxKraus);
}

// The same for complex64 states with 16-byte loads: when the channel's lowest
// position is 0 (LOW0), amplitudes m and m + 1 of a group are adjacent; else
// the groups 2h and 2h + 1 differ only in position 0, so amplitude m of both is
// one float4.  Each thread takes U units (groups, or pairs of groups) per step.
template <int K, bool LOW0>
__global__ void __launch_bounds__(kRedThreads) k_kraus_probs_c64(const float4 *__restrict__ psi, int n,
                                                                const KrausDev Kd, double *partials)
{
    constexpr int D = 1 << K;
    constexpr int G = LOW0 ? 1 : 2;                // groups per unit
    constexpr int L = LOW0 ? D / 2 : D;            // float4 loads per unit
    constexpr int U = K == 3 ? (LOW0 ? 2 : 1) : 4;
    Acc<kMaxKraus> acc;
#pragma unroll
    for (int i = 0; i < kMaxKraus; ++i) acc.v[i] = 0.0;
    const uint64_t units = uint64_t(1) << (n - K - (LOW0 ? 0 : 1));
    const uint64_t stride = uint64_t(kRedBlocks) * kRedThreads;
    for (uint64_t h0 = uint64_t(blockIdx.x) * kRedThreads + threadIdx.x; h0 < units; h0 += U * stride) {
        float4 v[U][L];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const uint64_t h = h0 + u * stride;
            uint64_t base = h < units ? (LOW0 ? h : h << 1) : 0;
#pragma unroll
            for (int j = 0; j < K; ++j) {
                const uint64_t low = base & ((uint64_t(1) << Kd.pos[j]) - 1);
                base = ((base - low) << 1) | low;
            }
#pragma unroll
            for (int l = 0; l < L; ++l) {
                const int m = LOW0 ? 2 * l : l;
                uint64_t idx = base;
#pragma unroll
                for (int j = 0; j < K; ++j)
                    if ((m >> j) & 1) idx |= uint64_t(1) << Kd.pos[j];
                v[u][l] = psi[idx >> 1];
            }
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (h0 + u * stride >= units) continue;
#pragma unroll
            for (int gsel = 0; gsel < G; ++gsel) {
                double xr[D], xi[D];
#pragma unroll
                for (int m = 0; m < D; ++m) {
                    const float4 w = LOW0 ? v[u][m >> 1] : v[u][m];
                    const bool hi = LOW0 ? (m & 1) : gsel;
                    xr[m] = hi ? w.z : w.x;
                    xi[m] = hi ? w.w : w.y;
                }
#pragma unroll
                for (int i = 0; i < kMaxKraus; ++i) {
                    if (i >= Kd.n_ops) continue;  // uniform
                    const double *M = Kd.m + size_t(2) * D * D * i;
                    double s = 0.0;
#pragma unroll
                    for (int r = 0; r < D; ++r) {
                        double yr = 0.0, yi = 0.0;
#pragma unroll
                        for (int c = 0; c < D; ++c) {
                            const double mr = M[2 * (r * D + c)], mi = M[2 * (r * D + c) + 1];
                            yr = fma(mr, xr[c], fma(-mi, xi[c], yr));
                            yi = fma(mr, xi[c], fma(mi, xr[c], yi));
                        }
                        s = fma(yr, yr, fma(yi, yi, s));
                    }
                    acc.v[i] += s;
                }
            }
        }
    }
    block_reduce_store<kMaxKraus>(acc, partials + size_t(blockIdx.x) * kMaxKraus);
}

template <typename T>
__global__ void __launch_bounds__(256) k_pauli_apply(const T *__restrict__ psi, T *__restrict__ out, uint64_t N,
                                                    const PauliDev H)
{
    const uint64_t stride = uint64_t(gridDim.x) * blockDim.x;
    for (uint64_t i = uint64_t(blockIdx.x) * blockDim.x + threadIdx.x; i < N; i += stride) {
        double sr = 0.0, si = 0.0;
        for (int g = 0; g < H.n_groups; ++g) {
            const uint64_t j = i ^ (H.gx[g] & ~kPauliImag);
            double pr, pi;
            ld(psi, j, pr, pi);
            add_weighted(H.gx[g], group_weight(H, g, j), pr, pi, sr, si);
        }
        out[2 * i] = T(sr);
        out[2 * i + 1] = T(si);
    }
}

// <psi|H|psi> and H psi over LDS tiles, for states of at least kPauliTileMin
// qubits.
//
// What bounds it.  One thread per amplitude (k_pauli_expect, k_pauli_apply)
// spends its time on a popcount, a table load and a 8-byte gather per term and
// amplitude: 4.8 and 3.4 ms for the 26-qubit chain with 8 random strings (59
// terms, 35 groups) where reading the state takes 0.1 ms.  Here
//   * a tile is 2048 16-byte slots (2^12 complex64 or 2^11 complex128
//     amplitudes, 32 KiB: several workgroups per compute unit, one loading
//     while others compute), spanned by the lowest 3 slot bits (128-byte runs)
//     and a window of 8 consecutive ones, so that a partner i ^ x whose x lies
//     inside comes from LDS;
//   * <psi|H|psi> takes one pass per window that holds groups (its sums are
//     FP64 partials, so passes add up exactly as one would); a group that no
//     window holds gathers its partners from memory in the first pass;
//   * H psi is one pass (its sums must be whole when they are rounded to the
//     amplitude type): partners outside the tile are gathered, 16 bytes a lane,
//     and the tiles in flight on one XCD differ in the top bits, so those
//     gathers find their lines in that XCD's L2 and the lower ones in the
//     memory-side cache;
//   * a thread holds R = 8 (4) amplitudes that differ in the tile's top two
//     bits (and in position 0), so a term costs it one popcount and one add:
//     the term goes to the bucket of its z bits on those positions, and a
//     Walsh-Hadamard transform of the R buckets gives the R weights.  A group
//     of one term skips the transform.
// Measured at 26 qubits, the terms above: 1.0 and 1.33 ms (before: 4.8 and 3.4).
template <typename T>
struct PauliTile {
    static constexpr int PB = sizeof(T) == 4 ? 1 : 0;  // position bits inside a 16-byte slot
    static constexpr int R = 4 << PB;                  // amplitudes per thread
};
constexpr int kPauliTileThreads = 512;
constexpr int kPauliWindow = 8;                                // window bits
constexpr int kPauliTileSlotBits = 3 + kPauliWindow;           // 512 threads of 4 slots
constexpr uint32_t kPauliWinMask = (1u << kPauliWindow) - 1;

// the tables of dev::PauliDev
struct PauliTables {
    const uint64_t *gx;
    const int32_t *goff;
    const uint64_t *tz;
    const double *tc;
};

__device__ __forceinline__ double flip_sign(double v, uint32_t parity)
{
    return __longlong_as_double(__double_as_longlong(v) ^ (uint64_t(parity) << 63));
}

template <typename T, bool APPLY>
__global__ void __launch_bounds__(kPauliTileThreads, 4)
    k_pauli_tile(const T *__restrict__ psi_, T *__restrict__ out_, int slot_bits, int w, int g0, int g1, const PauliTables H,
                 double *__restrict__ partials, int add)
{
    using Slot = typename std::conditional<sizeof(T) == 4, vf4, vd2>::type;
    constexpr int PB = PauliTile<T>::PB, R = PauliTile<T>::R, NA = 1 << PB;
    __shared__ Slot X[1 << kPauliTileSlotBits];
    const Slot *__restrict__ psi = reinterpret_cast<const Slot *>(psi_);
    const int tid = threadIdx.x;
    // slot bits of the tile: 0..2 and w..w+7
    const uint64_t tile_mask = 7u | (uint64_t(kPauliWinMask) << w);
    const uint64_t n_tiles = uint64_t(1) << (slot_bits - kPauliTileSlotBits);
    auto in_tile = [&](uint64_t v) { return uint32_t(v & 7u) | (uint32_t(v >> w) & kPauliWinMask) << 3; };
    const int tile_bits = slot_bits - kPauliTileSlotBits;
    double e = 0.0;
    for (uint64_t v = blockIdx.x; v < n_tiles; v += gridDim.x) {
        // H psi: the 64 tiles that one XCD (v % 8) has in flight differ in the
        // top six tile bits, the XCDs in the next three
        uint64_t tile = v;
        if (APPLY && tile_bits >= 9)
            tile = ((v >> 3) & 63u) << (tile_bits - 6) | (v & 7u) << (tile_bits - 9) | v >> 9;
        const uint64_t low = tile & ((uint64_t(1) << (w - 3)) - 1);
        const uint64_t base = low << 3 | (tile >> (w - 3)) << (w + kPauliWindow);
        auto slot_of = [&](int rr) {
            const uint32_t s = uint32_t(tid) | uint32_t(rr) << 9;
            return base | (s & 7u) | uint64_t(s >> 3) << w;
        };
        {
            Slot buf[4];
#pragma unroll
            for (int rr = 0; rr < 4; ++rr) buf[rr] = psi[slot_of(rr)];
            __syncthreads();  // the previous tile's readers are done
#pragma unroll
            for (int rr = 0; rr < 4; ++rr) X[tid | rr << 9] = buf[rr];
        }
        __syncthreads();
        double sr[R], si[R];
#pragma unroll
        for (int r = 0; r < R; ++r) sr[r] = si[r] = 0.0;
        for (int g = g0; g < g1; ++g) {
            const uint64_t gx = scalar_load(H.gx, g);
            const uint64_t x = gx & ~kPauliImag, xs = x >> PB;
            const bool imag = (gx & kPauliImag) != 0, swap = PB && (x & 1u);
            const int t0 = scalar_load(H.goff, g), t1 = scalar_load(H.goff, g + 1);
            // a term's coefficient with its sign on this thread's amplitude r = 0
            // and the r bits (rr, position 0) that its z masks
            auto term = [&](uint64_t z, double c, uint32_t &zr) __attribute__((always_inline)) {
                const uint64_t zs = z >> PB;
                const uint32_t zl = in_tile(zs);
                zr = (zl >> 9) << PB | (PB ? uint32_t(z & 1u) : 0u);
                const uint32_t uni = uint32_t(__popcll(z & x) + __popcll(zs & ~tile_mask & base)) & 1u;
                return flip_sign(c, (uni + __popc(zl & uint32_t(tid))) & 1u);
            };
            // adds weight(r) times the partner of amplitude r: (pr, pi), its slot
            // neighbour where x holds position 0, times i in an imaginary group
            auto add_all = [&](auto partner, auto weight, auto swapped, auto times_i) __attribute__((always_inline)) {
#pragma unroll
                for (int rr = 0; rr < 4; ++rr) {
                    double pr[NA], pi[NA];
                    slot_amps(partner(rr), pr, pi);
#pragma unroll
                    for (int b = 0; b < NA; ++b) {
                        const int r = rr << PB | b, o = decltype(swapped)::value ? NA - 1 - b : b;
                        if constexpr (decltype(times_i)::value) {
                            sr[r] = fma(weight(r), -pi[o], sr[r]);
                            si[r] = fma(weight(r), pr[o], si[r]);
                        } else {
                            sr[r] = fma(weight(r), pr[o], sr[r]);
                            si[r] = fma(weight(r), pi[o], si[r]);
                        }
                    }
                }
            };
            auto accumulate = [&](auto partner, auto weight) __attribute__((always_inline)) {
                constexpr std::true_type yes{};
                constexpr std::false_type no{};
                if (imag) {
                    if (swap) add_all(partner, weight, yes, yes);
                    else add_all(partner, weight, no, yes);
                } else {
                    if (swap) add_all(partner, weight, yes, no);
                    else add_all(partner, weight, no, no);
                }
            };
            auto group = [&](auto partner) __attribute__((always_inline)) {
                if (t1 - t0 == 1) {
                    uint32_t zr;
                    const double c = term(scalar_load(H.tz, t0), scalar_load(H.tc, t0), zr);
                    if (zr == 0)
                        accumulate(partner, [&](int) { return c; });
                    else
                        accumulate(partner, [&](int r) { return flip_sign(c, __popc(uint32_t(r) & zr) & 1u); });
                    return;
                }
                double a[R];
#pragma unroll
                for (int r = 0; r < R; ++r) a[r] = 0.0;
                for (int t = t0; t < t1; t += 4) {
                    // four terms' table entries on their way at once
                    uint64_t z[4];
                    double c[4];
#pragma unroll
                    for (int u = 0; u < 4; ++u) {
                        const int tu = t + u < t1 ? t + u : t1 - 1;
                        z[u] = scalar_load(H.tz, tu);
                        c[u] = scalar_load(H.tc, tu);
                    }
#pragma unroll
                    for (int u = 0; u < 4; ++u) {
                        if (t + u >= t1) break;  // uniform
                        uint32_t zr;
                        const double v = term(z[u], c[u], zr);
                        // one bucket is touched: the empty statement keeps each
                        // add behind its (uniform) branch
#pragma unroll
                        for (int r = 0; r < R; ++r)
                            if (zr == uint32_t(r)) {
                                a[r] += v;
                                asm volatile("" : "+v"(a[r]));
                            }
                    }
                }
#pragma unroll
                for (int h = 1; h < R; h <<= 1)
#pragma unroll
                    for (int r = 0; r < R; ++r)
                        if (!(r & h)) {
                            const double u = a[r], d = a[r | h];
                            a[r] = u + d;
                            a[r | h] = u - d;
                        }
                accumulate(partner, [&](int r) { return a[r]; });
            };
            if (xs & ~tile_mask) {  // uniform
                Slot p[4];
#pragma unroll
                for (int rr = 0; rr < 4; ++rr) p[rr] = psi[slot_of(rr) ^ xs];
                group([&](int rr) { return p[rr]; });
            } else {
                const uint32_t at = uint32_t(tid) ^ in_tile(xs);
                group([&](int rr) { return X[at ^ uint32_t(rr) << 9]; });
            }
        }
#pragma unroll
        for (int rr = 0; rr < 4; ++rr) {
            if constexpr (APPLY) {
                Slot o;
                if constexpr (PB == 1) {
                    o.x = T(sr[2 * rr]); o.y = T(si[2 * rr]); o.z = T(sr[2 * rr + 1]); o.w = T(si[2 * rr + 1]);
                } else {
                    o.x = sr[rr]; o.y = si[rr];
                }
                reinterpret_cast<Slot *>(out_)[slot_of(rr)] = o;
            } else {
                double cr[NA], ci[NA];
                slot_amps(X[tid | rr << 9], cr, ci);
#pragma unroll
                for (int b = 0; b < NA; ++b)  // Re(conj(psi_i) (H psi)_i)
                    e = fma(cr[b], sr[rr << PB | b], fma(ci[b], si[rr << PB | b], e));
            }
        }
    }
    if constexpr (!APPLY) {
        __shared__ double sh[kPauliTileThreads / 64];
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) e += __shfl_xor(e, o, 64);
        if ((tid & 63) == 0) sh[tid >> 6] = e;
        __syncthreads();
        if (tid == 0) {
            double v = add ? partials[blockIdx.x] : 0.0;
            for (int i = 0; i < kPauliTileThreads / 64; ++i) v += sh[i];
            partials[blockIdx.x] = v;
        }
    }
}

// Probabilities of the 2^m values of m positions, each amplitude's |psi|^2
// times a product weight: bin v of d_out gets
//   scale sum_{i : bits of i on S = v} prod_p w[p][bit p of i] |psi_i|^2.
// Channels whose operators have diagonal K^dagger K draw their outcomes from
// these sums alone, several channels to a pass; the weights stand for operators
// that are drawn but not applied yet.
//
// What bounds it: reading the state.  One channel at a time (k_kraus_probs, a
// second stage, a copy back and a pass that applies the operator) costs 115 us
// at 24 qubits, 29 of them this read.  A workgroup keeps the positions of S
// above its 2^11-amplitude tiles fixed, so every sum it makes belongs to one
// value of them; the positions below are fixed for each of a thread's 8
// accumulators, and so are their weights, which are multiplied in once at the
// end.  The rest of the weight is one number per tile, from three LDS tables.
// Measured at 24 qubits: 36 us a pass of 10 positions and 5 us for its second
// stage; 96 channels and 4 measured qubits with their gates, 12.1 -> 2.7 ms.
constexpr int kBinTileBits = 11;
struct BinArgs {
    int n, nl, ml, mh;            // nl = min(n, kBinTileBits)
    int lpos[kMaxBins], hpos[kMaxBins];  // S below and above nl, ascending
    double w[SV_MAX_QUBITS_C64][2];
    double scale;
};

template <typename T>
__global__ void __launch_bounds__(256) k_weighted_bins(const T *__restrict__ psi, const BinArgs a,
                                                       double *__restrict__ partials)
{
    constexpr int NA = sizeof(T) == 4 ? 2 : 1;  // amplitudes of a 16-byte load
    constexpr int L = 8 / NA;
    using Slot = typename std::conditional<sizeof(T) == 4, vf4, vd2>::type;
    __shared__ double tab[3][256];
    __shared__ double sums[1 << kBinTileBits];
    const int tid = threadIdx.x;
#pragma unroll
    for (int t = 0; t < 3; ++t) {
        double v = t == 0 ? a.scale : 1.0;
        for (int b = 0; b < 8; ++b) {
            const int p = a.nl + 8 * t + b;
            if (p < a.n) v *= a.w[p][(tid >> b) & 1];
        }
        tab[t][tid] = v;
    }
    __syncthreads();
    const uint32_t hv = blockIdx.x & ((1u << a.mh) - 1u);
    uint64_t fixed = 0;
    for (int j = 0; j < a.mh; ++j) fixed |= uint64_t((hv >> j) & 1u) << a.hpos[j];
    const uint64_t tiles = uint64_t(1) << (a.n - a.nl - a.mh);
    const uint64_t N = uint64_t(1) << a.n;
    double acc[8];
#pragma unroll
    for (int r = 0; r < 8; ++r) acc[r] = 0.0;
    const Slot *__restrict__ slots = reinterpret_cast<const Slot *>(psi);
    for (uint64_t t = blockIdx.x >> a.mh; t < tiles; t += gridDim.x >> a.mh) {
        uint64_t base = t << a.nl;
        for (int j = 0; j < a.mh; ++j) {
            const uint64_t low = base & ((uint64_t(1) << a.hpos[j]) - 1);
            base = ((base - low) << 1) | low;
        }
        base |= fixed;
        Slot v[L];
#pragma unroll
        for (int l = 0; l < L; ++l) {
            const uint64_t i = base + uint64_t(l * 256 + tid) * NA;
            v[l] = Slot(0);
            if (i < N) v[l] = slots[i / NA];
        }
        const uint64_t h = base >> a.nl;
        const double wt = tab[0][h & 255u] * tab[1][(h >> 8) & 255u] * tab[2][(h >> 16) & 255u];
#pragma unroll
        for (int l = 0; l < L; ++l) {
            double re[NA], im[NA];
            slot_amps(v[l], re, im);
#pragma unroll
            for (int b = 0; b < NA; ++b) acc[l * NA + b] = fma(wt, fma(re[b], re[b], im[b] * im[b]), acc[l * NA + b]);
        }
    }
    // the weights of the positions inside the tile, then the sums over those of
    // them that are not in S, the highest position first
#pragma unroll
    for (int r = 0; r < 8; ++r) {
        const int i = ((r / NA) * 256 + tid) * NA + r % NA;
        for (int p = 0; p < a.nl; ++p) acc[r] *= a.w[p][(i >> p) & 1];
        sums[i] = acc[r];
    }
    __syncthreads();
    int size = a.nl, j = a.ml - 1;
    for (int p = a.nl - 1; p >= 0; --p) {
        if (j >= 0 && a.lpos[j] == p) {
            --j;
            continue;
        }
        --size;
        double v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int i = tid + 256 * u;
            if (i < (1 << size)) {
                const int lo = i & ((1 << p) - 1), at = ((i - lo) << 1) | lo;
                v[u] = sums[at] + sums[at | (1 << p)];
            }
        }
        __syncthreads();
#pragma unroll
        for (int u = 0; u < 4; ++u)
            if (tid + 256 * u < (1 << size)) sums[tid + 256 * u] = v[u];
        __syncthreads();
    }
    for (int i = tid; i < (1 << a.ml); i += 256) partials[(size_t(blockIdx.x) << a.ml) | uint32_t(i)] = sums[i];
}

// bin b = hv 2^ml + lv: the partials of the workgroups whose fixed value is hv
__global__ void __launch_bounds__(256) k_bins_final(const double *__restrict__ partials, int ml, int mh, int grid,
                                                    double *out)
{
    const uint32_t bin = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (bin >= (1u << (ml + mh))) return;
    const uint32_t hv = bin >> ml, lv = bin & ((1u << ml) - 1u);
    double v = 0.0;
    for (int k = threadIdx.x & 63; k < grid >> mh; k += 64) v += partials[(size_t(uint32_t(k) << mh | hv) << ml) | lv];
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    if ((threadIdx.x & 63) == 0) out[bin] = v;
}

// Second stage: sums C-component partials of `nb` blocks for `slots` slots
// (one workgroup per slot) in a fixed order.
template <int C>
__global__ void __launch_bounds__(kRedThreads) k_final(const double *__restrict__ partials, int nb, double *out)
{
    const double *p = partials + size_t(blockIdx.x) * nb * C;
    Acc<C> a;
#pragma unroll
    for (int c = 0; c < C; ++c) a.v[c] = 0.0;
    for (int i = threadIdx.x; i < nb; i += kRedThreads) {
#pragma unroll
        for (int c = 0; c < C; ++c) a.v[c] += p[size_t(i) * C + c];
    }
    block_reduce_store<C>(a, out + size_t(blockIdx.x) * C);
}

}  // namespace

hipError_t launch_norm(int dtype, const void *psi, int n, double *d_partials, double *d_out, hipStream_t st)
{
    const uint64_t N = uint64_t(1) << n;
    if (dtype == SV_C64 && n >= 1)
        hipLaunchKernelGGL(k_norm_c64, dim3(kRedBlocks), dim3(kRedThreads), 0, st, static_cast<const float4 *>(psi), N / 2,
                           d_partials);
    else if (dtype == SV_C64)
        hipLaunchKernelGGL(k_norm<float>, dim3(kRedBlocks), dim3(kRedThreads), 0, st, static_cast<const float *>(psi), N, d_partials);
    else
        hipLaunchKernelGGL(k_norm<double>, dim3(kRedBlocks), dim3(kRedThreads), 0, st, static_cast<const double *>(psi), N, d_partials);
    hipLaunchKernelGGL(k_final<1>, dim3(1), dim3(kRedThreads), 0, st, d_partials, kRedBlocks, d_out);
    return hipGetLastError();
}

hipError_t launch_inner(int dtype_a, const void *a, int dtype_b, const void *b, int n, double *d_partials,
                        double *d_out, hipStream_t st)
{
    const uint64_t N = uint64_t(1) << n;
    const dim3 g(kRedBlocks), t(kRedThreads);
    if (dtype_a == SV_C64 && dtype_b == SV_C64)
        hipLaunchKernelGGL((k_inner<float, float>), g, t, 0, st, static_cast<const float *>(a), static_cast<const float *>(b), N, d_partials);
    else if (dtype_a == SV_C64)
        hipLaunchKernelGGL((k_inner<float, double>), g, t, 0, st, static_cast<const float *>(a), static_cast<const double *>(b), N, d_partials);
    else if (dtype_b == SV_C64)
        hipLaunchKernelGGL((k_inner<double, float>), g, t, 0, st, static_cast<const double *>(a), static_cast<const float *>(b), N, d_partials);
    else
        hipLaunchKernelGGL((k_inner<double, double>), g, t, 0, st, static_cast<const double *>(a), static_cast<const double *>(b), N, d_partials);
    hipLaunchKernelGGL(k_final<2>, dim3(1), dim3(kRedThreads), 0, st, d_partials, kRedBlocks, d_out);
    return hipGetLastError();
}

namespace {

unsigned pauli_tile_grid(int slot_bits, unsigned cap)
{
    const uint64_t tiles = uint64_t(1) << (slot_bits - kPauliTileSlotBits);
    return unsigned(tiles < cap ? tiles : cap);
}

template <typename T>
hipError_t pauli_expect_t(const T *psi, int n, const PauliDev &H, double *d_partials, double *d_out, hipStream_t st)
{
    unsigned blocks;
    if (H.tile_expect) {
        const int slot_bits = n - PauliTile<T>::PB;
        blocks = pauli_tile_grid(slot_bits, kRedBlocks);
        int add = 0;
        for (int p = 0; p < H.n_pass; ++p) {
            if (H.pass_end[p] == (p ? H.pass_end[p - 1] : 0)) continue;
            hipLaunchKernelGGL((k_pauli_tile<T, false>), dim3(blocks), dim3(kPauliTileThreads), 0, st, psi,
                               static_cast<T *>(nullptr), slot_bits, H.pass_w[p], p ? H.pass_end[p - 1] : 0,
                               H.pass_end[p], PauliTables{H.gx, H.goff, H.tz, H.tc}, d_partials, add);
            add = 1;
        }
    } else {
        const uint64_t N = uint64_t(1) << n, b = (N + kRedThreads - 1) / kRedThreads;
        blocks = unsigned(b < kRedBlocks ? b : kRedBlocks);
        hipLaunchKernelGGL(k_pauli_expect<T>, dim3(blocks), dim3(kRedThreads), 0, st, psi, N, H, d_partials);
    }
    hipLaunchKernelGGL(k_final<1>, dim3(1), dim3(kRedThreads), 0, st, d_partials, int(blocks), d_out);
    return hipGetLastError();
}

template <typename T>
hipError_t pauli_apply_t(const T *psi, T *out, int n, const PauliDev &H, hipStream_t st)
{
    if (H.tile_apply) {
        const int slot_bits = n - PauliTile<T>::PB;
        hipLaunchKernelGGL((k_pauli_tile<T, true>), dim3(pauli_tile_grid(slot_bits, 512)), dim3(kPauliTileThreads), 0, st,
                           psi, out, slot_bits, 3, 0, H.n_groups, PauliTables{H.gx, H.goff, H.tz, H.tc},
                           static_cast<double *>(nullptr), 0);
    } else {
        const uint64_t N = uint64_t(1) << n, b = (N + 255) / 256;
        hipLaunchKernelGGL(k_pauli_apply<T>, dim3(unsigned(b < 16384 ? b : 16384)), dim3(256), 0, st, psi, out, N, H);
    }
    return hipGetLastError();
}

}  // namespace

int pauli_passes(int n, int dtype, int *w)
{
    if (n < kPauliTileMin) {
        w[0] = 3;
        return 1;
    }
    const int slot_bits = n - (dtype == SV_C64 ? 1 : 0);
    int p = 0;
    for (int at = 3; p == 0 || at < slot_bits; at += kPauliWindow) w[p++] = std::min(at, slot_bits - kPauliWindow);
    return p;
}

int pauli_pass_of(uint64_t x, int dtype, int n_pass, const int *w)
{
    const uint64_t xs = dtype == SV_C64 ? x >> 1 : x;
    for (int p = 0; p < n_pass; ++p)
        if (!(xs & ~(uint64_t(7) | uint64_t(kPauliWinMask) << w[p]))) return p;
    return 0;
}

// Where the tiled kernels win.  An amplitude's thread costs 9 us a term and 9 us
// a group at 24 qubits of complex64 (the gather), hidden behind the reading of
// the state up to some 3 terms; a tile 20 us more than reading the state, 1.5 us a
// term and, for a group that no window holds, the same gather.  So what counts
// is terms and, twice, groups that the window holds; measured for one to 40
// terms on one X mask, on a position each, and random (us, amplitudes and tiles):
//   complex64, H psi: 24 qubits, Z terms, four 67 and 76, eight 103 and 78; X
//     terms, two 60 and 74, four 95 and 87; random, four 98 and 127, eight 174
//     and 166; 19 qubits, 16 X terms 27 and 27.
//   complex128: gathers of 16 bytes a lane gain nothing (24 qubits, 24 random
//     terms 668 and 734; eight Z 108 and 119, sixteen 176 and 122), until the
//     state outgrows the memory-side cache (26 qubits, two random 705 and 583).
//   <H>: a pass per window and one for the groups of none; two or three terms of
//     which half are in none read the state too often (24 qubits, two random
//     terms, complex64 84 and 95, complex128 84 and 133).
void pauli_choose(int n, int dtype, int n_terms, const uint64_t *gx, int n_groups, PauliDev &H)
{
    const bool c64 = dtype == SV_C64;
    int near = 0, none = 0;  // groups in H psi's window, groups in no window of <H>
    for (int g = 0; g < n_groups; ++g) {
        const uint64_t xs = (gx[g] & ~kPauliImag) >> (c64 ? 1 : 0);
        bool any = false;
        for (int p = 0; p < H.n_pass; ++p) {
            const bool in = !(xs & ~(uint64_t(7) | uint64_t(kPauliWinMask) << H.pass_w[p]));
            any = any || in;
            if (p == 0) near += in;
        }
        none += !any;
    }
    const int far = n_groups - near;
    bool apply;
    if (c64) apply = n_terms + 2 * near >= (n == 19 ? 40 : n >= 23 && n <= 25 ? 7 : 6);
    else if (n <= 21) apply = true;
    else if (n <= 25) apply = n_terms + 4 * near - 4 * far >= 12;
    else apply = n_terms > 1 || near > 0;
    H.tile_apply = n >= kPauliTileMin && apply;
    H.tile_expect = n >= kPauliTileMin && !(2 * none >= n_groups && n_terms <= (c64 ? 2 : 3) && n >= (c64 ? 24 : 22));
}

hipError_t launch_pauli_expect(int dtype, const void *psi, int n, const PauliDev &H, double *d_partials,
                               double *d_out, hipStream_t st)
{
    if (dtype == SV_C64) return pauli_expect_t(static_cast<const float *>(psi), n, H, d_partials, d_out, st);
    return pauli_expect_t(static_cast<const double *>(psi), n, H, d_partials, d_out, st);
}

hipError_t launch_dm_expect(int dtype, const void *rho, int n, const PauliDev &H, double *d_partials, double *d_out,
                            hipStream_t st)
{
    if (dtype == SV_C64)
        hipLaunchKernelGGL(k_dm_expect<float>, dim3(kRedBlocks), dim3(kRedThreads), 0, st, static_cast<const float *>(rho), n, H, d_partials);
    else
        hipLaunchKernelGGL(k_dm_expect<double>, dim3(kRedBlocks), dim3(kRedThreads), 0, st, static_cast<const double *>(rho), n, H, d_partials);
    hipLaunchKernelGGL(k_final<1>, dim3(1), dim3(kRedThreads), 0, st, d_partials, kRedBlocks, d_out);
    return hipGetLastError();
}

namespace {

int bins_grid(int n, int mh)
{
    const int tile_bits = n - std::min(n, kBinTileBits);
    return 1 << std::max(mh, std::min(tile_bits, 10));
}

}  // namespace

size_t weighted_bins_bytes(int n, const int *pos, int m)
{
    int mh = 0;
    for (int j = 0; j < m; ++j) mh += pos[j] >= std::min(n, kBinTileBits);
    return (sizeof(double) * size_t(bins_grid(n, mh))) << (m - mh);
}

hipError_t launch_weighted_bins(int dtype, const void *psi, int n, const int *pos, int m, const double (*w)[2],
                                double scale, double *d_partials, double *out, hipStream_t st)
{
    if (m < 0 || m > kMaxBins || m > n) return hipErrorInvalidValue;
    BinArgs a;
    a.n = n;
    a.nl = std::min(n, kBinTileBits);
    a.ml = a.mh = 0;
    for (int j = 0; j < m; ++j) {
        if (pos[j] < 0 || pos[j] >= n || (j && pos[j] <= pos[j - 1])) return hipErrorInvalidValue;
        if (pos[j] < a.nl) a.lpos[a.ml++] = pos[j];
        else a.hpos[a.mh++] = pos[j];
    }
    for (int p = 0; p < n; ++p) a.w[p][0] = w[p][0], a.w[p][1] = w[p][1];
    a.scale = scale;
    const int grid = bins_grid(n, a.mh);
    if (dtype == SV_C64)
        hipLaunchKernelGGL(k_weighted_bins<float>, dim3(grid), dim3(256), 0, st, static_cast<const float *>(psi), a, d_partials);
    else
        hipLaunchKernelGGL(k_weighted_bins<double>, dim3(grid), dim3(256), 0, st, static_cast<const double *>(psi), a, d_partials);
    hipLaunchKernelGGL(k_bins_final, dim3(((1 << m) + 3) / 4), dim3(256), 0, st, d_partials, a.ml, a.mh, grid, out);
    return hipGetLastError();
}

hipError_t launch_kraus_probs(int dtype, const void *psi, int n, const KrausDev &K, double *d_partials,
                              double *d_out, hipStream_t st)
{
    if (K.k < 1 || K.k > 3 || K.k > n || K.n_ops < 1 || K.n_ops > kMaxKraus) return hipErrorInvalidValue;
    const dim3 g(kRedBlocks), t(kRedThreads);
    const bool c64 = dtype == SV_C64;
    const float *pf = static_cast<const float *>(psi);
    const double *pd = static_cast<const double *>(psi);
    // complex64 with 16-byte loads (needs a pair of groups when position 0 is free)
    if (c64 && (K.pos[0] == 0 || n - K.k >= 1)) {
        const float4 *p4 = static_cast<const float4 *>(psi);
        const bool low0 = K.pos[0] == 0;
        switch (K.k) {
        case 1:
            if (low0) hipLaunchKernelGGL((k_kraus_probs_c64<1, true>), g, t, 0, st, p4, n, K, d_partials);
            else hipLaunchKernelGGL((k_kraus_probs_c64<1, false>), g, t, 0, st, p4, n, K, d_partials);
            break;
        case 2:
            if (low0) hipLaunchKernelGGL((k_kraus_probs_c64<2, true>), g, t, 0, st, p4, n, K, d_partials);
            else hipLaunchKernelGGL((k_kraus_probs_c64<2, false>), g, t, 0, st, p4, n, K, d_partials);
            break;
        default:
            if (low0) hipLaunchKernelGGL((k_kraus_probs_c64<3, true>), g, t, 0, st, p4, n, K, d_partials);
            else hipLaunchKernelGGL((k_kraus_probs_c64<3, false>), g, t, 0, st, p4, n, K, d_partials);
            break;
        }
        hipLaunchKernelGGL(k_final<kMaxKraus>, dim3(1), dim3(kRedThreads), 0, st, d_partials, kRedBlocks, d_out);
        return hipGetLastError();
    }
    switch (K.k) {
    case 1:
        if (c64) hipLaunchKernelGGL((k_kraus_probs<float, 1>), g, t, 0, st, pf, n, K, d_partials);
        else hipLaunchKernelGGL((k_kraus_probs<double, 1>), g, t, 0, st, pd, n, K, d_partials);
        break;
    case 2:
        if (c64) hipLaunchKernelGGL((k_kraus_probs<float, 2>), g, t, 0, st, pf, n, K, d_partials);
        else hipLaunchKernelGGL((k_kraus_probs<double, 2>), g, t, 0, st, pd, n, K, d_partials);
        break;
    default:
        if (c64) hipLaunchKernelGGL((k_kraus_probs<float, 3>), g, t, 0, st, pf, n, K, d_partials);
        else hipLaunchKernelGGL((k_kraus_probs<double, 3>), g, t, 0, st, pd, n, K, d_partials);
        break;
    }
    hipLaunchKernelGGL(k_final<kMaxKraus>, dim3(1), dim3(kRedThreads), 0, st, d_partials, kRedBlocks, d_out);
    return hipGetLastError();
}

hipError_t launch_pauli_apply(int dtype, const void *psi, void *out, int n, const PauliDev &H, hipStream_t st)
{
    if (dtype == SV_C64) return pauli_apply_t(static_cast<const float *>(psi), static_cast<float *>(out), n, H, st);
    return pauli_apply_t(static_cast<const double *>(psi), static_cast<double *>(out), n, H, st);
}

}  // namespace dev
}  // namespace sv
