// Adjoint gradients.
//
// E(theta) = <psi|H|psi>, psi = U_G..U_1 psi_0.  With phi = U_{g+1}^+..U_G^+ psi
// and lam = U_{g+1}^+..U_G^+ H psi, and a rotation U_g = exp(-i theta P / 2),
//   dE/dtheta_g = 2 Re <lam| dU_g/dtheta |phi_{g-1}> = 2 Re <lam| (-i/2) P |phi>
//               = Im <lam|P|phi>.
// The sweep (api.hip) undoes the gates on both states, two buffers and no
// stored trajectory, and stops at runs of one-qubit gates to take the sums
// below.
#include <hip/hip_runtime.h>

#include <type_traits>

#include "device.h"
#include "kernels.h"

namespace sv {
namespace dev {

namespace {

// Transition sums of qubits q between lam and phi: with M[a][b] = sum over the
// other qubits of conj(lam_a) phi_b (a, b the values of q), the kernel gives
//   S = M00 + M11, Z = M00 - M11, A = M01 + M10, B = M01 - M10,
// from which <lam|O|phi> follows for any operator O on q.  One pass serves all
// one-qubit gates of a run, however many there are on a qubit: a rotation's
// generator P is seen through the run's later gates V on its qubit as
// V P V^dagger.
//
// What bounds it: a partner load (from L2 or the memory-side cache) and four
// FP64 multiply-adds per amplitude and qubit.  A thread takes 2 (tiny states:
// 1) slots of 16 bytes that differ in the top index bits and works on up to
// kTransQubits qubits (blockIdx.y: the next ones).  The per-rotation form, a
// pass over both states for every 16 rotations and the rotations of different
// axes apart, took 32 us a pass at 20 qubits and four passes a layer of 20 RY
// and 20 RZ; this takes
// 29 us for the layer.
struct TransArgs {
    int nq;
    int q[SV_MAX_QUBITS_C64];
};

template <typename T, int LOGR, int Q>
__global__ void __launch_bounds__(kRedThreads) k_transitions(const T *__restrict__ phi_, const T *__restrict__ lam_,
                                                            int slot_bits, const TransArgs a,
                                                            double *__restrict__ partials)
{
    using Slot = typename std::conditional<sizeof(T) == 4, vf4, vd2>::type;
    constexpr int NA = sizeof(T) == 4 ? 2 : 1, PB = NA - 1, R = 1 << LOGR;
    const Slot *__restrict__ phi = reinterpret_cast<const Slot *>(phi_);
    const Slot *__restrict__ lam = reinterpret_cast<const Slot *>(lam_);
    const int q0 = int(blockIdx.y) * Q, nq = a.nq - q0 < Q ? a.nq - q0 : Q;
    double sum[2] = {0.0, 0.0}, z[Q][2], s[Q][2], d[Q][2];
#pragma unroll
    for (int k = 0; k < Q; ++k) z[k][0] = z[k][1] = s[k][0] = s[k][1] = d[k][0] = d[k][1] = 0.0;
    const uint64_t U = uint64_t(1) << (slot_bits - LOGR);
    for (uint64_t u = uint64_t(blockIdx.x) * kRedThreads + threadIdx.x; u < U; u += uint64_t(gridDim.x) * kRedThreads) {
        auto slot = [&](int r) { return u | uint64_t(r) << (slot_bits - LOGR); };
        double lr[R][NA], li[R][NA];  // lam
        double tr[R][2], dp[2] = {0.0, 0.0};  // conj(lam) phi of each slot; first less second half over all of them
#pragma unroll
        for (int r = 0; r < R; ++r) {
            double fr[NA], fi[NA];
            slot_amps(lam[slot(r)], lr[r], li[r]);
            slot_amps(phi[slot(r)], fr, fi);
            double p[NA][2];
#pragma unroll
            for (int b = 0; b < NA; ++b) {
                p[b][0] = fma(lr[r][b], fr[b], li[r][b] * fi[b]);
                p[b][1] = fma(lr[r][b], fi[b], -(li[r][b] * fr[b]));
            }
#pragma unroll
            for (int c = 0; c < 2; ++c) {
                tr[r][c] = NA == 1 ? p[0][c] : p[0][c] + p[NA - 1][c];
                if (NA == 2) dp[c] += p[0][c] - p[NA - 1][c];
                sum[c] += tr[r][c];
            }
        }
#pragma unroll
        for (int k = 0; k < Q; ++k) {
            if (k >= nq) break;  // uniform
            __builtin_amdgcn_sched_barrier(0);  // one qubit's loads at a time: all of them at once take 484 registers
            const int q = a.q[q0 + k];
            const bool pair = PB && q == 0;  // the partner is the slot's other half
            const int sb = q - PB;
            Slot f[R];
#pragma unroll
            for (int r = 0; r < R; ++r) f[r] = phi[pair ? slot(r) : slot(r) ^ (uint64_t(1) << sb)];
#pragma unroll
            for (int r = 0; r < R; ++r) {
                double fr[NA], fi[NA], t[NA][2];
                slot_amps(f[r], fr, fi);
                const double sgn = !pair && (slot(r) >> sb) & 1u ? -1.0 : 1.0;
#pragma unroll
                for (int b = 0; b < NA; ++b) {
                    const double gr = pair ? fr[NA - 1 - b] : fr[b], gi = pair ? fi[NA - 1 - b] : fi[b];
                    t[b][0] = fma(lr[r][b], gr, li[r][b] * gi);
                    t[b][1] = fma(lr[r][b], gi, -(li[r][b] * gr));
                }
#pragma unroll
                for (int c = 0; c < 2; ++c) {
                    const double both = NA == 1 ? t[0][c] : t[0][c] + t[NA - 1][c];
                    s[k][c] += both;
                    d[k][c] = NA == 2 && pair ? d[k][c] + (t[0][c] - t[NA - 1][c]) : fma(sgn, both, d[k][c]);
                    if (!pair) z[k][c] = fma(sgn, tr[r][c], z[k][c]);
                }
            }
            if (pair) {
                z[k][0] += dp[0];
                z[k][1] += dp[1];
            }
        }
    }
    // workgroup sums through LDS: value v's 256 entries in 8 strided chains, then
    // a butterfly (64 lanes' butterflies of every value took 4 us); per qubit
    // (S, Z, A, B)
    constexpr int kValues = 2 + 6 * Q;
    __shared__ double sh[kValues][kRedThreads];
    const int tid = threadIdx.x;
    sh[0][tid] = sum[0];
    sh[1][tid] = sum[1];
#pragma unroll
    for (int k = 0; k < Q; ++k)
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            sh[2 + 6 * k + c][tid] = z[k][c];
            sh[4 + 6 * k + c][tid] = s[k][c];
            sh[6 + 6 * k + c][tid] = d[k][c];
        }
    __syncthreads();
    static_assert(8 * kValues <= kRedThreads, "one thread per chain");
    double v = 0.0;
    if (tid < 8 * kValues)
        for (int i = tid & 7; i < kRedThreads; i += 8) v += sh[tid >> 3][i];
#pragma unroll
    for (int o = 4; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    __syncthreads();
    if (tid < 8 * kValues && (tid & 7) == 0) sh[tid >> 3][0] = v;
    __syncthreads();
    if (tid < 8 * nq) {
        const int k = tid >> 3, c = tid & 7;
        partials[(size_t(q0 + k) * gridDim.x + blockIdx.x) * 8 + c] = sh[c < 2 ? c : 6 * k + c][0];
    }
}

// One step of a sweep whose run has one qubit with parameters and whose gates
// form one block of K qubits, that one among them: the sums above from the
// block's own amplitudes, then the block's dagger on both states, in one read
// and one write of each.  Local bit 0 is the qubit.
// What bounds it: the copy of both states (24 qubits: 512 MiB in 94 us a step),
// or a launch where they are small.  A sweep of steps of one RX and one CZ, the
// sums and the block as two launches and as this one: 14.9 and 10.7 us a step at
// 16 qubits, 26.3 and 15.7 at 20, 149 and 94 at 24.
template <typename T, int K>
struct StepArgs {
    int sorted[K], at[K];              // the positions, ascending and by local bit
    T m[2 << (2 * K)];                 // row-major (re, im)
};

template <typename T, int K>
__global__ void __launch_bounds__(kRedThreads) k_transition_step(T *__restrict__ phi, T *__restrict__ lam,
                                                                uint64_t groups, const StepArgs<T, K> a,
                                                                double *__restrict__ partials)
{
    constexpr int D = 1 << K;
    double S[2] = {0.0, 0.0}, Z[2] = {0.0, 0.0}, A[2] = {0.0, 0.0}, B[2] = {0.0, 0.0};
    for (uint64_t g = uint64_t(blockIdx.x) * kRedThreads + threadIdx.x; g < groups; g += uint64_t(gridDim.x) * kRedThreads) {
        uint64_t base = g, off[D];
#pragma unroll
        for (int j = 0; j < K; ++j) {
            const uint64_t low = base & ((uint64_t(1) << a.sorted[j]) - 1);
            base = (base - low) << 1 | low;
        }
#pragma unroll
        for (int x = 0; x < D; ++x) {
            off[x] = base;
#pragma unroll
            for (int j = 0; j < K; ++j)
                if ((x >> j) & 1) off[x] |= uint64_t(1) << a.at[j];
        }
        T fr[D], fi[D], lr[D], li[D];
#pragma unroll
        for (int x = 0; x < D; ++x) {
            fr[x] = phi[2 * off[x]];
            fi[x] = phi[2 * off[x] + 1];
            lr[x] = lam[2 * off[x]];
            li[x] = lam[2 * off[x] + 1];
        }
        // conj(lam_x) phi_y
        auto re = [&](int x, int y) { return fma(double(lr[x]), double(fr[y]), double(li[x]) * double(fi[y])); };
        auto im = [&](int x, int y) { return fma(double(lr[x]), double(fi[y]), -(double(li[x]) * double(fr[y]))); };
#pragma unroll
        for (int x = 0; x < D; x += 2) {
            const double r00 = re(x, x), r11 = re(x + 1, x + 1), r01 = re(x, x + 1), r10 = re(x + 1, x);
            const double i00 = im(x, x), i11 = im(x + 1, x + 1), i01 = im(x, x + 1), i10 = im(x + 1, x);
            S[0] += r00 + r11; Z[0] += r00 - r11; A[0] += r01 + r10; B[0] += r01 - r10;
            S[1] += i00 + i11; Z[1] += i00 - i11; A[1] += i01 + i10; B[1] += i01 - i10;
        }
        auto undo = [&](T *__restrict__ psi, const T (&vr)[D], const T (&vi)[D]) {
#pragma unroll
            for (int x = 0; x < D; ++x) {
                T sr = 0, si = 0;
#pragma unroll
                for (int y = 0; y < D; ++y) {
                    const T mr = a.m[2 * (x * D + y)], mi = a.m[2 * (x * D + y) + 1];
                    sr = fma(mr, vr[y], sr);
                    sr = fma(-mi, vi[y], sr);
                    si = fma(mr, vi[y], si);
                    si = fma(mi, vr[y], si);
                }
                psi[2 * off[x]] = sr;
                psi[2 * off[x] + 1] = si;
            }
        };
        undo(phi, fr, fi);
        undo(lam, lr, li);
    }
    // as in k_transitions: 8 strided chains a value, then a butterfly
    __shared__ double sh[8][kRedThreads];
    const int tid = threadIdx.x;
#pragma unroll
    for (int c = 0; c < 2; ++c) {
        sh[c][tid] = S[c];
        sh[2 + c][tid] = Z[c];
        sh[4 + c][tid] = A[c];
        sh[6 + c][tid] = B[c];
    }
    __syncthreads();
    if (tid < 64) {
        double v = 0.0;
        for (int i = tid & 7; i < kRedThreads; i += 8) v += sh[tid >> 3][i];
#pragma unroll
        for (int o = 4; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
        if ((tid & 7) == 0) partials[size_t(blockIdx.x) * 8 + (tid >> 3)] = v;
    }
}

// out[slot][c] = sum over the slot's blocks of partials (fixed order).
__global__ void __launch_bounds__(64) k_transitions_final(const double *__restrict__ partials, int blocks,
                                                          double *__restrict__ out)
{
    const double *p = partials + size_t(blockIdx.x) * blocks * 8;
    const int c = threadIdx.x & 7;
    double v = 0.0;
    for (int b = threadIdx.x >> 3; b < blocks; b += 8) v += p[size_t(b) * 8 + c];
#pragma unroll
    for (int o = 32; o >= 8; o >>= 1) v += __shfl_xor(v, o, 64);
    if (threadIdx.x < 8) out[size_t(blockIdx.x) * 8 + c] = v;
}

template <typename T>
hipError_t transitions_t(const TransArgs &a, const T *phi, const T *lam, int n, double *d_partials, hipStream_t st)
{
    const int slot_bits = n - (sizeof(T) == 4 ? 1 : 0);
    const int per = a.nq == 1 ? 1 : kTransQubits;
    const dim3 grid(unsigned(transition_blocks(n)), unsigned((a.nq + per - 1) / per));
    auto launch = [&](auto kernel) { hipLaunchKernelGGL(kernel, grid, dim3(kRedThreads), 0, st, phi, lam, slot_bits, a, d_partials); };
    if (slot_bits >= 10) {
        if (per == 1) launch(k_transitions<T, 1, 1>);
        else launch(k_transitions<T, 1, kTransQubits>);
    } else {
        if (per == 1) launch(k_transitions<T, 0, 1>);
        else launch(k_transitions<T, 0, kTransQubits>);
    }
    return hipGetLastError();
}

template <typename T, int K>
hipError_t transition_step_t(const int *sorted_q, const cd *m, int qubit, T *phi, T *lam, int n, double *part,
                             hipStream_t st)
{
    constexpr int D = 1 << K;
    StepArgs<T, K> a;
    int bit[K], own = -1, next = 1;  // the block's canonical bit of each local bit
    for (int j = 0; j < K; ++j) {
        a.sorted[j] = sorted_q[j];
        if (sorted_q[j] == qubit) own = j;
    }
    if (own < 0) return hipErrorInvalidValue;
    bit[0] = own;
    for (int j = 0; j < K; ++j)
        if (j != own) bit[next++] = j;
    int canon[D];
    for (int x = 0; x < D; ++x) {
        canon[x] = 0;
        for (int j = 0; j < K; ++j)
            if ((x >> j) & 1) canon[x] |= 1 << bit[j];
    }
    for (int j = 0; j < K; ++j) a.at[j] = sorted_q[bit[j]];
    for (int x = 0; x < D; ++x)
        for (int y = 0; y < D; ++y) {
            a.m[2 * (x * D + y)] = T(m[canon[x] * D + canon[y]].real());
            a.m[2 * (x * D + y) + 1] = T(m[canon[x] * D + canon[y]].imag());
        }
    hipLaunchKernelGGL((k_transition_step<T, K>), dim3(unsigned(transition_blocks(n))), dim3(kRedThreads), 0, st, phi, lam,
                       uint64_t(1) << (n - K), a, part);
    return hipGetLastError();
}

}  // namespace

int transition_blocks(int n)
{
    // 16 amplitudes a thread, so that the sums over a workgroup do not outweigh
    // its own work; down to 4 below 18 qubits, where the workgroups are few and
    // each waits for its loads one after another
    const uint64_t N = uint64_t(1) << n, few = N / (4 * kRedThreads), many = N / (16 * kRedThreads);
    const uint64_t b = many >= 64 ? many : few < 64 ? few : 64;
    return int(b < 1 ? 1 : b > 512 ? 512 : b);
}

hipError_t launch_transitions(int dtype, int nq, const int *q, const void *phi, const void *lam, int n,
                              double *d_partials, int slot0, hipStream_t st)
{
    if (nq < 1 || nq > n || n > SV_MAX_QUBITS_C64) return hipErrorInvalidValue;
    TransArgs a;
    a.nq = nq;
    for (int k = 0; k < nq; ++k) {
        if (q[k] < 0 || q[k] >= n) return hipErrorInvalidValue;
        a.q[k] = q[k];
    }
    double *part = d_partials + size_t(slot0) * transition_blocks(n) * 8;
    if (dtype == SV_C64)
        return transitions_t(a, static_cast<const float *>(phi), static_cast<const float *>(lam), n, part, st);
    return transitions_t(a, static_cast<const double *>(phi), static_cast<const double *>(lam), n, part, st);
}

hipError_t launch_transition_step(int dtype, int k, const int *sorted_q, const cd *m, int qubit, void *phi, void *lam,
                                  int n, double *d_partials, int slot, hipStream_t st)
{
    if (k < 1 || k > 3 || k > n || n > SV_MAX_QUBITS_C64) return hipErrorInvalidValue;
    for (int j = 0; j < k; ++j)
        if (sorted_q[j] < 0 || sorted_q[j] >= n || (j && sorted_q[j] <= sorted_q[j - 1])) return hipErrorInvalidValue;
    double *part = d_partials + size_t(slot) * transition_blocks(n) * 8;
    auto run = [&](auto *p, auto *l) {
        if (k == 1) return transition_step_t<std::remove_reference_t<decltype(*p)>, 1>(sorted_q, m, qubit, p, l, n, part, st);
        if (k == 2) return transition_step_t<std::remove_reference_t<decltype(*p)>, 2>(sorted_q, m, qubit, p, l, n, part, st);
        return transition_step_t<std::remove_reference_t<decltype(*p)>, 3>(sorted_q, m, qubit, p, l, n, part, st);
    };
    if (dtype == SV_C64) return run(static_cast<float *>(phi), static_cast<float *>(lam));
    return run(static_cast<double *>(phi), static_cast<double *>(lam));
}

hipError_t launch_transitions_final(const double *d_partials, int n_slots, int n, double *out, hipStream_t st)
{
    if (n_slots <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_transitions_final, dim3(n_slots), dim3(64), 0, st, d_partials, transition_blocks(n), out);
    return hipGetLastError();
}

}  // namespace dev
}  // namespace sv
