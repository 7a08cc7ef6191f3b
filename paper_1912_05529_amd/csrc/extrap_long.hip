// Depth stepping beyond the register-tap kernels: sections of more than 2048 points and
// filters of more than 35 taps (any nx <= MIG_MAX_NX, any N <= MIG_MAX_NTAPS).
//
// As in the other depth-stepping kernels a workgroup owns a frequency for the whole
// depth range, its plane (two of them, ping-pong, zero halo) in LDS, and one barrier
// separates two depth steps.  A thread owns 4 or 2 adjacent outputs, or more runs of 4
// where the section is wider than the workgroup.  A thread's taps depend on what
// its wave sees in this depth row:
//   * every lane's outputs share one table entry (each lane its own): the taps of
//     that entry stay in registers, reloaded only when some lane's entry changes;
//   * some lane's outputs have different entries (a wave that an interface crosses,
//     or a velocity that varies from point to point): every output's taps are read
//     from the table (L1/L2) as the FIR goes, two taps per load, a pair ahead.
// The window slides through registers: per pair of taps one 16-byte LDS read on each
// side of the outputs.
//
// Bound by the FP32 instruction rate of the CUs that hold a workgroup (a multiply-add
// occupies a SIMD for 4 cycles, an add for 2).  3001 points, 101 frequencies, 300 depths,
// 35 taps, layered, without the rows' sum: 6430 -> 760 us (before: 256 threads, one output at a time, its taps
// read from the table every step).
#include <type_traits>
#include <utility>

#include "extrap_dev.hpp"

namespace mig {
namespace {

constexpr int kLongThreads = 768;  // three waves per SIMD: up to 168 registers

// Q outputs with the lane's taps h.
template <int M, int Q>
__device__ __forceinline__ void fir_shared(const float2* P, const float2 (&h)[M + 1], float2 (&o)[Q])
{
    Window<M, Q> W;
    W.P = P;
    W.begin();
#pragma unroll
    for (int q = 0; q < Q; ++q) o[q] = cmulf(h[0], W.w[W.PM + q]);
#pragma unroll
    for (int i = 0; i < (M + 1) / 2; ++i) {
        W.load_pair(i + W.kAhead);
#pragma unroll
        for (int n = 2 * i + 1; n <= (2 * i + 2 < M ? 2 * i + 2 : M); ++n)
#pragma unroll
            for (int q = 0; q < Q; ++q) o[q] = cfmaf(h[n], W.pair_sum(q, n), o[q]);
        __builtin_amdgcn_sched_barrier(0);
    }
}

// Q outputs, each with the taps of its own table row.
template <int M, int Q>
__device__ __forceinline__ void fir_mixed(const float2* P, const float2* (&row)[Q], float2 (&o)[Q])
{
    constexpr int NP = (M + 1) / 2;
    Window<M, Q> W;
    W.P = P;
    float2 h0[Q];
    v4f hp[2][Q];
#pragma unroll
    for (int q = 0; q < Q; ++q) h0[q] = load_global(row[q]);
    if (M > 0)
#pragma unroll
        for (int q = 0; q < Q; ++q) hp[0][q] = tap_pair(row[q], 1, M >= 2);
    W.begin();
#pragma unroll
    for (int q = 0; q < Q; ++q) o[q] = cmulf(h0[q], W.w[W.PM + q]);
#pragma unroll
    for (int i = 0; i < NP; ++i) {
        if (i + 1 < NP) {
#pragma unroll
            for (int q = 0; q < Q; ++q) hp[(i + 1) & 1][q] = tap_pair(row[q], 2 * i + 3, 2 * i + 4 <= M);
        }
        W.load_pair(i + W.kAhead);
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            const v4f h = hp[i & 1][q];
            o[q] = cfmaf(make_float2(h.x, h.y), W.pair_sum(q, 2 * i + 1), o[q]);
            if (2 * i + 2 <= M) o[q] = cfmaf(make_float2(h.z, h.w), W.pair_sum(q, 2 * i + 2), o[q]);
        }
        __builtin_amdgcn_sched_barrier(0);
    }
}

template <int M, int Q>
__global__ void __launch_bounds__(kLongThreads) k_extrap_long(BatchArgs a)
{
    extern __shared__ float4 smem4[];
    const bool rows_on = a.rows != 0;
    if (rows_on && (int)blockIdx.x < a.nred) {
        reduce_role(a, blockIdx.x, reinterpret_cast<int*>(smem4));
        return;
    }
    const ItemDev it = item_of(a, blockIdx.x - (rows_on ? a.nred : 0));
    const SecDev S = sec_of(a, it.sec);
    float2* const sm = reinterpret_cast<float2*>(smem4);
    const int nx = S.nx, nw = S.nw, T = blockDim.x, t = threadIdx.x;
    const int r = it.r0;  // one frequency per workgroup: always inside the section
    const int LB = long_plane(nx, M), H = long_halo(M);
    const int nrun = (nx + Q * T - 1) / (Q * T);  // runs of outputs per thread
    const double ar = S.omega[r] / a.dk;

    for (int i = t; i < 2 * LB; i += T) sm[i] = make_float2(0.0f, 0.0f);
    __syncthreads();
    for (int x = t; x < nx; x += T) sm[H + x] = S.win[(size_t)x * nw + r];

    // The state of a run: kept from step to step when it is the only one.
    int j[Q];            // table entries of its outputs
    bool mixed = false;  // some lane's outputs have different entries
    float2 h[M + 1];     // else the lanes' taps
    // slowness of a run's outputs in one row; lanes past nx read the section's first
    const auto slowness = [&](const double* sp, int s, double (&v)[Q]) {
        const int x0 = Q * (t + s * T), x = x0 < nx ? x0 : 0;
#pragma unroll
        for (int q = 0; q < Q; q += 2) {
            const double2 p = load_global(reinterpret_cast<const double2*>(sp + x + q));
            v[q] = p.x;
            v[q + 1] = p.y;
        }
    };
    // the state where the slowness changed (or always)
    const auto update = [&](const double (&v)[Q], bool always) {
        bool chg = always;
#pragma unroll
        for (int q = 0; q < Q; ++q) chg = chg || slowness_changed(v[q]);
        if (__builtin_amdgcn_ballot_w64(chg) == 0) return;
        bool differ = false;
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            j[q] = index_of_slowness(ar, a.b, a.nk, slowness_value(v[q]));
            differ = differ || j[q] != j[0];
        }
        mixed = __builtin_amdgcn_ballot_w64(differ) != 0;
        if (!mixed) {
            const float2* row = a.tab + (size_t)j[0] * (M + 1);
#pragma unroll
            for (int n = 0; n <= M; ++n) h[n] = load_global(row + n);
        }
    };
    double v[Q];
    slowness(S.slow, 0, v);
    update(v, true);
    __syncthreads();
    // Memory operations of a step: the partial row of the step before, the next row's
    // slowness (both at its start), the taps that follow from it (at its end).  The one
    // wait at the start of a step finds all but those taps long complete; a row stored
    // at the end of its own step would be waited for by the next update (a
    // write-through to memory: 1125 against 977 us at 3001 points with reducers beside).
    float re[Q] = {};    // real parts of the last step's outputs (one run only)
    const auto store_row = [&](int k, int x0, const float (&v)[Q]) {
        if (x0 < nx) {  // the row stride holds whole runs of Q
            float* pr = S.part + ((size_t)k * nw + r) * S.ldp + x0;
            // Without reducers in the launch nobody reads the rows before its end: one
            // streaming store (write-through pairs 1026, plain 869, streaming 845 us
            // with the rows summed after the launch, 749 without rows).
            if (a.nred > 0) {
#pragma unroll
                for (int q = 0; q < Q; q += 2) store_partial2(pr + q, v[q], v[q + 1]);
            } else if constexpr (Q == 4) {
                __builtin_nontemporal_store(v4f{v[0], v[1], v[2], v[3]}, as_global(reinterpret_cast<v4f*>(pr)));
            } else {
                typedef float v2f __attribute__((ext_vector_type(2)));
                __builtin_nontemporal_store(v2f{v[0], v[1]}, as_global(reinterpret_cast<v2f*>(pr)));
            }
        }
    };
    for (int k = 0; k < S.nsteps; ++k) {
        wait_vmem_all();
        if (nrun == 1) {
            if (rows_on && k >= 1) store_row(k - 1, Q * t, re);
            // flagged where it differs from this row's
            slowness(S.slow + (size_t)(k + 1 < S.nsteps ? k + 1 : k) * S.ldp, 0, v);
        }
        for (int s = 0; s < nrun; ++s) {
            const int x0 = Q * (t + s * T);
            if (__builtin_amdgcn_readfirstlane(x0) >= nx) break;  // the whole wave is past nx
            if (nrun > 1) {
                slowness(S.slow + (size_t)k * S.ldp, s, v);
                update(v, true);
            }
            const float2* P = sm + (k & 1) * LB + H + (x0 < nx ? x0 : 0);
            float2 o[Q];
            if (mixed) {
                const float2* row[Q];
#pragma unroll
                for (int q = 0; q < Q; ++q) row[q] = a.tab + (size_t)j[q] * (M + 1);
                fir_mixed<M, Q>(P, row, o);
                // the taps are loaded again before they are used: nothing to keep
#pragma unroll
                for (int n = 0; n <= M; ++n) asm volatile("" : "=v"(h[n].x), "=v"(h[n].y));
            } else {
                fir_shared<M, Q>(P, h, o);
            }
            float2* dst = sm + ((k + 1) & 1) * LB + H + x0;
#pragma unroll
            for (int q = 0; q < Q; ++q) {
                if (x0 + q < nx) dst[q] = o[q];
                re[q] = o[q].x;
            }
            if (nrun > 1 && rows_on) store_row(k, x0, re);
        }
        if (nrun == 1 && k + 1 < S.nsteps) update(v, false);
        __syncthreads();
        if (rows_on && publishes_at(k)) publish_block(a, S, k / kPublish - 1);
    }
    if (rows_on) {
        if (nrun == 1) store_row(S.nsteps - 1, Q * t, re);
        wait_vmem_all();
        __syncthreads();
        for (int b = published_in_loop(S.nsteps); b * kPublish < S.nsteps; ++b) publish_block(a, S, b);
    }
    if (S.wout) {
        const float2* src = sm + (S.nsteps & 1) * LB + H;
        for (int x = t; x < nx; x += T) S.wout[(size_t)x * nw + r] = src[x];
    }
}

template <int M, int Q>
int launch_long_as(const BatchArgs& a, int threads, size_t lds, hipStream_t s)
{
    if (lds > 65536 &&
        hipFuncSetAttribute(reinterpret_cast<const void*>(&k_extrap_long<M, Q>),
                            hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds) != hipSuccess)
        return MIG_E_DEVICE;
    hipLaunchKernelGGL((k_extrap_long<M, Q>), dim3(a.nitems + a.nred), dim3(threads), lds, s, a);
    return hipGetLastError() == hipSuccess ? MIG_OK : MIG_E_DEVICE;
}

template <int M>
int launch_long_m(const BatchArgs& a, int max_nx, hipStream_t s)
{
    // Two outputs per thread while one run holds the section that way (only filters of
    // more than 35 taps come here with so few points): twice the waves to hide latency;
    // else four, for which a window read serves twice the outputs.
    const int Q = max_nx <= 2 * kLongThreads ? 2 : 4;
    int threads = ((max_nx + Q - 1) / Q + 63) / 64 * 64;
    if (threads > kLongThreads) threads = kLongThreads;
    const size_t lds = (size_t)2 * long_plane(max_nx, M) * sizeof(float2);
    if constexpr (M >= 18)
        if (Q == 2) return launch_long_as<M, 2>(a, threads, lds, s);
    return launch_long_as<M, 4>(a, threads, lds, s);
}

template <int... M>
int launch_long_any(std::integer_sequence<int, M...>, const BatchArgs& a, int max_nx, hipStream_t s)
{
    int rc = MIG_E_ARG;
    (void)((a.M == M ? (rc = launch_long_m<M>(a, max_nx, s), true) : false) || ...);
    return rc;
}

}  // namespace

int launch_general(const BatchArgs& a, int max_nx, hipStream_t s)
{
    return launch_long_any(std::make_integer_sequence<int, MIG_MAX_NTAPS / 2 + 1>{}, a, max_nx, s);
}

}  // namespace mig
