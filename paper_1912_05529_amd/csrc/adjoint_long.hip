// Adjoint (demigration) beyond the kernels of adjoint.hip: sections of more than 1024
// points whose velocity changes too often for the folded kernel, or of more than 1536;
// filters of more than 35 taps; single-tap filters; any velocity.
//
//     (E^H q)[x] = sum_{n=-M..M} conj(h_{j(x+n)}[|n|]) q[x+n]
//
// A workgroup owns one frequency and walks the depths upward, the plane (two of them,
// ping-pong, zero halo) in LDS, one barrier per step; a thread owns 2 adjacent outputs
// or runs of 4.  What a wave does depends on the points its outputs depend
// on (M more on each side):
//   * they share one table entry: the folded FIR with that entry's conjugated taps,
//     which are the same for the whole wave and come through scalar loads;
//   * else the products g_m[y] = conj(h_{j(y)}[m]) q[y] of those points, some taps at a
//     time: each lane forms those of its own points and of one point of the halo
//     (2 M <= 62 lanes), writes them to the wave's rows in LDS and adds g_m[x-m] +
//     g_m[x+m] from them (LDS keeps a wave's accesses in order, so no barrier is
//     needed).  Taps are read from the table two per load, some taps ahead.  (One FIR
//     per entry over the points that have it, for two or three entries, was 10 % slower
//     at 45 taps.)
//
// Bound by the FP32 instruction rate of the CUs that hold a workgroup, and in waves of
// the second kind by the round trips of their product rows.  2000 points, 100
// frequencies, 200 depths, 25 taps, layered: 2550 -> 885 us; 645 points, 120 frequencies,
// 300 depths, 45 taps: 2567 -> 855 us; 1501 points, 101 frequencies, 300 depths, 35 taps,
// a velocity that varies from point to point: 3600 -> 1380 us (before: products of every
// point through LDS a chunk of taps at a time, taps read from the table every step).
#include <type_traits>
#include <utility>

#include "extrap_dev.hpp"

namespace mig {
namespace {

constexpr int kAdjLongThreads = 768;
constexpr size_t kLdsBytes = 160 * 1024;

// Points of a wave's product row: its 64 Q outputs and a halo on each side, then a place
// for the products of lanes that have no halo point.
__host__ __device__ constexpr int adj_row_len(int M, int Q) { return 64 * Q + 2 * long_halo(M) + 2; }

// LDS of a workgroup: two planes, R product rows per wave.
__host__ __device__ constexpr size_t adj_long_lds(int nx, int M, int Q, int R, int threads)
{
    return (size_t)(2 * long_plane(nx, M) + threads / 64 * R * adj_row_len(M, Q)) * sizeof(float2);
}

__device__ __forceinline__ float2 cmulc(float2 h, float2 u)  // conj(h) u
{
    return make_float2(fmaf(h.y, u.y, h.x * u.x), fmaf(-h.y, u.x, h.x * u.y));
}

__device__ __forceinline__ float2 cfmac(float2 h, float2 s, float2 acc)  // acc + conj(h) s
{
    acc.x = fmaf(h.x, s.x, acc.x);
    acc.x = fmaf(h.y, s.y, acc.x);
    acc.y = fmaf(h.x, s.y, acc.y);
    acc.y = fmaf(-h.y, s.x, acc.y);
    return acc;
}

// Folded FIR with the conjugated taps of table row `row` (the same in every lane); odd
// and even taps in two sums, which halves the chains of additions.
template <int M, int Q>
__device__ __forceinline__ void fir_conj(const float2* P, const float2* row, float2 (&o)[Q])
{
    typedef const __attribute__((address_space(4))) float* const_f32_ptr;
    const const_f32_ptr ht = (const_f32_ptr)reinterpret_cast<const float*>(row);
    const auto tap = [&](int n) { return make_float2(ht[2 * n], ht[2 * n + 1]); };
    Window<M, Q> W;
    W.P = P;
    W.begin();
    float2 odd[Q];
#pragma unroll
    for (int q = 0; q < Q; ++q) {
        o[q] = cmulc(tap(0), W.w[W.PM + q]);
        odd[q] = make_float2(0.0f, 0.0f);
    }
#pragma unroll
    for (int i = 0; i < (M + 1) / 2; ++i) {
        W.load_pair(i + W.kAhead);
#pragma unroll
        for (int q = 0; q < Q; ++q) odd[q] = cfmac(tap(2 * i + 1), W.pair_sum(q, 2 * i + 1), odd[q]);
        if (2 * i + 2 <= M)
#pragma unroll
            for (int q = 0; q < Q; ++q) o[q] = cfmac(tap(2 * i + 2), W.pair_sum(q, 2 * i + 2), o[q]);
        __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int q = 0; q < Q; ++q) o[q] = cadd(o[q], odd[q]);
}

// Q consecutive values of a product row from an index of either parity.
template <int Q>
__device__ __forceinline__ void row_get(const float2* g, int m, bool even, float2 (&v)[Q])
{
    if (!even) v[0] = g[m];
#pragma unroll
    for (int q = even ? 0 : 1; q + 1 < Q; q += 2) {
        const v4f a = *reinterpret_cast<const v4f*>(g + m + q);
        v[q] = make_float2(a.x, a.y);
        v[q + 1] = make_float2(a.z, a.w);
    }
    if (!even) v[Q - 1] = g[m + Q - 1];
}

// Products of the wave's points through its rows G (index PM + i = point xw + i), R taps
// at a time, for lanes whose own points have values u and table rows `row`, and whose
// halo point has value uh, table row rowh and place ph.
template <int M, int Q, int R>
__device__ __forceinline__ void products(float2* G, int lane, const float2 (&u)[Q],
                                         const float2* const (&row)[Q], float2 uh,
                                         const float2* rowh, int ph, float2 (&o)[Q])
{
    constexpr int PM = long_halo(M), LR = adj_row_len(M, Q);
    constexpr int RP = R < 2 ? 2 : R;  // taps loaded at a time
    float2* const left = G + Q * lane;  // PM points left of its own: offsets are positive
    float2 h0[Q], odd[Q];
    v4f hp[RP / 2][Q + 1], hn[RP / 2][Q + 1];
#pragma unroll
    for (int q = 0; q < Q; ++q) h0[q] = load_global(row[q]);
    const auto fetch = [&](v4f (&h)[RP / 2][Q + 1], int m0) {  // taps m0 .. m0 + RP - 1
#pragma unroll
        for (int e = 0; e < RP / 2; ++e)
            if (m0 + 2 * e <= M) {
#pragma unroll
                for (int q = 0; q < Q; ++q) h[e][q] = tap_pair(row[q], m0 + 2 * e, m0 + 2 * e + 1 <= M);
                h[e][Q] = tap_pair(rowh, m0 + 2 * e, m0 + 2 * e + 1 <= M);
            }
    };
    if constexpr (M > 0) fetch(hp, 1);
#pragma unroll
    for (int q = 0; q < Q; ++q) {
        o[q] = cmulc(h0[q], u[q]);
        odd[q] = make_float2(0.0f, 0.0f);
    }
#pragma unroll
    for (int m0 = 1; m0 <= M; m0 += RP) {
        if (m0 + RP <= M) fetch(hn, m0 + RP);
#pragma unroll
        for (int c = 0; c < RP; c += R) {
            // R products per point to the rows, then all the sums that read them
#pragma unroll
            for (int e = c; e < c + R; ++e)
                if (m0 + e <= M) {
                    float2 g[Q + 1];
#pragma unroll
                    for (int q = 0; q <= Q; ++q) {
                        const v4f h = hp[e / 2][q];
                        g[q] = cmulc(e % 2 == 0 ? make_float2(h.x, h.y) : make_float2(h.z, h.w),
                                     q < Q ? u[q < Q ? q : 0] : uh);
                    }
                    float2* const w = left + (e - c) * LR + PM;
#pragma unroll
                    for (int q = 0; q < Q; q += 2)
                        *reinterpret_cast<v4f*>(w + q) = v4f{g[q].x, g[q].y, g[q + 1].x, g[q + 1].y};
                    G[(e - c) * LR + ph] = g[Q];
                }
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            float2 l[R][Q], r[R][Q];
#pragma unroll
            for (int e = c; e < c + R; ++e)
                if (m0 + e <= M) {
                    const int m = m0 + e;
                    row_get<Q>(left + (e - c) * LR, PM - m, m % 2 == 0, l[e - c]);
                    row_get<Q>(left + (e - c) * LR, PM + m, m % 2 == 0, r[e - c]);
                }
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
#pragma unroll
            for (int e = c; e < c + R; ++e)
                if (m0 + e <= M)
#pragma unroll
                    for (int q = 0; q < Q; ++q) {
                        float2& s = (m0 + e) % 2 == 0 ? o[q] : odd[q];
                        s = cadd(s, cadd(l[e - c][q], r[e - c][q]));
                    }
            // the sums exist here: sunk to their use after the last tap, every value
            // read from the rows would stay in registers until then
#pragma unroll
            for (int q = 0; q < Q; ++q)
                asm volatile("" : "+v"(o[q].x), "+v"(o[q].y), "+v"(odd[q].x), "+v"(odd[q].y));
            __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
        for (int e = 0; e < RP / 2; ++e)
#pragma unroll
            for (int q = 0; q <= Q; ++q) hp[e][q] = hn[e][q];
    }
#pragma unroll
    for (int q = 0; q < Q; ++q) o[q] = cadd(o[q], odd[q]);
}

template <int M, int Q, int R>
__global__ void __launch_bounds__(kAdjLongThreads) k_demigrate_long(AdjArgs a)
{
    constexpr int H = long_halo(M), XW = 64 * Q;  // outputs per wave and run
    extern __shared__ float4 smem4[];
    // launched after the folded kernel: runs only when some row has more change points
    // than that kernel handles (the flag is uniform)
    if (a.dense && *as_global(a.dense) == 0) return;
    float2* const sm = reinterpret_cast<float2*>(smem4);
    const int nx = a.nx, nz = a.nz, nw = a.nw, T = blockDim.x, t = threadIdx.x, r = blockIdx.x;
    const int lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const int LB = long_plane(nx, M);
    float2* const G = sm + 2 * LB + wave * R * adj_row_len(M, Q);
    const int nrun = (nx + Q * T - 1) / (Q * T);
    const double ar = a.omega[r] / a.dk;

    for (int i = t; i < 2 * LB; i += T) sm[i] = make_float2(0.0f, 0.0f);
    __syncthreads();
    for (int x = t; x < nx; x += T)
        sm[((nz - 1) & 1) * LB + H + x] = make_float2((float)a.image[(size_t)(nz - 1) * nx + x], 0.0f);

    // The state of a run: kept from step to step when it is the only one.
    int j[Q], jh = 0;    // table entries of its own points and of its halo point
    bool same = false;   // all points the wave depends on share one entry
    // This lane's halo point: lanes 0 .. M-1 left of the wave's outputs, M .. 2M-1 right.
    const int hofs = lane < M ? lane - M : XW + lane - M;  // from the wave's first output
    const auto load_slow = [&](const double* sp, int xw, double (&v)[Q], double& vh) {
        const int x0 = xw + Q * lane, x = x0 < nx ? x0 : (nx - 1) / Q * Q;
        const int xh = xw + hofs;
#pragma unroll
        for (int q = 0; q < Q; q += 2) {
            const double2 p = load_global(reinterpret_cast<const double2*>(sp + x + q));
            v[q] = p.x;
            v[q + 1] = p.y;
        }
        vh = *as_global(sp + (xh < 0 ? 0 : (xh < nx ? xh : nx - 1)));
    };
    const auto update = [&](const double (&v)[Q], double vh, bool always) {
        bool chg = always || slowness_changed(vh);
#pragma unroll
        for (int q = 0; q < Q; ++q) chg = chg || slowness_changed(v[q]);
        if (__builtin_amdgcn_ballot_w64(chg) == 0) return;
#pragma unroll
        for (int q = 0; q < Q; ++q) j[q] = index_of_slowness(ar, a.b, a.nk, slowness_value(v[q]));
        jh = index_of_slowness(ar, a.b, a.nk, slowness_value(vh));
        const int j0 = __builtin_amdgcn_readfirstlane(j[0]);
        bool differ = lane < 2 * M && jh != j0;
#pragma unroll
        for (int q = 0; q < Q; ++q) differ = differ || j[q] != j0;
        same = __builtin_amdgcn_ballot_w64(differ) == 0;
    };
    const auto load_image = [&](int k, int x0, double (&v)[Q]) {
        const double* p = a.image + (size_t)k * nx;
#pragma unroll
        for (int q = 0; q < Q; ++q) v[q] = *as_global(p + (x0 + q < nx ? x0 + q : nx - 1));
    };
    double v[Q], vh, im[Q];
    if (nz > 1 && nrun == 1) {
        load_slow(a.slow + (size_t)(nz - 2) * a.ldp, wave * XW, v, vh);
        load_image(nz - 2, Q * t, im);
        update(v, vh, true);
    }
    __syncthreads();
    for (int k = nz - 2; k >= 0; --k) {
        float add[Q];
        if (nrun == 1) {
            // the image row of this step, loaded a step ahead; then the next step's rows
            // (slowness flagged where it differs from this step's)
            wait_vmem_all();
            const int kn = k >= 1 ? k - 1 : 0;
#pragma unroll
            for (int q = 0; q < Q; ++q) add[q] = (float)im[q];
            load_slow(a.slow + (size_t)kn * a.ldp, wave * XW, v, vh);
            load_image(kn, Q * t, im);
        }
        const float2* const src = sm + ((k + 1) & 1) * LB + H;
        float2* const dst = sm + (k & 1) * LB + H;
        for (int s = 0; s < nrun; ++s) {
            const int xw = Q * s * T + wave * XW, x0 = xw + Q * lane;
            if (xw >= nx) break;  // the whole wave is past nx
            if (nrun > 1) {
                load_slow(a.slow + (size_t)k * a.ldp, xw, v, vh);
                load_image(k, x0, im);
                update(v, vh, true);
#pragma unroll
                for (int q = 0; q < Q; ++q) add[q] = (float)im[q];
            }
            const float2* const P = src + (x0 < nx ? x0 : 0);
            float2 o[Q];
            if (same) {
                fir_conj<M, Q>(P, a.tab + (size_t)__builtin_amdgcn_readfirstlane(j[0]) * (M + 1), o);
            } else {
                const float2* row[Q];
                float2 u[Q];
#pragma unroll
                for (int q = 0; q < Q; ++q) {
                    row[q] = a.tab + (size_t)j[q] * (M + 1);
                    u[q] = x0 < nx ? P[q] : make_float2(0.0f, 0.0f);  // zeros past nx - 1
                }
                const int xh = xw + hofs;
                const bool in = xh >= 0 && xh < nx;
                const float2 uh = src[in ? xh : 0];
                products<M, Q, R>(G, lane, u, row, in ? uh : make_float2(0.0f, 0.0f),
                                  a.tab + (size_t)jh * (M + 1),
                                  lane < 2 * M ? H + hofs : adj_row_len(M, Q) - 2, o);
            }
#pragma unroll
            for (int q = 0; q < Q; ++q)
                if (x0 + q < nx) dst[x0 + q] = make_float2(o[q].x + add[q], o[q].y);
        }
        if (nrun == 1 && k >= 1) update(v, vh, false);
        __syncthreads();
    }
    for (int x = t; x < nx; x += T) a.out[(size_t)x * nw + r] = sm[H + x];
}

template <int M, int Q, int R>
int launch_long_as(const AdjArgs& a, int threads, hipStream_t s)
{
    const size_t lds = adj_long_lds(a.nx, M, Q, R, threads);
    if (lds > 65536 &&
        hipFuncSetAttribute(reinterpret_cast<const void*>(&k_demigrate_long<M, Q, R>),
                            hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds) != hipSuccess)
        return MIG_E_DEVICE;
    hipLaunchKernelGGL((k_demigrate_long<M, Q, R>), dim3(a.nw), dim3(threads), lds, s, a);
    return hipGetLastError() == hipSuccess ? MIG_OK : MIG_E_DEVICE;
}

// Two outputs per thread while one run of them holds the section: with four, 1501 points
// are six waves, whose product waves set the step's time (layered: 1437 against 982 us);
// else four.
// Taps of products at a time: four with two outputs per thread, two with four (their
// registers), one where LDS does not hold two rows per wave beside the planes.
// (With four outputs the instances of 45 taps and more spill 2 to 40 of their 168
// registers, with two that of 63 taps 8: 4000 points, 60 depths, 60 frequencies, 55 taps, a
// velocity that varies from point to point, still 3.9 -> 1.06 ms.)
template <int M>
int launch_long(const AdjArgs& a, hipStream_t s)
{
    const int Q = a.nx <= 2 * kAdjLongThreads ? 2 : 4;
    int threads = ((a.nx + Q - 1) / Q + 63) / 64 * 64;
    if (threads > kAdjLongThreads) threads = kAdjLongThreads;
    if (Q == 2) return launch_long_as<M, 2, 4>(a, threads, s);
    if (adj_long_lds(a.nx, M, 4, 2, threads) <= kLdsBytes) return launch_long_as<M, 4, 2>(a, threads, s);
    return launch_long_as<M, 4, 1>(a, threads, s);
}

template <int... M>
int launch_any(std::integer_sequence<int, M...>, const AdjArgs& a, hipStream_t s)
{
    int rc = MIG_E_ARG;
    (void)((a.M == M ? (rc = launch_long<M>(a, s), true) : false) || ...);
    return rc;
}

static_assert(adj_long_lds(MIG_MAX_NX, MIG_MAX_NTAPS / 2, 4, 1, kAdjLongThreads) <= kLdsBytes &&
                  adj_long_lds(2 * kAdjLongThreads, MIG_MAX_NTAPS / 2, 2, 4, kAdjLongThreads) <= kLdsBytes,
              "LDS of the widest sections");

}  // namespace

int launch_demigrate(const AdjArgs& a, hipStream_t s)
{
    return launch_any(std::make_integer_sequence<int, MIG_MAX_NTAPS / 2 + 1>{}, a, s);
}

}  // namespace mig
