// Depth stepping (Eq. 1 with per-point filters), imaging and table look-up.
//
// Design (MI355X / gfx950):
//   * Frequencies never interact during extrapolation (Sec. II: the process
//     runs independently for each frequency), only through the image sum.  So
//     a frequency is owned by one workgroup for the whole depth range: its
//     plane (nx complex64, a few KB) stays in LDS, depth steps are separated by
//     a workgroup barrier instead of a kernel exit (the "block level
//     synchronization" the paper names as future work, Sec. V), and there is
//     no traffic between frequency workgroups.
//   * A workgroup item owns G frequencies of one section (G sub-groups of
//     `tsub` threads; G > 1 fills a workgroup when nx is small).  Items of many
//     sections of different nx, nz and nw run in one launch (the batched form).
//   * Lanes run along x (coalesced, conflict-free LDS windows); each thread
//     owns two (or four) adjacent outputs and reads its window with 16-byte LDS
//     loads.  Even taps are folded: h_n (u[x-n] + u[x+n]).
//   * Taps live in registers.  The filter of an output only changes when the
//     velocity under it changes (omega is fixed per sub-group), which in
//     layered media is a few times per column.  Two register sets alternate
//     between even and odd steps; the set for step k+1 is refilled during step
//     k, by waves some output of which changes its slowness.  The loads stand
//     between the stages of the FIR, whose arithmetic hides them; the slowness
//     is read two steps ahead, and a partial row is stored at the end of its
//     step (three and four outputs: at the start of the next) and first waited
//     for a step later.
//   * The look-up needs 1/v in FP64; it is computed once per (depth, x) by a
//     small pre-pass (shared by all frequencies) instead of once per refill.
//   * The image row needs a sum over frequencies, i.e. across workgroups.
//     Each frequency sub-group writes Re of its new plane (float32, exact) to a
//     partial buffer [step][omega][x], write-through; every kPublish steps the
//     workgroup publishes its progress (its stores complete, then a counter
//     increment).  Reducer workgroups in the same launch -- the first
//     workgroups of the grid, so they run beside the frequency workgroups from
//     the start even when items outnumber the CUs -- take blocks in the order
//     they are expected to be published, wait for a block of steps to be
//     published by every workgroup of the section, acquire, and sum it over
//     omega in increasing order in FP64, so images are run-to-run identical
//     and the reduction overlaps the extrapolation; the last block of a plain
//     launch is summed after it (k_rows) by the whole GPU.  Frequency
//     workgroups never wait on anyone; reducer waits are bounded: after
//     kStallTicks (or the caller's limit) without any publish in the launch,
//     the launch is abandoned as a whole -- every remaining task writes NaN
//     rows without waiting -- and the call's status word says so.
#include "extrap_dev.hpp"

namespace mig {
namespace {

template <int M>
__device__ __forceinline__ void load_taps(float2 (&h)[M + 1], const float2* __restrict__ row)
{
#pragma unroll
    for (int n = 0; n <= M; ++n) h[n] = row[n];
}

// slow[k][x] = slowness_of(vel[k][min(x, nx-1)]) for x < ldp, every section,
// with the sign bit set where it differs (bitwise) from row k - dist (when
// that row exists); also
// zeroes each section's block counters (one launch fewer before the depth
// stepping).
__global__ void k_slowness(BatchArgs a, int dist)
{
    const SecDev S = sec_of(a, blockIdx.y);
    // the section's published-block counters start the coming launch at zero
    if (S.cnt && blockIdx.x == 0)
        for (int i = threadIdx.x; i < (S.nsteps + kPublish - 1) / kPublish; i += blockDim.x)
            S.cnt[i] = 0;
    if (blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x == 0) {
        if (a.progress) {
            a.progress[0] = 0;
            a.progress[1] = 0;
        }
        if (a.status && a.reset_status) *a.status = 0;
    }
    double* slow = const_cast<double*>(S.slow);
    const size_t total = (size_t)S.nsteps * S.ldp;
    for (size_t e = (size_t)blockIdx.x * blockDim.x + threadIdx.x; e < total;
         e += (size_t)gridDim.x * blockDim.x) {
        size_t k = e / S.ldp;
        int x = (int)(e % S.ldp);
        const int xc = x < S.nx ? x : S.nx - 1;
        double v = slowness_of(S.vel[k * S.nx + xc]);
        long long bits = __double_as_longlong(v);
        // dist > 0: flag against the row dist steps earlier (depth stepping
        // downward); dist < 0: against the row -dist steps later (the adjoint
        // walks upward)
        const long long kr = (long long)k - dist;
        if (dist != 0 && kr >= 0 && kr < S.nsteps) {
            long long prev = __double_as_longlong(slowness_of(S.vel[(size_t)kr * S.nx + xc]));
            if (bits != prev) bits |= (long long)kSignBit;
        }
        slow[e] = __longlong_as_double(bits);
    }
}

// Refills.  Where some output of a wave changes, taps are loaded for all its outputs,
// between the stages of the FIR: a load of 16 bytes per lane keeps the data path of the L1
// busy for 16 clocks however many lanes ask and wherever the rows are cached, and a wave
// waits until its loads are accepted.  As one masked block before the FIR they took 155 of
// 575 us at 1024 points, 512 depths, 200 frequencies, layered, and 165 of 420 us at 601
// points, 301 depths, 97 frequencies where every point changes at every step (now 487 and
// 335 in all).
template <int Q>
struct Refill {
    bool any;  // some output of the wave changes
    int j[Q];  // its outputs' entries, where any
    __device__ __forceinline__ void look_up(const BatchArgs& a, double ar, const double (&v)[Q])
    {
        bool chg = false;
#pragma unroll
        for (int q = 0; q < Q; ++q) chg = chg || slowness_changed(v[q]);
        any = __builtin_amdgcn_ballot_w64(chg) != 0;
#pragma unroll
        for (int q = 0; q < Q; ++q) j[q] = 0;
        if (any)
#pragma unroll
            for (int q = 0; q < Q; ++q) j[q] = index_of_slowness(ar, a.b, a.nk, slowness_value(v[q]));
    }
};

// Slowness of Q outputs.
template <int Q>
__device__ __forceinline__ void load_slowness(const double* p, double (&v)[Q])
{
    if constexpr (Q % 2 == 0) {
#pragma unroll
        for (int q = 0; q < Q; q += 2) {
            const double2 d = load_global(reinterpret_cast<const double2*>(p + q));
            v[q] = d.x;
            v[q + 1] = d.y;
        }
    } else {
#pragma unroll
        for (int q = 0; q < Q; ++q) v[q] = *as_global(p + q);
    }
}

// Write-through store of one partial-row value (see store_partial2).
__device__ __forceinline__ void store_partial1(float* p, float a)
{
    __hip_atomic_store(as_global(p), a, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

template <int M, int Q>
struct FastLane {
    int win;        // its window in the first plane
    int plane;      // points of a plane
    int out[2][Q];  // its outputs in either plane; past the section: a point that no one reads
    int x0;
    double ar;
    size_t row;     // floats between partial rows (none where the frequency is not the section's)
};

// One depth step k with the current tap set: from plane PL to the other.  sp: the
// slowness of step k+2, pr: the partial row of step k.
template <int M, int Q, bool ROWS, int PL>
__device__ __forceinline__ void step_fast(const BatchArgs& a, float2* sm, const FastLane<M, Q>& L,
                                          const double* sp, float*& pr, bool publishes,
                                          float2 (&hc)[Q][M + 1], float2 (&ho)[Q][M + 1],
                                          double (&sn)[Q], float2 (&o)[Q])
{
    Refill<Q> next;
    next.look_up(a, L.ar, sn);
    load_slowness<Q>(sp + L.x0, sn);
    const float2* row[Q];
#pragma unroll
    for (int q = 0; q < Q; ++q) row[q] = a.tab + (size_t)next.j[q] * (M + 1);
    const auto refill = [&](int s) {
        if (s % kRefillStages != 0 || !next.any) return;
#pragma unroll
        for (int i = s; i < s + kRefillStages && 2 * i <= M; ++i)
#pragma unroll
            for (int q = 0; q < Q; ++q) load_pair<M>(ho[q], row[q], i);
    };
    firq<M, Q>(sm + L.win + PL * L.plane, hc, o, refill);
    refill(kStages<M, Q>);
#pragma unroll
    for (int q = 0; q < Q; ++q) sm[L.out[1 - PL][q]] = o[q];
    if (ROWS) {
        if (publishes) wait_vmem_all();
        if constexpr (Q == 2) store_partial2(pr, o[0].x, o[1].x);
        else store_partial1(pr, o[0].x);
        pr += L.row;
    }
    __syncthreads();
}

// Register-tap kernel, one or two outputs per thread.  Sub-group of tsub threads per
// frequency; LDS per sub-group = two planes of Q*tsub + 2M + 2 points, P[x] at
// offset M + x, zero elsewhere (the zero boundary of Eq. 1).  A step has no branch but
// those of the refills and of publishing: with fewer than two waves per SIMD every
// instruction costs 5 clocks.
template <int M, int Q, bool ROWS>
__global__ void __launch_bounds__(512) k_extrap_fast(BatchArgs a)
{
    extern __shared__ float4 smem4[];
    if (ROWS && (int)blockIdx.x < a.nred) {
        reduce_role(a, blockIdx.x, reinterpret_cast<int*>(smem4));
        return;
    }
    const ItemDev it = item_of(a, blockIdx.x - (ROWS ? a.nred : 0));
    const SecDev S = sec_of(a, it.sec);
    const int tsub = ((S.nx + Q - 1) / Q + 63) / 64 * 64, G = S.G;
    const int g = threadIdx.x / tsub;
    const int LB = Q * tsub + 2 * M + 2;
    if (g >= G) {
        idle_barriers(2 + S.nsteps + (ROWS ? 1 : 0));
        return;
    }
    float2* const sm = reinterpret_cast<float2*>(smem4);
    const int t = threadIdx.x - g * tsub;
    const bool live = it.r0 + g < S.nw;
    const int r = live ? it.r0 + g : S.nw - 1;
    const int base = g * 2 * LB;
    FastLane<M, Q> L;
    L.x0 = Q * t;
    L.win = base + Q * t;
    L.plane = LB;
    bool ok[Q];
#pragma unroll
    for (int q = 0; q < Q; ++q) {
        ok[q] = live && L.x0 + q < S.nx;
        for (int pl = 0; pl < 2; ++pl)
            L.out[pl][q] = ok[q] ? base + pl * LB + M + L.x0 + q : G * 2 * LB;
    }
    L.ar = S.omega[r] / a.dk;
    L.row = live ? (size_t)S.nw * S.ldp : 0;

    for (int i = t; i < 2 * LB; i += tsub) sm[base + i] = make_float2(0.0f, 0.0f);
    __syncthreads();
#pragma unroll
    for (int q = 0; q < Q; ++q)
        if (ok[q]) sm[base + M + L.x0 + q] = S.win[(size_t)(L.x0 + q) * S.nw + r];

    float2 hA[Q][M + 1], hB[Q][M + 1];
    {
        double v[Q];
        load_slowness<Q>(S.slow + L.x0, v);
#pragma unroll
        for (int q = 0; q < Q; ++q)
            load_taps<M>(hA[q], a.tab + (size_t)index_of_slowness(L.ar, a.b, a.nk, slowness_value(v[q])) * (M + 1));
        load_slowness<Q>(S.slow + (size_t)(S.nsteps > 1 ? 1 : 0) * S.ldp + L.x0, v);
#pragma unroll
        for (int q = 0; q < Q; ++q)
            load_taps<M>(hB[q], a.tab + (size_t)index_of_slowness(L.ar, a.b, a.nk, slowness_value(v[q])) * (M + 1));
    }
    double sn[Q] = {};  // slowness of the step after, flagged where the other set is to be refilled
    const double* sp = S.slow + (size_t)(S.nsteps > 2 ? 2 : S.nsteps - 1) * S.ldp;
    float* pr = live ? S.part + (size_t)r * S.ldp + L.x0 : a.trash + L.x0;
    __syncthreads();

    float2 o[Q] = {};
    for (int k = 0; k < S.nsteps; k += 2) {
        step_fast<M, Q, ROWS, 0>(a, sm, L, sp, pr, false, hA, hB, sn, o);
        if (k + 1 >= S.nsteps) break;
        sp += k + 3 < S.nsteps ? S.ldp : 0;
        const bool publishes = ROWS && publishes_at(k + 1);
        step_fast<M, Q, ROWS, 1>(a, sm, L, sp, pr, publishes, hB, hA, sn, o);
        sp += k + 4 < S.nsteps ? S.ldp : 0;
        if (publishes) publish_block(a, S, (k + 1) / kPublish - 1);
    }
    if (ROWS) {
        wait_vmem_all();
        __syncthreads();
        for (int b = published_in_loop(S.nsteps); b * kPublish < S.nsteps; ++b) publish_block(a, S, b);
    }
    if (S.wout) {
#pragma unroll
        for (int q = 0; q < Q; ++q)
            if (ok[q]) S.wout[(size_t)(L.x0 + q) * S.nw + r] = o[q];
    }
}

// Partial row of Q outputs.  Q = 4: x0 is a multiple of 4 and 4 * tsub is
// the row stride, so every lane stores (lanes past nx into the padding).
// Q = 3: 3 * tsub can pass the row stride, so only outputs inside the section
// are stored.
template <int Q>
__device__ __forceinline__ void store_partial_q(float* pr, const float2 (&o)[Q], const bool (&ok)[Q])
{
    if constexpr (Q == 4) {
        store_partial2(pr, o[0].x, o[1].x);
        store_partial2(pr + 2, o[2].x, o[3].x);
    } else {
#pragma unroll
        for (int q = 0; q < Q; ++q)
            if (ok[q]) store_partial1(pr + q, o[q].x);
    }
}

// Register-tap kernel for wider sections (nx <= Q * 512): Q = 3 or 4 outputs
// per thread and one tap set (two do not fit in 256 VGPRs), whose taps are
// replaced as the FIR has used them for the last time, where the slowness of some
// output of the wave changes at the next step.  One frequency per workgroup.  Q = 3
// serves 1024 < nx <= 1536: there Q = 4 would leave 5 or 6 waves for 4 SIMDs (the
// SIMD with two waves sets the pace), while Q = 3 gives 6 to 8 waves and three
// quarters of the work per wave.  Bound by the FP32 instruction rate and, where
// waves refill, by the L1's data path.  1501 points, 300 depths, 101 frequencies:
// layered 587 -> 493 us, a velocity that varies from point to point 782 -> 675 us.
template <int M, int Q, bool ROWS>
__global__ void __launch_bounds__(512) k_extrap_wide(BatchArgs a)
{
    extern __shared__ float4 smem4[];
    if (ROWS && (int)blockIdx.x < a.nred) {
        reduce_role(a, blockIdx.x, reinterpret_cast<int*>(smem4));
        return;
    }
    const ItemDev it = item_of(a, blockIdx.x - (ROWS ? a.nred : 0));
    const SecDev S = sec_of(a, it.sec);
    const int tsub = ((S.nx + Q - 1) / Q + 63) / 64 * 64;
    if ((int)threadIdx.x >= tsub) {
        idle_barriers(2 + S.nsteps + (ROWS ? 1 : 0));
        return;
    }
    float2* sm = reinterpret_cast<float2*>(smem4);
    const int t = threadIdx.x;
    const int LB = Q * tsub + 2 * M + 4;
    const int x0 = Q * t;
    const bool live = it.r0 < S.nw;
    const int r = live ? it.r0 : S.nw - 1;
    bool ok[Q];
    int xs[Q];  // slowness columns, clamped into the section
#pragma unroll
    for (int q = 0; q < Q; ++q) {
        ok[q] = live && x0 + q < S.nx;
        xs[q] = x0 + q < S.nx ? x0 + q : S.nx - 1;
    }
    const double ar = S.omega[r] / a.dk;

    for (int i = t; i < 2 * LB; i += tsub) sm[i] = make_float2(0.0f, 0.0f);
    __syncthreads();
#pragma unroll
    for (int q = 0; q < Q; ++q)
        if (ok[q]) sm[M + x0 + q] = S.win[(size_t)(x0 + q) * S.nw + r];

    float2 h[Q][M + 1];
#pragma unroll
    for (int q = 0; q < Q; ++q)
        load_taps<M>(h[q], a.tab + (size_t)index_of_slowness(ar, a.b, a.nk, slowness_value(S.slow[xs[q]])) * (M + 1));
    __syncthreads();

    const auto slowness = [&](int k, double (&v)[Q]) {  // flagged where it differs from row k-1
        const double* sp = S.slow + (size_t)(k < S.nsteps ? k : S.nsteps - 1) * S.ldp;
        if constexpr (Q == 4) load_slowness<Q>(sp + x0, v);
        else
#pragma unroll
            for (int q = 0; q < Q; ++q) v[q] = *as_global(sp + xs[q]);
    };
    double sn[Q];
    slowness(1, sn);
    // Waited for here: left in flight, the one wait at the start of a step, for the first as
    // for the others, would be for everything in flight, the row of the step before included
    // (2000 points, 300 depths, 150 frequencies, constant velocity, rows stored at the end
    // of a step: 579 -> 483 us).  Q = 3, whose stores the compiler cannot count, keeps the
    // wait for all (1300 points: 431 us, waited for here 511).
    if constexpr (Q == 4)
#pragma unroll
        for (int q = 0; q < Q; ++q) asm volatile("" : "+v"(sn[q]));
    float* pr = live ? S.part + (size_t)r * S.ldp + x0 : a.trash + x0;
    const size_t row = live ? (size_t)S.nw * S.ldp : 0;

    float2 o[Q];
    for (int k = 0; k < S.nsteps; ++k) {
        Refill<Q> next;
        next.look_up(a, ar, sn);
        slowness(k + 2, sn);
        // A row is stored at the start of the step after, whose FIR it then runs beside:
        // at the end of its step every wave stores just before the barrier that all wait
        // at, behind the taps loaded last (2000 points, 300 depths, 150 frequencies,
        // layered 672 -> 654 us, 1907 points, 200 depths, 100 frequencies, 19 taps 305 ->
        // 286 us, batches of 1537 to 2048 points 6.44 -> 6.03 ms; three outputs, 1100 to
        // 1500 points, 10.2 -> 9.5 ms)
        if (ROWS && k >= 1) {
            store_partial_q<Q>(pr, o, ok);
            pr += row;
        }
        // after stage s: the pairs of taps that it and the stages before were the last to use
        constexpr int NS = kStages<M, Q>;
        const auto refill = [&](int s) {
            if ((s % kRefillStagesWide != kRefillStagesWide - 1 && s != NS) || !next.any) return;
#pragma unroll
            for (int q = 0; q < Q; ++q) {
                const float2* row = a.tab + (size_t)next.j[q] * (M + 1);
#pragma unroll
                for (int i = 0; 2 * i <= M; ++i)
                    if (refill_stage<M, Q, kRefillStagesWide>(i) == s) load_pair<M>(h[q], row, i);
            }
        };
        firq<M, Q>(sm + (k & 1) * LB + x0, h, o, refill);
        float2* dst = sm + ((k + 1) & 1) * LB + M + x0;
#pragma unroll
        for (int q = 0; q < Q; ++q)
            if (ok[q]) dst[q] = o[q];
        refill(NS);
        if (ROWS) {
            if (publishes_at(k)) wait_vmem_all();
        }
        __syncthreads();
        if (ROWS && publishes_at(k)) publish_block(a, S, k / kPublish - 1);
    }
    if (ROWS) {
        store_partial_q<Q>(pr, o, ok);
        wait_vmem_all();
        __syncthreads();
        for (int b = published_in_loop(S.nsteps); b * kPublish < S.nsteps; ++b) publish_block(a, S, b);
    }
    if (S.wout) {
#pragma unroll
        for (int q = 0; q < Q; ++q)
            if (ok[q]) S.wout[(size_t)(x0 + q) * S.nw + r] = o[q];
    }
}

// row[x] = sum_r Re wf[x][r]: one wavefront per x, lane-strided FP64 partial
// sums, then a xor-butterfly of cross-lane shuffles (fixed order).
__global__ void __launch_bounds__(256) k_image(const float2* __restrict__ wf,
                                               double* __restrict__ row, int nx, int nw)
{
    const int lane = threadIdx.x & 63;
    const int x = blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6);
    if (x >= nx) return;
    const float2* p = wf + (size_t)x * nw;
    double acc = 0.0;
    for (int r = lane; r < nw; r += 64) acc += (double)p[r].x;
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) acc += __shfl_xor(acc, off, 64);
    if (lane == 0) row[x] = acc;
}

__global__ void k_index(const float* __restrict__ vel, const double* __restrict__ omega,
                        int nx, int nw, int nrows, int nk, double dk, double b,
                        int32_t* __restrict__ idx)
{
#pragma clang fp contract(off)
    const size_t total = (size_t)nrows * nx * nw;
    for (size_t e = (size_t)blockIdx.x * blockDim.x + threadIdx.x; e < total;
         e += (size_t)gridDim.x * blockDim.x) {
        int r = (int)(e % nw);
        size_t kx = e / nw;
        double a = omega[r] / dk;
        idx[e] = table_index(a, b, nk, vel[kx]);
    }
}


// Image rows of depth steps [s0, s1) from their partial rows, once the
// depth-stepping launch is over: four points per thread, the frequencies added in
// increasing order in FP64, the order of the reducer workgroups, so a row is the
// same whichever of the two forms it.  Small workgroups spread the rows over
// every CU; 16 loads of 16 bytes in flight per thread (row strides are multiples of 256
// points; the last thread of a row reads its padding, which frequency workgroups of
// odd widths leave unwritten, and does not store those sums).
__device__ __forceinline__ void sum_rows(const float* __restrict__ part, double* __restrict__ rows,
                                         int st, int x, int nx, int nw, int ldp)
{
    const float* p = part + (size_t)st * nw * ldp + x;
    double acc[4] = {0.0, 0.0, 0.0, 0.0};
    const auto add = [&](const v4f& v) {
        acc[0] += (double)v.x;
        acc[1] += (double)v.y;
        acc[2] += (double)v.z;
        acc[3] += (double)v.w;
    };
    int r = 0;
    for (; r + 16 <= nw; r += 16) {
        v4f v[16];
#pragma unroll
        for (int j = 0; j < 16; ++j) v[j] = *reinterpret_cast<const v4f*>(p + (size_t)(r + j) * ldp);
#pragma unroll
        for (int j = 0; j < 16; ++j) add(v[j]);
    }
    for (; r < nw; ++r) add(*reinterpret_cast<const v4f*>(p + (size_t)r * ldp));
    double* row = rows + (size_t)st * nx + x;
#pragma unroll
    for (int q = 0; q < 4; ++q)
        if (x + q < nx) row[q] = acc[q];
}

// Steps s0 .. of one section: nbx workgroups per row.
__global__ void __launch_bounds__(64) k_rows(const float* __restrict__ part,
                                             double* __restrict__ rows, int s0, int nx, int nw,
                                             int ldp, int nbx)
{
    const int x = 4 * (blockIdx.x % nbx * 64 + threadIdx.x);
    if (x < nx) sum_rows(part, rows, s0 + blockIdx.x / nbx, x, nx, nw, ldp);
}

// Every step of every section of a batch: each section's workgroups walk its rows, so
// that sections of any sizes share a launch (one workgroup per row of the longest section
// and part of the widest, for every section, overran the grid's 2^32 threads at 8192
// points beside 2^21 depths: rows were left out; and 40 sections of 100 to 2048 points, 10
// to 400 depths took 7.31 instead of 7.25 ms).
__global__ void __launch_bounds__(64) k_rows_batch(BatchArgs a)
{
    const SecDev S = sec_of(a, blockIdx.y);
    const int nbx = (S.nx + 255) / 256;
    const size_t total = (size_t)S.nsteps * nbx;
    for (size_t i = blockIdx.x; i < total; i += gridDim.x) {
        const int st = (int)(i / nbx), x = 4 * ((int)(i % nbx) * 64 + threadIdx.x);
        if (x < S.nx) sum_rows(S.part, S.rows, st, x, S.nx, S.nw, S.ldp);
    }
}

template <int M, int Q>
int launch_fast_as(const BatchArgs& a, int threads, size_t lds, hipStream_t s)
{
    if (a.rows)
        hipLaunchKernelGGL((k_extrap_fast<M, Q, true>), dim3(a.nitems + a.nred), dim3(threads), lds,
                           s, a);
    else
        hipLaunchKernelGGL((k_extrap_fast<M, Q, false>), dim3(a.nitems), dim3(threads), lds, s, a);
    return hipGetLastError() == hipSuccess ? MIG_OK : MIG_E_DEVICE;
}

template <int M>
int launch_fast(const BatchArgs& a, int threads, size_t lds, hipStream_t s)
{
    return launch_fast_as<M, 2>(a, threads, lds, s);
}

template <int M>
int launch_narrow(const BatchArgs& a, int threads, size_t lds, hipStream_t s)
{
    return launch_fast_as<M, 1>(a, threads, lds, s);
}

template <int M, int Q>
int launch_wide(const BatchArgs& a, int threads, size_t lds, hipStream_t s)
{
    if (a.rows)
        hipLaunchKernelGGL((k_extrap_wide<M, Q, true>), dim3(a.nitems + a.nred), dim3(threads),
                           lds, s, a);
    else
        hipLaunchKernelGGL((k_extrap_wide<M, Q, false>), dim3(a.nitems), dim3(threads), lds, s, a);
    return hipGetLastError() == hipSuccess ? MIG_OK : MIG_E_DEVICE;
}

template <int M>
int launch_wide4(const BatchArgs& a, int threads, size_t lds, hipStream_t s)
{
    return launch_wide<M, 4>(a, threads, lds, s);
}

template <int M>
int launch_wide3(const BatchArgs& a, int threads, size_t lds, hipStream_t s)
{
    return launch_wide<M, 3>(a, threads, lds, s);
}

typedef int (*launch_fn)(const BatchArgs&, int, size_t, hipStream_t);

// Register-tap kernels are instantiated for N = 1..35 (M = 0..17); beyond
// that two tap sets no longer fit in 256 VGPRs without spilling.
#define MIG_INST(f)                                                                   \
    {&f<0>, &f<1>, &f<2>, &f<3>, &f<4>, &f<5>, &f<6>, &f<7>, &f<8>, &f<9>, &f<10>,     \
     &f<11>, &f<12>, &f<13>, &f<14>, &f<15>, &f<16>, &f<17>}
const launch_fn kFast[] = MIG_INST(launch_fast);
const launch_fn kNarrow[] = MIG_INST(launch_narrow);
const launch_fn kWide[] = MIG_INST(launch_wide4);
const launch_fn kMid[] = MIG_INST(launch_wide3);
constexpr int kRegMaxM = 17;
constexpr int kFastMaxNx = 2 * 512;
constexpr int kMidMaxNx = 3 * 512;
constexpr int kWideMaxNx = 4 * 512;

}  // namespace

int extrap_kernel_kind(int nx, int M)
{
    if (M > kRegMaxM) return 0;
    if (nx <= kFastMaxNx) return 1;
    if (nx <= kMidMaxNx) return 3;
    if (nx <= kWideMaxNx) return 2;
    return 0;
}

// One output per thread instead of two: twice the waves, half the chain of each, but
// windows of 8-byte LDS reads (twice the LDS clocks per output).  Up to 256 points (four
// waves, one per SIMD) always: 300 depths, 150 frequencies, 35 taps, layered, 200 points:
// 257 -> 182 us, 290 frequencies: 270 -> 216 us.  Up to 512 points (eight waves) where
// every workgroup has a CU to itself: 150 frequencies, 400 points: 261 -> 235 us, 512
// points: 264 -> 242 us, but 290 frequencies of 450 points: 329 -> 374 us.
// (A batch's launch holds sections of any of these widths and keeps to two.)
bool extrap_narrow(int kind, int nx, int nitems, int cus)
{
    return kind == 1 && nx <= 512 && (nx <= 256 || nitems <= cus);
}

int threads_narrow(int nx) { return (nx + 63) / 64 * 64; }

int threads_per_omega(int kind, int nx)
{
    if (kind == 1) return ((nx + 1) / 2 + 63) / 64 * 64;
    if (kind == 2) return ((nx + 3) / 4 + 63) / 64 * 64;
    return ((nx + 2) / 3 + 63) / 64 * 64;
}

int launch_slowness(const BatchArgs& a, int max_rows, int max_ldp, int dist, hipStream_t s)
{
    size_t per = (size_t)max_rows * max_ldp;
    size_t blocks = (per + 255) / 256;
    if (blocks > 4096) blocks = 4096;
    hipLaunchKernelGGL(k_slowness, dim3((unsigned)blocks, a.nsec), dim3(256), 0, s, a, dist);
    return hipGetLastError() == hipSuccess ? MIG_OK : MIG_E_DEVICE;
}

int launch_extrap(const BatchArgs& a, int kind, int threads, bool narrow, hipStream_t s)
{
    // LDS: G sub-groups x two planes; the host picks threads = G * tsub.
    if (kind == 1) {
        const int Q = narrow ? 1 : 2;
        const size_t lds = (size_t)2 * (Q * threads + threads / 64 * (2 * a.M + 2) + 1) * sizeof(float2);
        if (Q == 1) return kNarrow[a.M](a, threads, lds, s);
        return kFast[a.M](a, threads, lds, s);
    }
    if (kind == 2 || kind == 3) {
        const int Q = kind == 2 ? 4 : 3;
        size_t lds = (size_t)2 * (Q * threads + 2 * a.M + 4) * sizeof(float2);
        return (kind == 2 ? kWide : kMid)[a.M](a, threads, lds, s);
    }
    return MIG_E_ARG;
}

int launch_rows(const float* part, double* rows, int s0, int s1, int nx, int nw, int ldp,
                hipStream_t s)
{
    if (s1 <= s0) return MIG_OK;
    const int nbx = (nx + 255) / 256;
    const dim3 grid((unsigned)nbx * (unsigned)(s1 - s0));
    hipLaunchKernelGGL(k_rows, grid, dim3(64), 0, s, part, rows, s0, nx, nw, ldp, nbx);
    return hipGetLastError() == hipSuccess ? MIG_OK : MIG_E_DEVICE;
}

int launch_rows_batch(const BatchArgs& a, int max_nx, int max_rows, hipStream_t s)
{
    // eight waves per CU and section: 2 MB of loads in flight per CU
    const size_t most = (size_t)((max_nx + 255) / 256) * max_rows;
    const dim3 grid((unsigned)(most < 2048 ? most : 2048), a.nsec);
    hipLaunchKernelGGL(k_rows_batch, grid, dim3(64), 0, s, a);
    return hipGetLastError() == hipSuccess ? MIG_OK : MIG_E_DEVICE;
}

namespace {
__global__ void k_clear_status(int* status) { *status = 0; }
}  // namespace

int launch_clear_status(int* status, hipStream_t s)
{
    hipLaunchKernelGGL(k_clear_status, dim3(1), dim3(1), 0, s, status);
    return hipGetLastError() == hipSuccess ? MIG_OK : MIG_E_DEVICE;
}

int launch_image(const float2* wf, double* row, int nx, int nw, hipStream_t s)
{
    dim3 grid((nx + 3) / 4);
    hipLaunchKernelGGL(k_image, grid, dim3(256), 0, s, wf, row, nx, nw);
    return hipGetLastError() == hipSuccess ? MIG_OK : MIG_E_DEVICE;
}

int launch_index(const float* vel, const double* omega, int nx, int nw, int nrows,
                 int nk, double dk, double b, int32_t* idx, hipStream_t s)
{
    size_t total = (size_t)nrows * nx * nw;
    size_t blocks = (total + 255) / 256;
    if (blocks > 65536) blocks = 65536;
    hipLaunchKernelGGL(k_index, dim3((unsigned)blocks), dim3(256), 0, s, vel, omega, nx, nw,
                       nrows, nk, dk, b, idx);
    return hipGetLastError() == hipSuccess ? MIG_OK : MIG_E_DEVICE;
}

}  // namespace mig
