// Device code shared by the depth-stepping kernels: complex arithmetic of the FIR,
// partial rows and their publication, the reducer role.
#pragma once

#include "common.hpp"

namespace mig {
namespace {

// s_waitcnt vmcnt(0), other counters left alone (GFX9 encoding:
// vmcnt[3:0] | expcnt[6:4] | lgkmcnt[11:8] | vmcnt[5:4] in bits 15:14).
__device__ __forceinline__ void wait_vmem_all()
{
    __builtin_amdgcn_s_waitcnt((7 << 4) | (15 << 8));
}

__device__ __forceinline__ float2 cmulf(float2 h, float2 u)
{
    return make_float2(fmaf(-h.y, u.y, h.x * u.x), fmaf(h.y, u.x, h.x * u.y));
}

__device__ __forceinline__ float2 cfmaf(float2 h, float2 s, float2 acc)
{
    acc.x = fmaf(h.x, s.x, acc.x);
    acc.x = fmaf(-h.y, s.y, acc.x);
    acc.y = fmaf(h.x, s.y, acc.y);
    acc.y = fmaf(h.y, s.x, acc.y);
    return acc;
}

// the same with conj(h)
__device__ __forceinline__ float2 cmulf_conj(float2 h, float2 u)
{
    return make_float2(fmaf(h.y, u.y, h.x * u.x), fmaf(-h.y, u.x, h.x * u.y));
}

__device__ __forceinline__ float2 cfmaf_conj(float2 h, float2 s, float2 acc)
{
    acc.x = fmaf(h.x, s.x, acc.x);
    acc.x = fmaf(h.y, s.y, acc.x);
    acc.y = fmaf(h.x, s.y, acc.y);
    acc.y = fmaf(-h.y, s.x, acc.y);
    return acc;
}

__device__ __forceinline__ float2 cadd(float2 a, float2 b)
{
    return make_float2(a.x + b.x, a.y + b.y);
}

// Partial image rows are stored write-through (agent-scope relaxed atomic
// stores): reducers on other XCDs read them once their block is counted, and
// nothing of them is left in this XCD's L2 to write back first.
__device__ __forceinline__ void store_partial2(float* p, float a, float b)
{
    const unsigned long long u =
        (unsigned long long)__float_as_uint(a) | ((unsigned long long)__float_as_uint(b) << 32);
    __hip_atomic_store(as_global(reinterpret_cast<unsigned long long*>(p)), u, __ATOMIC_RELAXED,
                       __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ SecDev sec_of(const BatchArgs& a, int i)
{
    return a.nsec == 1 ? a.one : a.secs[i];
}

__device__ __forceinline__ ItemDev item_of(const BatchArgs& a, int i)
{
    return a.nsec == 1 ? ItemDev{0, i * a.one.G} : a.items[i];
}

__device__ __forceinline__ TaskDev task_of(const BatchArgs& a, int i)
{
    if (a.nsec != 1) return a.tasks[i];
    const int p = i % a.parts;
    const int span = ((a.one.nx + a.parts - 1) / a.parts + 1) & ~1;  // even part width
    const int x0 = p * span;
    return TaskDev{0, i / a.parts, x0, x0 + span < a.one.nx ? x0 + span : a.one.nx};
}

// Thread 0 of a frequency workgroup, after a barrier that follows the stores of
// the partial rows of block c: count the block (and the launch's publishes).  The partial rows are stored
// write-through (agent-scope atomic stores) and every wave waits for its own
// stores to complete before that barrier (wait_vmem_all), so when the counter
// moves the rows are already where other XCDs read them.  No release fence:
// at agent scope it would write back the whole L2 of the XCD, which the
// barrier after the next step would make every wave of the workgroup wait for.
__device__ __forceinline__ void publish_block(const BatchArgs& a, const SecDev& S, int c)
{
    if (threadIdx.x == 0) {
        __hip_atomic_fetch_add(as_global(S.cnt + c), 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __hip_atomic_fetch_add(as_global(a.progress), 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
}

// Block b (steps 32b .. 32b+31) is published at the end of step 32b+33.  Its last partial
// row is stored at the latest at the start of step 32b+32; in step 32b+33 every wave
// waits for its memory operations before it stores that step's row, and the barrier that
// ends the step means every wave of the workgroup has passed that wait, which by then
// finds the stores complete.  Blocks whose publishing step lies past the last step are
// published after the loop.
__device__ __forceinline__ bool publishes_at(int k) { return k >= kPublish + 1 && k % kPublish == 1; }
__device__ __forceinline__ int published_in_loop(int nsteps)
{
    return nsteps - 1 >= kPublish + 1 ? (nsteps - 1 - (kPublish + 1)) / kPublish + 1 : 0;
}

__device__ __forceinline__ int load_relaxed(int* p)
{
    return __hip_atomic_load(as_global(p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Thread 0 of a reducer: wait until block T.block of section S is published
// by all its frequency workgroups.  Returns false when the launch has been
// abandoned: by this reducer, after kStallTicks (or the caller's limit)
// without any publish in the launch, or by another reducer before.  The
// first reducer to give up sets the launch's abandon word and the call's
// status word; every later wait of the launch returns at once.
__device__ bool wait_block(const BatchArgs& a, const SecDev& S, int block)
{
    int* const abandon = a.progress + 1;
    const int need = S.nprod + a.extra_wait;
    int v, last = -1, seen = -1;
    unsigned long long t0 = wall_clock64();
    while ((v = load_relaxed(S.cnt + block)) < need) {
        if (load_relaxed(abandon) != 0) return false;
        // the stall clock restarts whenever the block's counter or the
        // launch's publish count moves: a section whose items start late in
        // a long batch is waited for, a launch that stops is not
        const int g = load_relaxed(a.progress);
        const unsigned long long now = wall_clock64();
        if (v != last || g != seen) {
            last = v;
            seen = g;
            t0 = now;
        } else if (now - t0 > a.stall_ticks) {
            __hip_atomic_store(as_global(abandon), 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if (a.status)
                __hip_atomic_store(as_global(a.status), kStatusAbandoned, __ATOMIC_RELAXED,
                                   __HIP_MEMORY_SCOPE_AGENT);
            return false;
        }
        __builtin_amdgcn_s_sleep(kPollSleep);
    }
    return true;
}

// Reducer workgroup q of a.nred: tasks q, q + nred, ... (ordered block-major
// across sections, i.e. in production order).  One wait and one acquire per
// task: an acquire invalidates the L2 of the reducer's XCD, which the
// frequency workgroups there pay for in table refills, so tasks are whole
// published blocks (split along x only when there are few blocks).
constexpr int kRedDepth = 32;

__device__ void reduce_role(const BatchArgs& a, int q, int* flag)
{
    for (int i = q; i < a.ntasks; i += a.nred) {
        const TaskDev T = task_of(a, i);
        const SecDev S = sec_of(a, T.sec);
        if (T.block * kPublish >= S.nsteps) continue;  // no such block (uniform)
        if (threadIdx.x == 0) {
            const bool ok = wait_block(a, S, T.block);
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
            *flag = ok ? 1 : 0;
        }
        __syncthreads();
        const bool ok = *flag != 0;
        __syncthreads();
        const int s0 = T.block * kPublish;
        const int s1 = s0 + kPublish < S.nsteps ? s0 + kPublish : S.nsteps;
        const int npair = (T.x1 - T.x0 + 1) / 2;
        const int items = (s1 - s0) * npair;
        for (int it = threadIdx.x; it < items; it += blockDim.x) {
            const int st = s0 + it / npair;
            const int x0 = T.x0 + 2 * (it % npair);
            const float* p = S.part + (size_t)st * S.nw * S.ldp;
            __attribute__((address_space(1))) double* row = as_global(S.rows + (size_t)st * S.nx);
            // kRedDepth loads in flight per thread (the reads are latency-bound);
            // rows past nw are clamped loads that are not added, so the sum
            // runs over r in increasing order like k_rows
            double a0 = 0.0, a1 = 0.0;
            for (int r = 0; r < S.nw; r += kRedDepth) {
                float2 v[kRedDepth];
#pragma unroll
                for (int j = 0; j < kRedDepth; ++j) {
                    const int rr = r + j < S.nw ? r + j : S.nw - 1;
                    v[j] = load_global(reinterpret_cast<const float2*>(p + (size_t)rr * S.ldp + x0));
                }
                __builtin_amdgcn_sched_barrier(0);  // every load issued before the first add
#pragma unroll
                for (int j = 0; j < kRedDepth; ++j)
                    if (r + j < S.nw) {
                        a0 += (double)v[j].x;
                        a1 += (double)v[j].y;
                    }
            }
            const double nan = __builtin_nan("");
            row[x0] = ok ? a0 : nan;
            if (x0 + 1 < T.x1) row[x0 + 1] = ok ? a1 : nan;
        }
        __syncthreads();  // *flag is reused by the next task
    }
}

// Threads of a workgroup beyond its G sub-groups take no part in the work but
// must meet every barrier of the active threads.
__device__ __forceinline__ void idle_barriers(int n)
{
    for (int i = 0; i < n; ++i) __syncthreads();
}

typedef float v4f __attribute__((ext_vector_type(4)));
typedef float v4f_a8 __attribute__((ext_vector_type(4), aligned(8)));

// Halo of the planes on each side: M rounded up to whole 16-byte reads.
__host__ __device__ constexpr int long_halo(int M) { return (M + 1) & ~1; }
// Points of one plane with its halos; lanes read whole runs of Q <= 4 outputs.
__host__ __device__ constexpr int long_plane(int nx, int M) { return (nx + 3) / 4 * 4 + 2 * long_halo(M); }

// The window around outputs P[0 .. Q-1]: w[PM + i] = P[i].
template <int M, int Q>
struct Window {
    static constexpr int PM = long_halo(M);
    // pairs of taps whose points are read ahead of their use (three: 3 % slower)
    static constexpr int kAhead = 1;
    static constexpr int NP = (M + 1) / 2;
    float2 w[2 * PM + Q];
    const float2* P;
    __device__ __forceinline__ void load(int i)  // points i, i + 1 (i even)
    {
        const v4f q = *reinterpret_cast<const v4f*>(P + i);
        w[PM + i] = make_float2(q.x, q.y);
        w[PM + i + 1] = make_float2(q.z, q.w);
    }
    // the points that taps 2 i + 1 and 2 i + 2 reach beyond those of smaller taps
    __device__ __forceinline__ void load_pair(int i)
    {
        if (i < NP) {
            load(-(2 * i + 2));
            load(2 * i + Q);
        }
    }
    // the outputs' own points and the first pairs
    __device__ __forceinline__ void begin()
    {
#pragma unroll
        for (int i = 0; i < Q; i += 2) load(i);
#pragma unroll
        for (int i = 0; i < kAhead; ++i) load_pair(i);
    }
    __device__ __forceinline__ float2 pair_sum(int q, int n) const { return cadd(w[PM + q - n], w[PM + q + n]); }
};

// Two consecutive taps of a table row (the second may lie past its end where unused).
__device__ __forceinline__ v4f tap_pair(const float2* row, int n, bool two)
{
    typedef const __attribute__((address_space(1))) v4f_a8* global_v4f;
    if (two) return *(global_v4f)reinterpret_cast<const v4f_a8*>(row + n);
    const float2 a = load_global(row + n);
    return v4f{a.x, a.y, 0.0f, 0.0f};
}

// Stages of the FIR between two groups of tap refills (a branch each: one group per stage
// costs waves that refill nothing 3 %; a FIR of its own for waves that refill makes the
// compiler move whole tap sets where the two meet).
constexpr int kRefillStages = 3;
// The same in kernels of three and four outputs per thread, whose groups are larger (2000
// points, 300 depths, 150 frequencies: layered 721 -> 695 us, 974 -> 934 us where the
// velocity varies from point to point).
constexpr int kRefillStagesWide = 2;

// Q adjacent outputs x0..x0+Q-1 from the window w[i] = P[x0 - M + i], i = 0..2M+Q-1.
// Even Q: x0 is even, so the window is read with 16-byte LDS loads; odd Q (x0 of either
// parity): 8-byte loads.  Points are read from the centre outwards, as the taps use them
// (two taps per stage), kStagesAhead stages before their use: after a barrier every wave
// of the CU reads at once, and a wave that asked for its whole window first would leave
// the SIMDs idle until most of the CU's reads were done (1024 points, 300 depths, 150
// frequencies, constant velocity: 280 -> 261 us).
constexpr int kStagesAhead = 2;

template <int M, int Q>
constexpr int kCentre = Q % 2 == 0 && M % 2 ? 1 : 0;  // last tap of stage 0
template <int M, int Q>
constexpr int kStages = (M - kCentre<M, Q> + 1) / 2;  // stages after stage 0

// CONJ: conjugated taps, and a sum each for even and odd taps (the adjoint of wide sections;
// the forward planes keep one sum in increasing order of taps).
template <int M, int Q, bool CONJ = false, int AHEAD = kStagesAhead, class F>
__device__ __forceinline__ void firq(const float2* __restrict__ win, const float2 (&h)[Q][M + 1],
                                     float2 (&o)[Q], const F& beside)
{
    // Stage 0: points M - E .. M + Q - 1 + E, for taps 0 .. E.  Stage s: two points more on
    // each side, for two taps more (the outermost may be cut short by the window's ends).
    constexpr int E = kCentre<M, Q>, NS = kStages<M, Q>;
    float2 w[2 * M + Q];
    const auto load = [&](int i) {  // points i, i + 1 (i even where Q is)
        if constexpr (Q % 2 == 0) {
            const float4 q = *reinterpret_cast<const float4*>(win + i);
            w[i] = make_float2(q.x, q.y);
            w[i + 1] = make_float2(q.z, q.w);
        } else {
            if (i >= 0 && i < 2 * M + Q) w[i] = win[i];
            if (i + 1 >= 0 && i + 1 < 2 * M + Q) w[i + 1] = win[i + 1];
        }
    };
    const auto stage = [&](int s) {
        if (s > NS) return;
        load(M - E - 2 * s);
        load(M + Q - 2 + E + 2 * s);
    };
#pragma unroll
    for (int i = M - E; i < M + Q + E; i += 2) {
        if (Q % 2 == 0 || i + 1 < M + Q) load(i);
        else w[i] = win[i];
    }
#pragma unroll
    for (int s = 1; s <= AHEAD; ++s) stage(s);
#pragma unroll
    for (int q = 0; q < Q; ++q) o[q] = CONJ ? cmulf_conj(h[q][0], w[M + q]) : cmulf(h[q][0], w[M + q]);
    float2 odd[Q] = {};
    // (the outputs are pinned: left alone, the compiler sums one after the other and keeps
    // the whole window in registers for it)
    const auto tap = [&](int n) {
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            const float2 s = cadd(w[M + q - n], w[M + q + n]);
            float2& to = CONJ && n % 2 ? odd[q] : o[q];
            to = CONJ ? cfmaf_conj(h[q][n], s, to) : cfmaf(h[q][n], s, to);
            asm volatile("" : "+v"(to.x), "+v"(to.y));
        }
    };
    if constexpr (E == 1) tap(1);
    if (NS > 0) beside(0);
#pragma unroll
    for (int s = 1; s <= NS; ++s) {
        __builtin_amdgcn_sched_barrier(0);
        stage(s + AHEAD);
        const int n = E + 2 * s - 1;
        tap(n);
        if (n + 1 <= M) tap(n + 1);
        if (s < NS) beside(s);
    }
    if constexpr (CONJ)
#pragma unroll
        for (int q = 0; q < Q; ++q) o[q] = cadd(o[q], odd[q]);
}

// Stage after which taps 2 i and 2 i + 1 are loaded anew where one set is all there is:
// the end of the group of stages that uses them last.
template <int M, int Q, int GROUP>
constexpr int refill_stage(int i)
{
    const int last = 2 * i + 1 <= kCentre<M, Q> ? 0 : (2 * i + 2 - kCentre<M, Q>) / 2;
    const int g = last / GROUP * GROUP + GROUP - 1;
    return g < kStages<M, Q> ? g : kStages<M, Q>;
}

// Taps 2 i and 2 i + 1 of a table row.
template <int M>
__device__ __forceinline__ void load_pair(float2 (&h)[M + 1], const float2* row, int i)
{
    const v4f v = tap_pair(row, 2 * i, 2 * i + 1 <= M);
    h[2 * i] = make_float2(v.x, v.y);
    if (2 * i + 1 <= M) h[2 * i + 1] = make_float2(v.z, v.w);
}

}  // namespace
}  // namespace mig
