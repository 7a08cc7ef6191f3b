// Extrapolator-table design in FP64 on the GPU (table row A0).
//
// The paper designs the 1-D FIR extrapolators in advance, as an optimization
// between filter length and propagation angle, and stresses that accurate
// designs are needed for the recursion of Eq. (1) to stay stable (Sec. II,
// Sec. III).  It does not give the method.  This file implements, per table
// entry, a weighted least-squares fit of even taps to the one-way phase shift
// over dz, with multiplicative reweighting of points whose gain exceeds one,
// and a final scale that bounds |H| below one for every wavenumber (Bernstein's
// inequality for trigonometric polynomials).  The formulas are in mig.h.
//
// Mapping (k_design, both dimensions): a team of 1 to 3 waves designs EB = 1 or 2 entries.  What
// costs is the normal matrix: K (K+1) / 2 + 2 K sums over the design grid, 31 times per
// entry.  Each sum runs over the grid in increasing order (another order moves the
// fitted table by 1e-10: the fit's conditioning), so a sum is one thread's; a thread
// owns a 2 x 2 tile of them for all EB entries, which share the basis rows: per grid
// point 4 basis values and a weight per entry from LDS for 10 operations per entry.
// The basis streams through LDS in chunks of 64 grid points; the response |H| that
// reweights a point is evaluated from the same chunk, just before the chunk is summed.
// The system is solved by one wave (or half of one) per entry: the rest of a row per lane
// in registers, one LDS exchange of the current column per elimination step, the
// right-hand sides as two more rows.
#include "common.hpp"

namespace mig {
namespace {

constexpr int kMaxM2 = MIG_MAX_NTAPS_2D / 2;      // 5
constexpr int kDesignMaxSlots = 2048;         // entries in flight (1-D: target values in the workspace)

// A[i][n] = 1 (n = 0) or 2 cos(n theta_i) on the design midpoint grid; Ct[n][c]
// likewise on the check grid, point fastest.
__global__ void k_design_basis(int L, int Lc, int K, double* A, double* Ct)
{
#pragma clang fp contract(off)
    int tid = blockIdx.x * blockDim.x + threadIdx.x;
    int total = (L + Lc) * K;
    for (int e = tid; e < total; e += gridDim.x * blockDim.x) {
        if (e < L * K) {
            const int i = e / K, n = e % K;
            double th = ((double)i + 0.5) * kPi / (double)L;
            A[e] = n == 0 ? 1.0 : 2.0 * cos((double)n * th);
        } else {
            const int n = (e - L * K) / Lc, c = (e - L * K) % Lc;
            double th = ((double)c + 0.5) * kPi / (double)Lc;
            Ct[(size_t)n * Lc + c] = n == 0 ? 1.0 : 2.0 * cos((double)n * th);
        }
    }
}

struct DesignParams {
    int nk, K, L, Lc, nreweight, M;
    double kmin, dk, dx, zeta, edge_sin;
    double w_pass, w_trans, w_evan, lambda, beta, tau, margin;
};

DesignParams design_params(const mig_table_desc* d)
{
    DesignParams P;
    P.nk = d->nk;
    P.K = 0;
    P.M = (d->ntaps - 1) / 2;
    P.L = d->ngrid;
    P.Lc = d->ncheck;
    P.nreweight = d->nreweight;
    P.kmin = d->kmin;
    P.dk = (d->kmax - d->kmin) / (double)(d->nk - 1);
    P.dx = d->dx;
    P.zeta = d->dz / d->dx;
    P.edge_sin = sin(d->theta_max_deg * kPi / 180.0);
    P.w_pass = d->w_pass;
    P.w_trans = d->w_trans;
    P.w_evan = d->w_evan;
    P.lambda = d->lambda;
    P.beta = d->beta;
    P.tau = d->tau;
    P.margin = d->margin;
    return P;
}

// ---- 2-D circularly symmetric extrapolators (3-D extension, Sec. II) ----
//
// Unique coefficient u = a (a + 1) / 2 + b, a >= b >= 0, stands for the taps
// (n1, n2) with max(|n1|,|n2|) = a and min = b.  Its basis function on
// (theta_x, theta_y) is the sum of cos(n1 tx) cos(n2 ty) over that orbit:
//   1;  2 (cos a tx + cos a ty);  4 cos a tx cos a ty;
//   4 (cos a tx cos b ty + cos b tx cos a ty)          (a = 0; b = 0; a = b; a > b).
__device__ __forceinline__ double orbit_basis(int a, int b, const double* cx, const double* cy)
{
#pragma clang fp contract(off)
    if (a == 0) return 1.0;
    if (b == 0) return 2.0 * (cx[a] + cy[a]);
    if (a == b) return 4.0 * cx[a] * cy[a];
    return 4.0 * (cx[a] * cy[b] + cx[b] * cy[a]);
}

// A[(i L + q)][u] on the L x L design midpoint grid; CS[c][n] = cos(n theta_c)
// on the Lc check grid (the check evaluates the basis from it).
__global__ void k_design2d_basis(int L, int Lc, int M, double* A, double* CS)
{
#pragma clang fp contract(off)
    const int NU = (M + 1) * (M + 2) / 2;
    const size_t nA = (size_t)L * L, total = nA + (size_t)Lc;
    for (size_t e = (size_t)blockIdx.x * blockDim.x + threadIdx.x; e < total;
         e += (size_t)gridDim.x * blockDim.x) {
        if (e < nA) {
            const int i = (int)(e / L), q = (int)(e % L);
            double cx[kMaxM2 + 1], cy[kMaxM2 + 1];
            const double tx = ((double)i + 0.5) * kPi / (double)L;
            const double ty = ((double)q + 0.5) * kPi / (double)L;
            for (int n = 0; n <= M; ++n) { cx[n] = cos((double)n * tx); cy[n] = cos((double)n * ty); }
            for (int a = 0, u = 0; a <= M; ++a)
                for (int b = 0; b <= a; ++b, ++u) A[e * NU + u] = orbit_basis(a, b, cx, cy);
        } else {
            const int c = (int)(e - nA);
            const double th = ((double)c + 0.5) * kPi / (double)Lc;
            for (int n = 0; n <= M; ++n) CS[(size_t)c * (M + 1) + n] = cos((double)n * th);
        }
    }
}

typedef double v2f64 __attribute__((ext_vector_type(2)));

// Stored weights and targets per entry: the grid, or in two dimensions its points
// with q <= i (basis row, target and weight of (i, q) and (q, i) are equal).
__host__ __device__ constexpr int design_points(int L, bool two_d) { return two_d ? L * (L + 1) / 2 : L; }

// Waves of a workgroup: as many as its tiles of 2 x 2 sums need (K (K+2) / 8
// of the normal matrix and K / 2 per entry of the right-hand sides: 63 at K = 18 and
// two entries, 102 at 24, 168 at 32).
__host__ __device__ constexpr int design_waves(int KT) { return KT <= 18 ? 1 : (KT <= 24 ? 2 : 3); }

// Teams of that many waves in a workgroup, at most: each designs its own entries.  With
// 256 registers two waves fit on a SIMD, and workgroups of one or two waves that share a
// CU are put on the same SIMDs while the others idle (11 x 11 taps, 1024 entries: 8.75
// ms); the four waves of one workgroup are spread over the four (6.15 ms: teams of two
// waves then meet at the same barriers).  Where two teams of two waves per CU are all
// there is, each wave asks for a SIMD of its own instead (5.78 ms; SOLO).
__host__ __device__ constexpr int design_teams(int KT) { return 4 / design_waves(KT); }

constexpr int kDesignChunk = 64;  // grid points per chunk of the basis

// A grid point's row in LDS, in doubles: KT basis values (an even count), the targets
// of the workgroup's EB entries, their weights.  Pairs are 16-byte aligned (LDS returns
// 16-byte reads at twice the rate of 8-byte ones) and the stride is an odd multiple of
// two pairs (no bank conflicts where each lane reads another row).
__host__ __device__ constexpr int design_target_col(int KT) { return (KT + 1) & ~1; }
__host__ __device__ constexpr int design_weight_col(int KT, int eb) { return design_target_col(KT) + 2 * eb; }
__host__ __device__ constexpr int design_stride(int KT, int eb)
{
    const int n = design_weight_col(KT, eb) + eb;
    return n <= 2 ? 2 : (n + 1) / 4 * 4 + 2;
}

// LDS, in doubles: weights (and, in two dimensions, targets) of every entry; the
// solver's exchange rows and solution; the chunk's rows or, between two passes over
// the grid, the systems.
struct DesignLds {
    int w, d, x, h, a, g, total;
};

__host__ __device__ inline DesignLds design_lds(int L, int KT, int eb, bool two_d)
{
    DesignLds o;
    const int np = design_points(L, two_d);
    int at = 0;
    o.w = at;
    at += (np * eb + 1) & ~1;
    o.d = at;
    at += two_d ? 2 * np * eb : 0;
    o.x = at;
    at += eb * 2 * (KT + 8);
    o.h = at;
    at += eb * 2 * KT;
    o.a = o.g = at;
    const int rows = kDesignChunk * design_stride(KT, eb) + 2, sys = eb * (KT + 2) * (KT | 1);
    o.total = (at + (rows > sys ? rows : sys) + 1) & ~1;
    return o;
}

__device__ __forceinline__ void wave_lds_fence()
{
    // LDS keeps one wave's accesses in order: only the compiler has to
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_sched_barrier(0);
}

// Cholesky of the lower triangle G (rows of stride KT | 1) with the right-hand sides
// as rows KT and KT + 1, then the back substitution, by the lanes r = 0 .. KT+1 of one
// wave or half of one: lane r keeps what is left of row r in registers, shifted by a
// place per column (so that the columns are a loop: unrolled they took the kernel to 512
// registers and spills), and per column the lanes exchange their column values and
// diagonals through x once.  Every element sees its subtractions in the order of a
// sequential Cholesky and substitution.
constexpr int kSolveAhead = 8;  // products read at a time in the substitution
template <int KT>
__host__ __device__ constexpr int design_exchange() { return KT + kSolveAhead; }  // pairs

template <int KT>
__device__ __forceinline__ void design_solve(double* G, v2f64* x, v2f64* h, int K, int r, int* fail)
{
#pragma clang fp contract(off)
    // a value the compiler cannot see through: what follows from it (a mask per column)
    // is formed here each time, not kept in registers over the passes
    asm volatile("" : "+v"(r), "+s"(K));
    constexpr int LD = KT | 1, U = kSolveAhead;
    const bool rhs = r == KT || r == KT + 1, in = r < K;
    double* const row = G + (rhs || in ? r : 0) * LD;
    double* const col = reinterpret_cast<double*>(x);
    double* const dg = col + KT + 2;
    double g[KT];
#pragma unroll
    for (int q = 0; q < KT; ++q) {
        const double v = row[q];
        g[q] = q < K && (rhs || (in && q <= r)) ? v : 0.0;
        if (q % 8 == 7) __builtin_amdgcn_sched_barrier(0);
    }
    double diag = in ? row[in ? r : 0] : 1.0;
    bool bad = false;
    // A column's values v after division by the root of its pivot.  (The empty statement
    // keeps the division out of a branch of its own.)
    const auto divided = [&](int m, double v, double pivot) {
        bad = bad || (m < K && !(pivot > 0.0));
        const double d = sqrt(pivot > 0.0 ? pivot : 1.0);
        v = v / d;
        asm volatile("" : "+v"(v));
        return r == m ? d : v;
    };
    double l = divided(0, g[0], G[0]);
    // lanes without a row: places that no one reads
    double* const my_col = col + (r < KT + 2 ? r : 2 * KT + 4);
    double* const my_dg = r < KT + 2 ? dg + r : col + 2 * KT + 5;
    for (int m = 0; m < K; ++m) {  // g[i]: column m + i
        *my_col = l;
        *my_dg = diag;
        if (rhs || in) row[m] = l;  // (above the diagonal: values that no one reads)
        wave_lds_fence();
        const double n = col[m + 1], dn = dg[m + 1];
        constexpr int NC = KT <= 24 ? KT : 16;
        double c[NC];  // the other columns' values arrive beside the root
#pragma unroll
        for (int i = 2; i < NC; ++i) c[i] = col[m + i];
        __builtin_amdgcn_sched_barrier(0);
        const double l_next = divided(m + 1, g[1 < KT ? 1 : 0] - l * n, dn - n * n);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int i = 2; i < KT; ++i)  // past column K - 1: unused
            g[i - 1] = g[i] - l * (i < NC ? c[i < NC ? i : 0] : col[m + i]);
        diag -= l * l;
        l = l_next;
        wave_lds_fence();
    }
    if (bad && r == 0) *fail = 1;
    // x: per unknown m, the products of the lanes q > m that are subtracted from it (zeros
    // past the last); what the next unknown needs is read an unknown ahead
    double xr = 0.0, xi = 0.0, lm = 0.0, d = G[(K - 1) * LD + K - 1];
    v2f64 s = {G[KT * LD + K - 1], G[(KT + 1) * LD + K - 1]};
    for (int m = K - 1; m >= 0; --m) {
        if (r < KT + U) x[r] = v2f64{lm * xr, lm * xi};
        wave_lds_fence();
        v2f64 v[U];
#pragma unroll
        for (int u = 0; u < U; ++u) v[u] = x[m + 1 + u];
        const int mn = m > 0 ? m - 1 : 0;
        const double d_next = G[mn * LD + mn];
        const v2f64 s_next = {G[KT * LD + mn], G[(KT + 1) * LD + mn]};
        const double row_next = row[mn];
        for (int q = m + 1; q < K; q += U) {
            v2f64 n[U];
            const int next = q + U < K ? q + U : m + 1;
#pragma unroll
            for (int u = 0; u < U; ++u) n[u] = x[next + u];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                s -= v[u];
                v[u] = n[u];
            }
        }
        const double yr = s.x / d, yi = s.y / d;
        xr = r == m ? yr : xr;
        xi = r == m ? yi : xi;
        d = d_next;
        s = s_next;
        lm = in && r > mn ? row_next : 0.0;
        wave_lds_fence();
    }
    if (in) h[r] = v2f64{xr, xi};
}

// Barrier of a team: of the workgroup, or within the wave (teams of one wave each go
// their own way: in step, with all of them at the sums at once, 1-D designs take 10 % more).
template <int W>
__device__ __forceinline__ void team_sync()
{
    if constexpr (W == 1) wave_lds_fence();
    else __syncthreads();
}

// Phase shift over dz at kz^2 = q (in units of dx), or the decay past the cutoff.  A
// function of its own keeps its constants out of the caller's registers.
__device__ __noinline__ v2f64 design_target(double zeta, double q, bool propagating)
{
#pragma clang fp contract(off)
    if (propagating) {
        double sn, cs;
        sincos(zeta * sqrt(q), &sn, &cs);
        return v2f64{cs, sn};
    }
    return v2f64{exp(-zeta * sqrt(-q)), 0.0};
}

// Basis rows and targets of the chunk at c0.
template <int NV, int NE, int T, bool TWO_D>
__device__ __forceinline__ void design_fetch(v2f64 (&pre)[NV], v2f64 (&dpre)[NE], const double* A,
                                             const v2f64* Dg, int c0, int LL, int K, int t, int ip)
{
    const int last = ((LL * K + 1) & ~1) - 2;
#pragma unroll
    for (int v = 0; v < NV; ++v) {
        const int at = c0 * K + 2 * (v * T + t);
        pre[v] = *reinterpret_cast<const v2f64*>(A + (at < last ? at : last));
    }
#pragma unroll
    for (int e = 0; e < NE; ++e)
        dpre[e] = TWO_D ? v2f64{0.0, 0.0} : Dg[e * LL + (c0 + ip < LL ? c0 + ip : LL - 1)];
}

// Bound by instruction issue (one wave per SIMD: about 6 cycles per FP64 operation).
// 35 taps, 2048 entries: 16.0 -> 2.90 ms per table; 11 x 11 taps, 1024 entries: 28.4 ->
// 5.78 ms; 63 taps, 2048 entries: 51.0 -> 9.1 ms (before: one workgroup per entry, a
// thread per sum reading the basis from L2, the solves on one thread).  Of a pass of two
// 35-tap entries the sums take 154 k of 224 k cycles, the solves 28 k, the responses
// 27 k, the chunks' copies 12 k.
//
// Every instance keeps to 256 registers, without accumulation registers, spills or
// scratch (tests/test_build_resources.py holds it to that): a build of this kernel that
// moved values to the accumulation file inside a branch of part of a wave gave that
// wave's idle lanes wrong addresses, and what the compiler does there was not found out.
// What it takes: columns of the solve as a loop, one point's coefficients read some at a
// time, sums pinned where they are formed.  With 390-512 registers instead, the solve's
// columns unrolled, the listed tables took 2.83, 5.72 and 14.7 ms.  (Threads past the
// tiles repeat the first one's sums: no branch of part of a wave holds them.)
template <int EB, int KT, bool TWO_D, bool SOLO>
__global__ void __launch_bounds__(64 * design_waves(KT) * (SOLO ? 1 : design_teams(KT)))
    __attribute__((amdgpu_waves_per_eu(SOLO ? 1 : 2, SOLO ? 1 : 8)))
k_design(DesignParams P, const double* __restrict__ A, const double* __restrict__ C, v2f64* D,
         mig_c128* tab64, mig_c64* tab32, double* maxgain, double* passerr, int* status)
{
#pragma clang fp contract(off)
    extern __shared__ v2f64 smem2[];
    constexpr int W = design_waves(KT), T = 64 * W, CH = kDesignChunk;
    constexpr int RS = design_stride(KT, EB), RP = RS / 2, LD = KT | 1;
    constexpr int DC = design_target_col(KT), WC = design_weight_col(KT, EB);
    constexpr int TM = SOLO ? 1 : design_teams(KT);  // teams of a workgroup, at most
    __shared__ double s_red_[TM][EB][TM * W];
    __shared__ int s_fail_[TM][EB];
    const int teams = blockDim.x / T, team = __builtin_amdgcn_readfirstlane(threadIdx.x / T);
    const int K = P.K, L = P.L, t = threadIdx.x - team * T, wave = __builtin_amdgcn_readfirstlane(t >> 6);
    double (&s_red)[EB][TM * W] = s_red_[team];
    int (&s_fail)[EB] = s_fail_[team];
    const int LL = TWO_D ? L * L : L, np = design_points(L, TWO_D);
    const DesignLds o = design_lds(L, KT, EB, TWO_D);
    v2f64* const dyn2 = smem2 + team * (o.total / 2);
    double* const dyn = reinterpret_cast<double*>(dyn2);
    double* const w = dyn + o.w;
    double* const rows = dyn + o.a;
    const v2f64* const rows2 = dyn2 + o.a / 2;
    v2f64* const hs = dyn2 + o.h / 2;

    // this thread's share of a chunk: point ip of entries e0 .. e0 + NE - 1 (a wave per
    // entry where there are enough)
    constexpr int NE = W >= EB ? 1 : EB;
    const int ip = t & 63, e0 = NE == 1 && wave < EB ? wave : 0;
    const bool mine = NE > 1 || wave < EB;
    // this thread's tile: coefficients 2 bp, 2 bp + 1 against 2 bq, 2 bq + 1, or
    // against the right-hand sides of entry aug
    const int nb = (K + 1) / 2, ntri = nb * (nb + 1) / 2;
    const bool tile = t < ntri + nb * EB;
    int bp = 0, bq = 0, aug = -1;
    if (t < ntri) {
        while ((bp + 1) * (bp + 2) / 2 <= t) ++bp;
        bq = t - bp * (bp + 1) / 2;
    } else if (tile) {
        aug = (t - ntri) / nb;
        bp = (t - ntri) % nb;
    }
    const v2f64* const pa = rows2 + bp;
    const v2f64* const qa = rows2 + (aug < 0 ? bq : DC / 2 + aug);
    const double* const wa = rows + WC;
    // LDS places of the basis values this thread copies per chunk (values past the
    // chunk's rows go to the place after them)
    constexpr int NV = (CH * KT / 2 + T - 1) / T;
    unsigned to[NV];  // two places in 16 bits each
#pragma unroll
    for (int v = 0; v < NV; ++v) {
        const auto place = [&](int at) -> unsigned {
            const int row = at / K;
            return row < CH ? row * RS + at - row * K : CH * RS;
        };
        to[v] = place(2 * (v * T + t)) | place(2 * (v * T + t) + 1) << 16;
    }

    for (int gi = blockIdx.x * teams; gi * EB < P.nk; gi += gridDim.x * teams) {
        // the entries of this team (past the table's end: the last one again)
        const int j0 = (gi + team) * EB;
        v2f64* const Dg = TWO_D ? dyn2 + o.d / 2 : D + (size_t)(blockIdx.x * teams + team) * EB * L;
        team_sync<W>();
        for (int v = t; v < np * EB; v += T) {
            const int e = v / np, x = v - e * np;
            const int j = j0 + e < P.nk ? j0 + e : P.nk - 1;
            const double kappa = (P.kmin + (double)j * P.dk) * P.dx;
            const double edge = kappa * P.edge_sin;
            double r, r2;
            if (TWO_D) {
                int i = (int)((sqrt(8.0 * (double)x + 1.0) - 1.0) * 0.5);
                while (i * (i + 1) / 2 > x) --i;
                while ((i + 1) * (i + 2) / 2 <= x) ++i;
                const double tx = ((double)i + 0.5) * kPi / (double)L;
                const double ty = ((double)(x - i * (i + 1) / 2) + 0.5) * kPi / (double)L;
                r2 = tx * tx + ty * ty;
                r = sqrt(r2);
            } else {
                r = ((double)x + 0.5) * kPi / (double)L;
                r2 = r * r;
            }
            const double k2 = kappa * kappa;
            Dg[v] = design_target(P.zeta, k2 - r2, TWO_D ? r2 <= k2 : r <= kappa);
            w[v] = r <= edge ? P.w_pass : (r <= kappa ? P.w_trans : P.w_evan);
        }
        for (int v = t; v < EB * KT; v += T) hs[v] = v2f64{0.0, 0.0};  // coefficients past K
        if (t < EB) s_fail[t] = 0;
        team_sync<W>();

        for (int it = 0; it <= P.nreweight; ++it) {
            double acc[EB][2][2];
#pragma unroll
            for (int e = 0; e < EB; ++e)
                acc[e][0][0] = acc[e][0][1] = acc[e][1][0] = acc[e][1][1] = 0.0;
            // basis columns K .. KT-1 are zeros (the systems had their place)
            for (int v = t; v < CH * (KT - K); v += T) rows[v / (KT - K) * RS + K + v % (KT - K)] = 0.0;
            // The chunk's basis rows (contiguous) and targets are loaded one chunk
            // ahead, without branches (a load that may not have been issued would be
            // waited for at once): addresses are clamped into the grid, whose last
            // pair may reach into the workspace's padding, and rows past the chunk's
            // are copied but not read.
            v2f64 pre[NV], dpre[NE];
            design_fetch<NV, NE, T, TWO_D>(pre, dpre, A, Dg + e0 * LL, 0, LL, K, t, ip);
            for (int c0 = 0; c0 < LL; c0 += CH) {
                const int n = LL - c0 < CH ? LL - c0 : CH;
                team_sync<W>();  // the previous chunk has been summed
                v2f64 dn[NE];
#pragma unroll
                for (int v = 0; v < NV; ++v) {
                    rows[to[v] & 0xffffu] = pre[v].x;
                    rows[to[v] >> 16] = pre[v].y;
                }
#pragma unroll
                for (int e = 0; e < NE; ++e) dn[e] = dpre[e];
                design_fetch<NV, NE, T, TWO_D>(pre, dpre, A, Dg + e0 * LL, c0 + CH < LL ? c0 + CH : 0, LL, K, t, ip);
                team_sync<W>();
                int x = c0 + ip < LL ? c0 + ip : LL - 1;
                asm volatile("" : "+v"(x));
                bool mirrored = false;
                if (TWO_D) {
                    const int i = x / L, q = x - i * L;
                    mirrored = i > q;  // its mirror image came first and updates the weight
                    x = mirrored ? i * (i + 1) / 2 + q : q * (q + 1) / 2 + i;
                }
                if (it > 0 && mine) {
                    // response of the last fit, and the weights where it exceeds one
                    const v2f64* const a2 = rows2 + ip * RP;
                    double Hr[NE] = {}, Hi[NE] = {};
                    // some coefficients (those past K are zero) are read while those
                    // before them are summed
                    constexpr int B = NE == 2 ? 2 : 4;
                    struct Coef {
                        v2f64 a[B / 2], h[NE][B];
                    };
                    const auto get = [&](Coef& c, int q) {
#pragma unroll
                        for (int u = 0; u < B; ++u)
                            if (q + u < KT) {
                                if (u % 2 == 0) c.a[u / 2] = a2[(q + u) / 2];
#pragma unroll
                                for (int e = 0; e < NE; ++e) c.h[e][u] = hs[(e0 + e) * KT + q + u];
                            }
                    };
                    Coef now, next;
                    get(now, 0);
#pragma unroll
                    for (int q = 0; q < KT; q += B) {
                        get(next, q + B);
                        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                        for (int u = 0; u < B; ++u)
                            if (q + u < KT)
#pragma unroll
                                for (int e = 0; e < NE; ++e) {
                                    const double a = u % 2 == 0 ? now.a[u / 2].x : now.a[u / 2].y;
                                    Hr[e] += a * now.h[e][u].x;
                                    Hi[e] += a * now.h[e][u].y;
                                }
                        // (sunk into the branch below, the sums would leave every value
                        // read above it in registers)
#pragma unroll
                        for (int e = 0; e < NE; ++e) asm volatile("" : "+v"(Hr[e]), "+v"(Hi[e]));
                        __builtin_amdgcn_sched_barrier(0);
                        now = next;
                    }
#pragma unroll
                    for (int e = 0; e < NE; ++e)
                        // clearly below one: no excess (hypot errs by an ulp)
                        if (ip < n && !mirrored && !(Hr[e] * Hr[e] + Hi[e] * Hi[e] < 1.0 - 1e-12)) {
                            const double excess = hypot(Hr[e], Hi[e]) - 1.0;
                            double& we = w[(e0 + e) * np + x];
                            if (excess > 0.0) we = we * (1.0 + P.beta * excess / P.tau);
                        }
                }
                if (TWO_D) team_sync<W>();  // both images of a point may lie in this chunk
                if (mine)
#pragma unroll
                    for (int e = 0; e < NE; ++e) {
                        rows[ip * RS + WC + e0 + e] = w[(e0 + e) * np + x];
                        *reinterpret_cast<v2f64*>(rows + ip * RS + DC + 2 * (e0 + e)) =
                            TWO_D ? Dg[(e0 + e) * np + x] : dn[e];
                    }
                team_sync<W>();
                // Few waves share a SIMD here, so the order is explicit: U grid points'
                // operands are read while the U before them are summed, and each point's
                // products stand apart from their sums.
                constexpr int U = 4;
                struct Ops {
                    v2f64 p, q;
                    double w[EB];
                };
                auto read1 = [&](Ops& v, int i) {
                    v.p = pa[i * RP];
                    v.q = qa[i * RP];
                    if constexpr (EB == 2) {
                        const v2f64 w2 = *reinterpret_cast<const v2f64*>(wa + i * RS);
                        v.w[0] = w2.x;
                        v.w[EB - 1] = w2.y;
                    } else {
                        v.w[0] = wa[i * RS];
                    }
                };
                auto read = [&](Ops (&v)[U], int i) {
#pragma unroll
                    for (int u = 0; u < U; ++u) read1(v[u], i + u);
                };
                auto add = [&](const Ops& v) {
                    double w0[EB], w1[EB], m[EB][2][2];
#pragma unroll
                    for (int e = 0; e < EB; ++e) {
                        w0[e] = v.w[e] * v.p.x;
                        w1[e] = v.w[e] * v.p.y;
                    }
#pragma unroll
                    for (int e = 0; e < EB; ++e) {
                        m[e][0][0] = w0[e] * v.q.x;
                        m[e][0][1] = w0[e] * v.q.y;
                        m[e][1][0] = w1[e] * v.q.x;
                        m[e][1][1] = w1[e] * v.q.y;
                    }
#pragma unroll
                    for (int e = 0; e < EB; ++e) {
                        acc[e][0][0] += m[e][0][0];
                        acc[e][0][1] += m[e][0][1];
                        acc[e][1][0] += m[e][1][0];
                        acc[e][1][1] += m[e][1][1];
                    }
                };
                const int full = n / (2 * U) * (2 * U);
                Ops va[U], vb[U];
                if (full > 0) read(va, 0);
                for (int i = 0; i < full; i += 2 * U) {
                    read(vb, i + U);
                    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                    for (int u = 0; u < U; ++u) add(va[u]);
                    __builtin_amdgcn_sched_barrier(0);
                    read(va, i + 2 * U < full ? i + 2 * U : 0);
                    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                    for (int u = 0; u < U; ++u) add(vb[u]);
                    __builtin_amdgcn_sched_barrier(0);
                }
                for (int i = full; i < n; ++i) {
                    Ops v;
                    read1(v, i);
                    add(v);
                }
            }
            // the systems take the rows' place
            team_sync<W>();
            if (tile)
#pragma unroll
                for (int e = 0; e < EB; ++e) {
                    double* const G = dyn + o.g + e * (KT + 2) * LD;
#pragma unroll
                    for (int u = 0; u < 2; ++u)
#pragma unroll
                        for (int v = 0; v < 2; ++v) {
                            const int p = 2 * bp + u, q = 2 * bq + v;
                            double s = acc[e][u][v];
                            if (aug >= 0) {
                                if (aug == e && p < K) G[(KT + v) * LD + p] = s;
                            } else if (p < K && q <= p) {
                                if (p == q) s += P.lambda;
                                G[p * LD + q] = s;
                            }
                        }
                }
            team_sync<W>();
            // a wave per entry, or half a wave (KT <= 18: 32 lanes hold the KT + 2 rows)
            {
                constexpr bool half = NE > 1;
                int se = half ? t >> 5 : wave;
                const int sr = half ? t & 31 : t & 63;
                asm volatile("" : "+v"(se));
                if (half || wave < EB)
                    design_solve<KT>(dyn + o.g + se * (KT + 2) * LD,
                                     dyn2 + o.x / 2 + se * design_exchange<KT>(), hs + se * KT, K, sr,
                                     &s_fail[se]);
            }
            team_sync<W>();
        }

        // Stability scale: |H|max <= max_grid |H| / cos(M pi / (2 Lc)) (in two dimensions
        // the bound applies along each axis, hence squared).
        // g2 screens points whose |H| cannot be the largest.
        auto raise = [&](double& g, double& g2, double Hr, double Hi) {
            const double s2 = Hr * Hr + Hi * Hi;
            if (!(s2 < g2)) {
                g = fmax(g, hypot(Hr, Hi));
                g2 = s2 * (1.0 - 1e-12);
            }
        };
        auto wave_max = [&](double v) {
#pragma unroll
            for (int off = 32; off >= 1; off >>= 1) v = fmax(v, __shfl_xor(v, off, 64));
            return v;
        };
        auto block_max = [&](double (&v)[EB]) {
#pragma unroll
            for (int e = 0; e < EB; ++e) {
                v[e] = wave_max(v[e]);
                if ((t & 63) == 0) s_red[e][t >> 6] = v[e];
            }
            team_sync<W>();
#pragma unroll
            for (int e = 0; e < EB; ++e)
#pragma unroll
                for (int q = 0; q < W; ++q) v[e] = fmax(v[e], s_red[e][q]);
            team_sync<W>();
        };
        double g[EB];
#pragma unroll
        for (int e = 0; e < EB; ++e) g[e] = 0.0;
        if constexpr (TWO_D) {
            // |H| is symmetric: points with q <= i
            const int Lc = P.Lc, M = P.M;
            double g2[EB] = {};
            for (int x = t; x < Lc * Lc; x += T) {
                const int i = x / Lc, q = x - i * Lc;
                if (q > i) continue;
                double cx[kMaxM2 + 1], cy[kMaxM2 + 1];
#pragma unroll
                for (int a = 0; a <= kMaxM2; ++a) {
                    cx[a] = C[(size_t)i * (M + 1) + (a <= M ? a : 0)];
                    cy[a] = C[(size_t)q * (M + 1) + (a <= M ? a : 0)];
                }
                double Hr[EB] = {}, Hi[EB] = {};
#pragma unroll
                for (int a = 0; a <= kMaxM2; ++a)
#pragma unroll
                    for (int b = 0; b <= a; ++b) {
                        const int u = a * (a + 1) / 2 + b;
                        if (u < KT && a <= M) {
                            const double f = orbit_basis(a, b, cx, cy);
#pragma unroll
                            for (int e = 0; e < EB; ++e) {
                                const v2f64 hv = hs[e * KT + (u < KT ? u : 0)];
                                Hr[e] += f * hv.x;
                                Hi[e] += f * hv.y;
                            }
                        }
                    }
#pragma unroll
                for (int e = 0; e < EB; ++e) raise(g[e], g2[e], Hr[e], Hi[e]);
            }
            block_max(g);
        } else {
            // The workgroup's teams share the points, and each point's basis values serve the
            // entries of all: each team reading the whole basis, some waited for it four
            // times as long as the arithmetic takes (35 taps, 2048 entries, in all 2.98 ->
            // 2.90 ms).  NP points at a time share the reads of the coefficients
            // (where registers allow).
            constexpr int NP = KT <= 12 || (KT <= 18 && EB == 1) ? 2 : 1;
            double ga[TM][EB] = {}, g2[TM][EB] = {};
            __syncthreads();  // every team's coefficients
            for (int c = threadIdx.x; c < P.Lc; c += NP * blockDim.x) {
                int Kc = K;
                asm volatile("" : "+s"(Kc));  // (hoisted, the rows' offsets would fill the scalar registers)
                double cc[NP][KT];
#pragma unroll
                for (int u = 0; u < NP; ++u) {
                    const int at = c + u * blockDim.x < P.Lc ? c + u * blockDim.x : c;  // past the grid: again
#pragma unroll
                    for (int q = 1; q < KT; ++q) cc[u][q] = C[(size_t)(q < Kc ? q : 0) * P.Lc + at];
                }
#pragma unroll
                for (int m = 0; m < TM; ++m) {
                    if (m >= teams) break;
                    const v2f64* const ht = smem2 + m * (o.total / 2) + o.h / 2;
#pragma unroll
                    for (int e = 0; e < EB; ++e) {
                        double Hr[NP], Hi[NP];
#pragma unroll
                        for (int u = 0; u < NP; ++u) {
                            Hr[u] = ht[e * KT].x;
                            Hi[u] = ht[e * KT].y;
                        }
#pragma unroll
                        for (int q = 1; q < KT; ++q) {  // coefficients past K are zero
                            const v2f64 hv = ht[e * KT + q];
#pragma unroll
                            for (int u = 0; u < NP; ++u) {
                                Hr[u] += cc[u][q] * hv.x;
                                Hi[u] += cc[u][q] * hv.y;
                                if (q % 8 == 7) asm volatile("" : "+v"(Hr[u]), "+v"(Hi[u]));
                            }
                            if (q % 8 == 7) __builtin_amdgcn_sched_barrier(0);
                        }
#pragma unroll
                        for (int u = 0; u < NP; ++u) raise(ga[m][e], g2[m][e], Hr[u], Hi[u]);
                    }
                }
            }
#pragma unroll
            for (int m = 0; m < TM; ++m)
#pragma unroll
                for (int e = 0; e < EB; ++e) {
                    const double v = wave_max(ga[m][e]);
                    if ((threadIdx.x & 63) == 0) s_red_[m][e][threadIdx.x >> 6] = v;
                }
            __syncthreads();
#pragma unroll
            for (int e = 0; e < EB; ++e)
                for (int q = 0; q < teams * W; ++q) g[e] = fmax(g[e], s_red[e][q]);
            team_sync<W>();
        }
        const double cb = cos((double)P.M * kPi / (2.0 * (double)P.Lc));
        const double lim = TWO_D ? (1.0 - P.margin) * cb * cb : (1.0 - P.margin) * cb;
        double s[EB], perr[EB];
#pragma unroll
        for (int e = 0; e < EB; ++e) {
            s[e] = g[e] > lim ? lim / g[e] : 1.0;
            perr[e] = 0.0;
        }
        for (int x = t; x < LL; x += T) {
            double r;
            int at = x;
            if (TWO_D) {
                const int i = x / L, q = x - i * L;
                if (q > i) continue;  // symmetric
                const double tx = ((double)i + 0.5) * kPi / (double)L;
                const double ty = ((double)q + 0.5) * kPi / (double)L;
                r = sqrt(tx * tx + ty * ty);
                at = i * (i + 1) / 2 + q;
            } else {
                r = ((double)x + 0.5) * kPi / (double)L;
            }
            const double* a = A + (size_t)x * K;
#pragma unroll
            for (int e = 0; e < EB; ++e) {
                const int j = j0 + e < P.nk ? j0 + e : P.nk - 1;
                const double kappa = (P.kmin + (double)j * P.dk) * P.dx;
                if (!(r <= kappa * P.edge_sin)) continue;
                double Hr = 0.0, Hi = 0.0;
                for (int q = 0; q < K; ++q) {
                    Hr += a[q] * (s[e] * hs[e * KT + q].x);
                    Hi += a[q] * (s[e] * hs[e * KT + q].y);
                }
                const v2f64 dv = Dg[e * np + at];
                perr[e] = fmax(perr[e], hypot(Hr - dv.x, Hi - dv.y));
            }
        }
        block_max(perr);
#pragma unroll
        for (int e = 0; e < EB; ++e) {
            const int j = j0 + e;
            if (j >= P.nk) continue;
            for (int q = t; q < K; q += T) {
                const double hr = s[e] * hs[e * KT + q].x, hi = s[e] * hs[e * KT + q].y;
                tab64[(size_t)j * K + q] = mig_c128{hr, hi};
                if (tab32) tab32[(size_t)j * K + q] = mig_c64{(float)hr, (float)hi};
            }
            if (t == 0) {
                const double mg = s[e] * g[e];
                if (maxgain) maxgain[j] = mg;
                if (passerr) passerr[j] = perr[e];
                status[j] = s_fail[e] ? 2 : (mg <= 1.0 ? 0 : 1);
            }
        }
    }
}

template <int EB, int KT, bool TWO_D, bool SOLO>
int launch_design_teams(const DesignParams& P, const double* A, const double* C, v2f64* D,
                        mig_c128* tab64, mig_c64* tab32, double* maxgain, double* passerr, int* status,
                        int groups, int teams, size_t lds, hipStream_t s)
{
    if (lds > 64000 &&
        hipFuncSetAttribute(reinterpret_cast<const void*>(&k_design<EB, KT, TWO_D, SOLO>),
                            hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds) != hipSuccess)
        return MIG_E_DEVICE;
    int blocks = groups / teams + (groups % teams != 0);
    if (blocks > kDesignMaxSlots / (EB * teams)) blocks = kDesignMaxSlots / (EB * teams);
    hipLaunchKernelGGL((k_design<EB, KT, TWO_D, SOLO>), dim3(blocks), dim3(64 * design_waves(KT) * teams),
                       lds, s, P, A, C, D, tab64, tab32, maxgain, passerr, status);
    return hipGetLastError() == hipSuccess ? MIG_OK : MIG_E_DEVICE;
}

template <int EB, int KT, bool TWO_D>
int launch_design_as(const DesignParams& P, const double* A, const double* C, v2f64* D,
                     mig_c128* tab64, mig_c64* tab32, double* maxgain, double* passerr, int* status,
                     int cus, hipStream_t s)
{
    const size_t lds = (size_t)design_lds(P.L, KT, EB, TWO_D).total * sizeof(double);
    const int groups = P.nk / EB + (P.nk % EB != 0);
    // teams of two waves, two of them per CU
    if constexpr (design_waves(KT) == 2)
        if (groups > cus && groups <= 2 * cus)
            return launch_design_teams<EB, KT, TWO_D, true>(P, A, C, D, tab64, tab32, maxgain, passerr,
                                                            status, groups, 1, lds, s);
    // as many teams as keep every CU busy, within its LDS
    int teams = design_teams(KT);
    while (teams > 1 && (teams * lds > 159 * 1024 || (long long)(teams - 1) * cus >= groups)) --teams;
    return launch_design_teams<EB, KT, TWO_D, false>(P, A, C, D, tab64, tab32, maxgain, passerr, status,
                                                     groups, teams, teams * lds, s);
}

// Loops over coefficients are KT long (zeros past K).  Two entries per team once
// single ones would put more than one wave on a SIMD: a thread's sums of two entries
// share their basis reads and fill one wave's issue slots better than two waves do
// (with one wave per SIMD, 35 taps, 2048 entries: 2.82 against 3.81 ms; 11 x 11 taps,
// 1024: 5.7 / 8.3 ms); below that the second entry only lengthens the work of each wave
// (25 taps, 512 entries: 2.58 against 1.85 ms; 9 x 9 taps, 1024: 5.9 / 4.2 ms).
template <int KT, bool TWO_D>
int launch_design_kt(const DesignParams& P, const double* A, const double* C, v2f64* D,
                     mig_c128* tab64, mig_c64* tab32, double* maxgain, double* passerr, int* status,
                     hipStream_t s)
{
    int dev = 0, cus = 256;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess)
        cus = 256;
    return (long long)P.nk * design_waves(KT) > 4LL * cus
               ? launch_design_as<2, KT, TWO_D>(P, A, C, D, tab64, tab32, maxgain, passerr, status, cus, s)
               : launch_design_as<1, KT, TWO_D>(P, A, C, D, tab64, tab32, maxgain, passerr, status, cus, s);
}

}  // namespace

int launch_design2d_basis(const mig_table_desc* d, double* A, double* CS, hipStream_t s)
{
    const int M = (d->ntaps - 1) / 2;
    const size_t total = (size_t)d->ngrid * d->ngrid + d->ncheck;
    size_t blocks = (total + 255) / 256;
    if (blocks > 4096) blocks = 4096;
    hipLaunchKernelGGL(k_design2d_basis, dim3((unsigned)blocks), dim3(256), 0, s, d->ngrid,
                       d->ncheck, M, A, CS);
    return hipGetLastError() == hipSuccess ? MIG_OK : MIG_E_DEVICE;
}

int launch_design2d(const mig_table_desc* d, const double* A, const double* CS,
                    mig_c128* tab64, mig_c64* tab32, double* maxgain, double* passerr,
                    int* status, hipStream_t s)
{
    DesignParams P = design_params(d);
    P.K = (P.M + 1) * (P.M + 2) / 2;
    if (P.K <= 15) return launch_design_kt<15, true>(P, A, CS, nullptr, tab64, tab32, maxgain, passerr, status, s);
    return launch_design_kt<21, true>(P, A, CS, nullptr, tab64, tab32, maxgain, passerr, status, s);
}

int launch_design_basis(const mig_table_desc* d, double* A, double* C, hipStream_t s)
{
    const int K = (d->ntaps - 1) / 2 + 1;
    int total = (d->ngrid + d->ncheck) * K;
    int blocks = (total + 255) / 256;
    if (blocks > 4096) blocks = 4096;
    hipLaunchKernelGGL(k_design_basis, dim3(blocks), dim3(256), 0, s, d->ngrid,
                       d->ncheck, K, A, C);
    return hipGetLastError() == hipSuccess ? MIG_OK : MIG_E_DEVICE;
}

size_t design_target_bytes(const mig_table_desc* d)
{
    const size_t slots = (size_t)d->nk + 8;  // the last workgroup's teams may pass the end
    return (slots < (size_t)kDesignMaxSlots ? slots : (size_t)kDesignMaxSlots) * d->ngrid * sizeof(double2);
}

int launch_design(const mig_table_desc* d, const double* A, const double* C, void* targets,
                  mig_c128* tab64, mig_c64* tab32, double* maxgain,
                  double* passerr, int* status, hipStream_t s)
{
    DesignParams P = design_params(d);
    P.K = P.M + 1;
    v2f64* const D = static_cast<v2f64*>(targets);
    if (P.K <= 12) return launch_design_kt<12, false>(P, A, C, D, tab64, tab32, maxgain, passerr, status, s);
    if (P.K <= 18) return launch_design_kt<18, false>(P, A, C, D, tab64, tab32, maxgain, passerr, status, s);
    if (P.K <= 24) return launch_design_kt<24, false>(P, A, C, D, tab64, tab32, maxgain, passerr, status, s);
    return launch_design_kt<32, false>(P, A, C, D, tab64, tab32, maxgain, passerr, status, s);
}

}  // namespace mig
