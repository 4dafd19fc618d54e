// Fitness evaluation of a population of allocation matrices on gfx950.
//
// Pollux (arXiv 2008.12260): goodput model Sec. 3 (Eq. 4), statistical
// efficiency Sec. 3.1 (Eq. 6), throughput Sec. 3.2 (Eq. 7-11), per-job tuning
// Sec. 4.1 (Eq. 13), SPEEDUP / FITNESS_p, re-allocation penalty and
// interference avoidance Sec. 4.2 (Eq. 14-15).
//
// Kernels of a call with the dense grid in fp64 (three launches on the caller's stream)
//   prepare_kernel    everything that depends on the jobs only.  Per job, placement class and GPU count K <= 64
//                     (the "one node" class only up to the largest node capacity): T_sync (Eq. 9) and, for every
//                     batch size of the grid, T_grad(m) (Eq. 8), the last pass of Eq. 10,
//                     (T_grad^g + T_sync^g)^(1/g), the two terms C and A0 the sweep needs of it, and the feasible
//                     accumulation counts.  They depend on the allocation only through K and on whether the job sits
//                     on one node, so they are shared by the population.  Per job: parameter checks, restart
//                     factor, fair-share goodput (denominator of Eq. 15).  Also the largest node capacity; clears
//                     the status word and the per-node counters
//   pairs_kernel      per (candidate, job) (one wavefront): row reduce, sweep of the
//                     (m, s) grid, argmax; the row's non-zero entries are added to
//                     per-candidate, per-node counters with integer atomics
//   candidates_kernel per candidate (one workgroup): SPEEDUP, penalty, constraint
//                     check from those counters and the generalized mean
// Other calls (launch_fitness decides; a call that keeps the job tables leaves out what makes them):
//   fp32              memoised, memo_kernel_f32 finds the argmaxes from prepare_kernel's tables; grids of more than 32 counts have their
//                     fair shares found so too (jobs_kernel_f32)
//   PX_FLAG_MEMOISE   prepare_kernel takes the argmax once per (job, placement class, K <= 64) and the population pass looks it
//                     up: memo_candidates_kernel for rows of 4 to 256 nodes, which takes a whole candidate per workgroup and
//                     finishes its fitness as well (no per-pair scratch, no candidates_kernel); other rows in pairs_kernel
//   PX_FLAG_SAMPLE_M  sweep_sampled (Sec. 4.3) replaces the sweep, the kernels instantiated with CH = 0; from 128 candidates
//                     on rows of 4 to 256 nodes take the memoised pass
//   small calls       small_kernel does everything in one launch: up to 252 candidates and 16 groups of 64 batch sizes over all
//                     jobs (small_call)
// For pollux_generation the population pass takes a list of candidates, the children of the search step.  With
// PX_GA_INHERIT_ROWS an unchanged row takes over the results of the row it was copied from: memoised, on rows of 4 to 64 nodes, in
// child_kernel, which forms the child as well; in the children's instance of memo_candidates_kernel on longer ones; not at all in
// small_kernel (a row there costs no launch); and otherwise in inherit_kernel, which also lists the rows the step has changed per
// job for pairs_kernel.
//
// How one wavefront sweeps the grid of a (candidate, job) pair.  Lane l owns
// the batch sizes m_i, i = l, l+64, ...; it walks s = 0..Gs-1.  Dividing Eq. 4
// through by M gives
//     GOODPUT = (phi + M0) / h,   h(m, s) = T_iter(m, s) * (1 + phi / M),
// and with u = phi/(K m), last = (T_grad^g + T_sync^g)^(1/g):
//     h(m, s) = (last + u T_grad) + s T_grad + (last - T_grad) u / (s + 1)
//             = A0 + T_grad w(s),    w(s) = s + C / (s + 1),   C = (last - T_grad) u / T_grad,
// with every term non-negative.  The argmax of GOODPUT is the argmin of h over the
// feasible points.  For one batch size (one lane) that is the argmin of w over its
// feasible s, which form an interval s_lo..s_hi that depends on (job, K, m) only and is
// tabled.  The lane takes the smallest w over ALL s, one fused multiply-add and one minimum per grid point.  w is convex
// in s (C >= 0) and w(s+1) < w(s) precisely when C > (s+1)(s+2), so two exact comparisons say whether that minimum lies
// within s_lo..s_hi; where it does not, the feasible optimum is w at the end towards it.  h is formed from it once per lane
// and group of 64 batch sizes.  The wave then takes the smallest h (equal values: lowest flat index; elect_scanned says where the
// scan's last places must not decide); only now the count
// of the elected batch size is found, from its C by the same exact rule (px_best_count), and the elected point is evaluated
// again with the formulas in the paper's own order (separate multiply and add, IEEE
// division), so the reported goodput does not depend on the fast form.
//
// The last pass of Eq. 10 is evaluated as
//     max(Tg, Ts) * exp( log1p( exp(-g |ln Tg - ln Ts|) ) / g ),
// which is the same quantity with the larger term factored out: every
// intermediate stays in [0, ln 2] or [1, 2], so plain fp64 log/exp give a result
// within a few ulp, where a direct pow(pow + pow, 1/g) would need an extended
// precision logarithm.  T_sync = 0 and g = 1 are taken exactly (T_grad and the
// plain sum).

#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include "../../include/pollux.h"
#include "pollux_device.h"
#include "pollux_host.h"
#include "pollux_launch.h"
#include "pollux_math.h"
#include "pollux_step.h"

namespace px {

constexpr int kRecipTable = 256;      // 1/K is tabled for K below this

// Result of the sweep for one (job, placement class, K); filled and used only in memoised mode.
struct __align__(16) MemoEntry {
    double goodput;
    int32_t m, s;
};

struct FitnessArgs {
    int P, J, N, Gm, Gs, flags;
    int cand_per_wave, cand_groups;   // pairs kernel: candidates each wavefront walks, groups of 4 * cand_per_wave
    const int32_t *population, *m_grid, *fair_share, *current_alloc, *node_capacity;
    const double *job_params;
    double p, delta;
    // workspace
    int32_t *status;              // the status word; in the 252 bytes behind it, per candidate of a small call, whether it met a negative entry
    double *rs, *rk, *lntg, *pu, *qh5, *ql5, *lt, *denom, *factor, *G;
    float *rsf;                   // 1/(s+1) in fp32, as long as rs
    double2 *tg;                  // [J,Gm] (T_grad, 1 / T_grad)
    double2 *ca;                  // [J,2,kTableK,Gm] (C, A0) of the sweep per (job, one node?, K, grid point) (see prepare_kernel)
    int32_t *srange;              // [J,kTableK,Gm] feasible accumulation counts per (job, K, grid point) (see prepare_kernel)
    int32_t *k1;                  // one word: the rows of the "one node" class are tabled for K <= *k1 only (prepare_kernel)
    int gs_pad;                   // Gs rounded up to a multiple of 32: length of rs
    int32_t *jobstat;             // [J] status bits of each job (prepare_kernel), OR-ed into the status word by the call's last kernel
    int32_t *meta;
    MemoEntry *memo;              // [J,2,kTableK] best point per (job, one node?, K), memoised mode only
    unsigned long long *curmask;  // [J] rows of at most 256 entries: bit g set when one of entries 4 g .. 4 g + 3 of the job's
                                  // current row is not zero (prepare_kernel)
    int32_t *zeros;               // 64 zero bytes (prepare_kernel): what lanes read where the current row holds nothing
    unsigned long long *colpack;  // [P,N] per node: GPUs asked (low 40 bits, signed) + multi-node jobs present << 40
    int need_constraints;
    int stage_rows;               // pairs_kernel: table rows that several pairs read are copied to LDS (see stage_candidates)
    const int32_t *sel;           // candidates to evaluate (device list of n_sel indices into the population), or null: all P
    int n_sel;
    // row inheritance (pollux_generation with PX_GA_INHERIT_ROWS; written by the search step, see GaArgs)
    const int32_t *src_row;       // [n_sel, J] the candidate whose row j the listed child holds unchanged, or -1
    const int32_t *odd;           // [n_sel] the listed child is to be evaluated in full
    int32_t *dirty_count, *dirty; // rows to sweep, per job: their number [J] and the candidates they belong to [J, n_sel]
    int or_job_status;            // this call's prepare_kernel has left per-job status bits: its last kernel ORs them into the status word
    int clear_counters;           // prepare_kernel clears colpack (fitness calls whose population pass keeps the counters in memory)
    // outputs
    double *fitness, *best_goodput, *speedup;
    int32_t *best_m, *best_s, *violations;
};

constexpr unsigned long long kPackJob = 1ull << 40;   // one multi-node job in a colpack word
constexpr int kNearRecips = 256;          // pairs kernel: reciprocals kept in LDS when Gs (rounded up to 32) is at most this
// The fp64 table in LDS (in doubles): per count s the pair (1 / (s + 1), s), so that one read brings both operands of
// w(s) = s + C / (s + 1) at an end of the feasible counts; behind the pairs the thresholds U[t] = t (t + 1).
constexpr int kNearU = 2 * kNearRecips;
// pairs kernel: the table rows (one per (placement class, K)) that most of a workgroup's pairs read are staged in LDS,
// behind the reciprocals and thresholds: (T_grad, 1 / T_grad) per batch size as in memory, then per row the (C, A0)
// pairs and the feasible ranges.  16-byte entries throughout, so that a lane's addresses are its number times 16
// (or times 4 for the ranges) plus a uniform offset, as they are for the tables in memory.
constexpr int kStageGm = 128;             // staged rows hold grids of at most this many batch sizes
constexpr int kStageRows = 4;             // rows staged at most (16.6 KB of LDS per workgroup with the rest: eight workgroups per CU)
// Candidates per wavefront from which staging pays for its two barriers; the children of a generation resemble each other, so more
// of their pairs share a row.  Kept calls on 128 nodes, us without, with: 50 x 16, 200 candidates of 100 jobs (one each) 23.0, 25.4;
// 500 of 200 (four each) 46.5, 48.1; 100 x 8, 1000 of 200 (eight each) 83.4, 80.9; its 500 children (four each) 89.5, 86.4.
constexpr int stage_candidates(bool children) { return children ? 4 : 5; }
constexpr int kStageRowDoubles = 2 * kStageGm + kStageGm / 2;
constexpr int kStageBase = kNearU + kNearRecips + 8;
constexpr int kStageDoubles = 2 * kStageGm + kStageRows * kStageRowDoubles;
constexpr int kPending = -2;             // pairs kernel: grid index of a row whose sweep is still to be done
constexpr int kClose = -4;               // grid index of a sweep whose scan cannot tell the best batch sizes apart (elect_scanned)
constexpr int kMetaChanged = 1 << 30;   // meta[pair] = nodes | (row differs from current ? kMetaChanged : 0)

// Parameters of one job (uniform across the wavefront).  The sweep itself needs only
// phi and a = phi + M0; the synchronisation parameters are read where T_sync is formed.
struct Job {
    const double *__restrict__ jp;   // job_params
    int J, j;
    double phi, a;
};

struct SyncParams {
    double alpha_sl, beta_sl, alpha_sn, beta_sn, gamma, inv_gamma;
};

__device__ __forceinline__ Job load_job(const double *__restrict__ jp, int J, int j)
{
    Job q;
    q.jp = jp; q.J = J; q.j = j;
    q.phi = jp[(size_t)PX_PHI * J + j];
    q.a = q.phi + jp[(size_t)PX_M0 * J + j];
    return q;
}

__device__ __forceinline__ SyncParams load_sync(const Job &q)
{
    SyncParams y;
    y.alpha_sl = q.jp[(size_t)PX_ALPHA_SL * q.J + q.j];
    y.beta_sl = q.jp[(size_t)PX_BETA_SL * q.J + q.j];
    y.alpha_sn = q.jp[(size_t)PX_ALPHA_SN * q.J + q.j];
    y.beta_sn = q.jp[(size_t)PX_BETA_SN * q.J + q.j];
    y.gamma = q.jp[(size_t)PX_GAMMA * q.J + q.j];
    y.inv_gamma = 1.0 / y.gamma;
    return y;
}

// ---- one batch size of a job's grid -------------------------------------------------
//   tg, rtg = T_grad(m) (Eq. 8) and its reciprocal     lntg = ln T_grad(m)
//   pu      = phi / m                      (u = phi / (K m) = pu / K)
//   qh5     = floor(M_max / m) + 1/2       ql5 = ceil(M0 / m) - 1/2
// M0 <= K m (s+1) <= M_max holds exactly when ceil(M0/m) <= K (s+1) <= floor(M_max/m),
// i.e. for s between trunc(ql5 / K) and trunc(qh5 / K) - 1; the halves keep the
// quotients at least 1/(2K) away from an integer, so a rounded 1/K cannot move them
// across one.
struct GridPoint {
    double tg, rtg, lntg, pu, qh5, ql5;
};

struct GridParams {
    double alpha_g, beta_g, phi, M0, Mmax;
};

__device__ __forceinline__ GridParams load_grid_params(const double *__restrict__ jp, int J, int j)
{
    return GridParams{jp[(size_t)PX_ALPHA_G * J + j], jp[(size_t)PX_BETA_G * J + j], jp[(size_t)PX_PHI * J + j],
                      jp[(size_t)PX_M0 * J + j], jp[(size_t)PX_MMAX * J + j]};
}

__device__ __forceinline__ GridPoint grid_point(const Coefs &c, const GridParams &q, int mi)
{
    GridPoint g;
    const double m = (double)mi;
    g.tg = q.alpha_g + q.beta_g * m;                     // Eq. 8
    g.rtg = g.tg > 0.0 ? 1.0 / g.tg : 0.0;
    g.lntg = px_log(c, g.tg);
    double qh = -1.5, ql = 1.0;
    if (mi > 0) {
        qh = floor(px_div(q.Mmax, m));               // (put right below where the quotient has been rounded across an integer)
        if (m * (qh + 1.0) <= q.Mmax) qh += 1.0;
        if (m * qh > q.Mmax) qh -= 1.0;
        ql = ceil(px_div(q.M0, m));
        if (m * (ql - 1.0) >= q.M0) ql -= 1.0;
        if (m * ql < q.M0) ql += 1.0;
        if (!(ql >= 1.0)) ql = 1.0;
        if (!(qh >= 0.0)) qh = -1.5;
    }
    g.pu = mi > 0 ? px_div(q.phi, m) : 0.0;
    g.qh5 = qh + 0.5;
    g.ql5 = ql - 0.5;
    return g;
}

// ---- T_sync and the last pass of Eq. 10 ------------------------------------------

// Eq. 9: no synchronisation for one GPU, the "local" pair on one node, the "node" pair otherwise.
__device__ __forceinline__ double t_sync(const SyncParams &y, int K, bool one_node)
{
    if (K <= 1) return 0.0;
    return one_node ? y.alpha_sl + y.beta_sl * (double)(K - 2) : y.alpha_sn + y.beta_sn * (double)(K - 2);
}

struct SyncTerm {
    double ts, lnts, gamma, inv_gamma;
    int mode;           // 0: T_sync = 0 (last pass = T_grad); 1: gamma = 1 (plain sum); 2: general
};

__device__ __forceinline__ SyncTerm sync_term(const Coefs &c, const SyncParams &y, int K, bool one_node)
{
    SyncTerm t;
    t.ts = t_sync(y, K, one_node);
    t.gamma = y.gamma;
    t.inv_gamma = y.inv_gamma;
    t.mode = (t.ts == 0.0) ? 0 : (y.gamma == 1.0 ? 1 : 2);
    t.lnts = (t.mode == 2) ? px_log(c, t.ts) : 0.0;
    return t;
}

__device__ __forceinline__ SyncTerm sync_term(const Job &q, int K, bool one_node) { return sync_term(plain_coefs(), load_sync(q), K, one_node); }

__device__ __forceinline__ double last_pass(const Coefs &c, const SyncTerm &t, double tg, double lntg)
{
    if (t.mode == 0) return tg;
    if (t.mode == 1) return tg + t.ts;
    const double e = px_exp(c, -t.gamma * fabs(lntg - t.lnts));
    return fmax(tg, t.ts) * px_exp(c, px_log1p_unit(c, e) * t.inv_gamma);
}

__device__ __forceinline__ double last_pass(const SyncTerm &t, double tg, double lntg) { return last_pass(plain_coefs(), t, tg, lntg); }

// The feasible accumulation counts of grid point i with K GPUs: s_lo <= s <= s_hi
// (empty when s_lo > s_hi), from the half-offset quotients of grid_point.
__device__ __forceinline__ void feasible_range(double ql5, double qh5, double rK, int Gs, int &s_lo, int &s_hi)
{
    s_lo = (int)(ql5 * rK);
    s_hi = (int)(qh5 * rK) - 1;
    s_hi = s_hi < Gs - 1 ? s_hi : Gs - 1;
}

// Whether the tables hold the row of (K, class): K = 1 .. kTableK for several nodes, 1 .. k1 for one node.
__device__ __forceinline__ bool tabled_row(int K, bool one_node, int k1)
{
    return K <= (one_node ? k1 : kTableK);
}

__device__ __forceinline__ double wave_read(double v, int src)
{
    return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), src), __builtin_amdgcn_readlane(__double2loint(v), src));
}

// ---- the sweep of one (job, K, nodes) ----------------------------------------

struct Best {
    double goodput;   // maximum of Eq. 4 over the grid, 0 if nothing is feasible
    int m, s;         // batch size and accumulation steps attaining it, -1/-1 if none
};

struct JobTables {
    const int32_t *__restrict__ m;
    const double2 *__restrict__ tg;   // (T_grad, 1 / T_grad)
    const double *__restrict__ lntg, *__restrict__ pu, *__restrict__ qh5, *__restrict__ ql5;
    const double *__restrict__ lt;    // rows of this job in the last-pass table
    const double2 *__restrict__ ca;   // rows of this job in the table of (C, A0)
    const int32_t *__restrict__ srange;   // feasible accumulation counts of this job, [kTableK, Gm]
    int k1;                               // rows of the "one node" class are tabled for K <= k1
};

// Wave-wide argmax of non-negative goodput values g (0 = the lane has no point): positive
// doubles order like their bit patterns, so the maximum is found as two unsigned 32-bit
// reductions (high words, then low words among the lanes that hold the highest high word),
// and ties go to the lowest flat index.  Every lane returns the same result.
__device__ __forceinline__ Best wave_argmax(double g, int flat, int m, int s)
{
    g = g > 0.0 ? g : 0.0;                                        // also drops a NaN
    const unsigned hi = (unsigned)__double2hiint(g), lo = (unsigned)__double2loint(g);
    const unsigned hmax = wave_max(hi);
    const unsigned lmax = wave_max(hi == hmax ? lo : 0u);
    if ((hmax | lmax) == 0u) return Best{0.0, -1, -1};
    const bool top = hi == hmax && lo == lmax;
    const int fmin_ = wave_min(top ? flat : 0x7FFFFFFF);
    const uint64_t wmask = __ballot(top && flat == fmin_);
    const int wl = __builtin_amdgcn_readfirstlane(__ffsll((unsigned long long)wmask) - 1);
    Best out;
    out.goodput = __hiloint2double((int)__builtin_amdgcn_readfirstlane((int)hmax), (int)__builtin_amdgcn_readfirstlane((int)lmax));
    out.m = __builtin_amdgcn_readlane(m, wl);
    out.s = __builtin_amdgcn_readlane(s, wl);
    return out;
}

// Eq. 4 at one grid point, in the paper's order of operations (no contraction).
__device__ __forceinline__ double goodput_point(const Job &q, double Km, double tg, double last, int s)
{
    const double M = Km * (double)(s + 1);
    const double t_iter = (double)s * tg + last;                 // Eq. 11
    const double throughput = M / t_iter;                        // Eq. 7
    const double efficiency = q.a / (q.phi + M);                 // Eq. 6
    return throughput * efficiency;                              // Eq. 4
}

// ---- the sweep of one batch size per lane over CH accumulation counts ---------------
// With C = B0 / T_grad the quantity to minimise is  h = A0 + T_grad w(s),  w(s) = s + C / (s+1),
// for the lane's batch size.  The lane takes the smallest w over all accumulation counts, feasible or not;
// C >= 0 makes w convex in s, and the feasible counts of a batch size form an interval (tabled
// per (job, K, i) by prepare_kernel), so the smallest feasible w is that minimum, or w at the end of the
// interval that lies towards it (Feasible below).  Inside a chunk of CH counts, per group of four
// positions b = 4 G .. 4 G + 3 and lane:
//   w_b  = C * r + (b mod 16)  one v_fma_f64 each (v_mul_f64 for 0): r = 1/(s0 + b + 1) from scalar
//                              registers, the addend an inline constant (1, 2, 4) or one of
//                              twelve register pairs that hold 3, 5, 6, .. 15 for the whole kernel
//   wmin = min(wmin, the four) four v_min_f64
// eight VALU instructions per four points; the reciprocals arrive through the scalar cache.  Each run of sixteen
// positions has a minimum of its own (values relative to the run's first position); the runs are merged after
// the chunk.  Which count attains the minimum is not looked for here: one lane of sixty-four wins the election, and
// its count follows from C when the elected point is priced (px_best_count).
// (With every group of four carrying its position in its low mantissa bits, nine instructions per four points, and every lane
// finding its count with five comparisons, a pair of 128 batch sizes x 32 counts took 248 vector instructions, 213 so: 4096 candidates
// of 1000 jobs 1.78 ms against 1.66, 1000 of 200 on 64 nodes 52.5 us against 46; fp32, which also loses its tags, 52.0 against 44.7.)
typedef const double __attribute__((address_space(4))) *ScalarDoubles;
typedef const double __attribute__((address_space(3))) *LdsDoubles;
typedef double Double2 __attribute__((ext_vector_type(2)));

constexpr int kRun = 16;
constexpr int runs_of(int CH) { return (CH + kRun - 1) / kRun; }

// The addends that are not inline constants (3, 5 .. 15) in vector registers.  Made once
// per kernel through an opaque statement, so that they stay in registers instead of being formed
// again at every use.
struct RunSteps {
    double x[kRun];
};

__device__ __forceinline__ RunSteps make_run_steps()
{
    RunSteps X;
#pragma unroll
    for (int t = 0; t < kRun; ++t) X.x[t] = (double)t;
    asm volatile("" : "+v"(X.x[3]), "+v"(X.x[5]), "+v"(X.x[6]), "+v"(X.x[7]), "+v"(X.x[8]), "+v"(X.x[9]), "+v"(X.x[10]),
                      "+v"(X.x[11]), "+v"(X.x[12]), "+v"(X.x[13]), "+v"(X.x[14]), "+v"(X.x[15]));
    return X;
}

// w at position B of a chunk, relative to the first position of its run.
template <int B>
__device__ __forceinline__ double point_w(double C, double r, const RunSteps &X)
{
    constexpr int t = B % kRun;
    double g;
    if constexpr (t == 0) asm("v_mul_f64 %0, %1, %2" : "=v"(g) : "v"(C), "s"(r));
    else if constexpr (t == 1) asm("v_fma_f64 %0, %1, %2, 1.0" : "=v"(g) : "v"(C), "s"(r));
    else if constexpr (t == 2) asm("v_fma_f64 %0, %1, %2, 2.0" : "=v"(g) : "v"(C), "s"(r));
    else if constexpr (t == 4) asm("v_fma_f64 %0, %1, %2, 4.0" : "=v"(g) : "v"(C), "s"(r));
    else asm("v_fma_f64 %0, %1, %2, %3" : "=v"(g) : "v"(C), "s"(r), "v"(X.x[t]));
    return g;
}

// Four points at positions 4 G .. 4 G + 3 of the chunk (G a compile-time group index): the
// four values and their minimum.  The volatile statements keep their order, so the
// reciprocals of a group are requested after the previous group's work and only one group's
// operands occupy scalar registers.
struct GroupRecips {
    double r0, r1, r2, r3;
};

template <int G>
__device__ __forceinline__ GroupRecips load_group(ScalarDoubles &rs)
{
    asm volatile("" : "+s"(rs));
    return GroupRecips{rs[4 * G + 0], rs[4 * G + 1], rs[4 * G + 2], rs[4 * G + 3]};
}

template <int CH, int G, int NC>
__device__ __forceinline__ void scan_group(double (&wmin)[NC][runs_of(CH)], const double (&C)[NC], const RunSteps &X, const GroupRecips &o)
{
#pragma unroll
    for (int n = 0; n < NC; ++n) {
        const double w0 = point_w<4 * G + 0>(C[n], o.r0, X);
        const double w1 = point_w<4 * G + 1>(C[n], o.r1, X);
        const double w2 = point_w<4 * G + 2>(C[n], o.r2, X);
        const double w3 = point_w<4 * G + 3>(C[n], o.r3, X);
        double &run = wmin[n][4 * G / kRun];
        double g, g2;
        if constexpr ((4 * G) % kRun == 0) {          // the first group of a run starts its minimum
            asm volatile("v_min_f64 %0, %2, %3\n\t"
                         "v_min_f64 %1, %4, %5\n\t"
                         "v_min_f64 %0, %0, %1"
                         : "=&v"(run), "=&v"(g)
                         : "v"(w0), "v"(w1), "v"(w2), "v"(w3));
        } else {
            asm volatile("v_min_f64 %1, %3, %4\n\t"
                         "v_min_f64 %2, %5, %6\n\t"
                         "v_min_f64 %0, %0, %1\n\t"
                         "v_min_f64 %0, %0, %2"
                         : "+v"(run), "=&v"(g), "=&v"(g2)
                         : "v"(w0), "v"(w1), "v"(w2), "v"(w3));
        }
    }
}

// The reciprocals of a group are requested one group ahead of their use.
template <int CH, int NC, int G = 0>
__device__ __forceinline__ void scan_groups(double (&wmin)[NC][runs_of(CH)], const double (&C)[NC], const RunSteps &X, ScalarDoubles &rs,
                                            GroupRecips cur)
{
    if constexpr (4 * G < CH) {
        asm volatile("" : "+s"(cur.r0), "+s"(cur.r1), "+s"(cur.r2), "+s"(cur.r3));
        GroupRecips next = cur;
        if constexpr (4 * (G + 1) < CH) next = load_group<G + 1>(rs);
        scan_group<CH, G, NC>(wmin, C, X, cur);
        scan_groups<CH, NC, G + 1>(wmin, C, X, rs, next);
    }
}

__device__ __forceinline__ double min_f64(double a, double b)
{
    double out;                                        // (the bare instruction: the operands are results of arithmetic)
    asm("v_min_f64 %0, %1, %2" : "=v"(out) : "v"(a), "v"(b));
    return out;
}

// CH points starting at accumulation count s0; rs points at s0.  out: the smallest w over the chunk, relative to s0.
template <int CH, int NC>
__device__ __forceinline__ void scan_chunk(double (&out)[NC], const double (&C)[NC], const RunSteps &X, ScalarDoubles rs)
{
    static_assert(CH == 8 || CH == 16 || CH == 24 || CH == 32, "one or two runs");
    double wmin[NC][runs_of(CH)];
    scan_groups<CH, NC>(wmin, C, X, rs, load_group<0>(rs));
#pragma unroll
    for (int n = 0; n < NC; ++n) {
        out[n] = wmin[n][0];
        if constexpr (runs_of(CH) == 2) {
            static_assert(kRun == 16, "the offset of the second run is a product of inline constants");
            double moved;
            asm("v_fma_f64 %0, 4.0, 4.0, %1" : "=v"(moved) : "v"(wmin[n][1]));
            out[n] = min_f64(out[n], moved);
        }
    }
}

// The same chunk for a GPU count beyond the tables, written as a plain loop (rare, so
// compactness counts more than speed): the lane's feasible positions are first..last.
template <int CH>
__device__ __forceinline__ double sweep_chunk_plain(double tg, double A0s, double B0, const double *__restrict__ rs,
                                                    int first, int last)
{
    double kmin = __builtin_inf();
#pragma unroll 1
    for (int b = 0; b < CH; ++b) {
        const double h = px_fma(B0, rs[b], px_fma((double)b, tg, A0s));
        const double key = __hiloint2double(__double2hiint(h), (__double2loint(h) & ~31) | b);
        if (first <= b && b <= last && key < kmin) kmin = key;
    }
    return kmin;
}

// The smallest w(s) = s + C / (s + 1) over s = 0, 1, ... (all counts of the grid, rounded up to whole chunks: the reciprocals
// are padded), for NC values C >= 0 of each lane, which share the reciprocals.
template <int CH, int NC>
__device__ __forceinline__ void scan_mins(double (&wmin)[NC], const double (&C)[NC], const RunSteps &X, ScalarDoubles rsc, int Gs)
{
    scan_chunk<CH, NC>(wmin, C, X, rsc);
    // (the bound goes through an opaque statement: every inlined copy of this loop then tests it with a scalar
    // comparison of its own, instead of sharing one truth value that the compiler carries around as a lane mask and
    // negates with two vector instructions)
    asm volatile("" : "+s"(Gs));
    for (int s0 = CH; s0 < Gs; s0 += CH) {
        double w[NC];
        scan_chunk<CH, NC>(w, C, X, rsc + s0);
#pragma unroll
        for (int n = 0; n < NC; ++n) wmin[n] = min_f64(wmin[n], w[n] + (double)s0);
    }
}

template <int CH>
__device__ __forceinline__ double scan_min(double C, const RunSteps &X, ScalarDoubles rsc, int Gs)
{
    const double Cs[1] = {C};
    double wmin[1];
    scan_mins<CH, 1>(wmin, Cs, X, rsc, Gs);
    return wmin[0];
}

// ---- the feasible counts of a batch size --------------------------------------------
// w(s+1) < w(s) precisely when C > (s+1)(s+2), both sides exact in fp64.  With U[t] = t (t+1) the argmin of w over all counts
// therefore lies below the feasible ones s_lo .. s_hi precisely when C <= U[s_lo] (for s_lo = 0 that is C = 0, where w(0) is the
// minimum anyway), and beyond them precisely when C > U[s_hi + 1]; the smallest feasible w is then w(s_lo) or w(s_hi), and the
// minimum over all counts else.  None of this waits for the scan.
struct Feasible {
    int outside;        // the argmin over all counts is not feasible
    double w;           // w at the end of the interval towards it
};

// bounds: s_lo | s_hi << 16.  near: pairs (1 / (s + 1), s) in LDS with the U[t] behind them.
__device__ __forceinline__ Feasible feasible_end(double C, int bounds, LdsDoubles near)
{
    const int s_lo = bounds & 0xFFFF, s_hi = bounds >> 16;
    const bool above = C > near[kNearU + 1 + s_hi];
    const Double2 rc = *(const Double2 __attribute__((address_space(3))) *)(near + 2 * (above ? s_hi : s_lo));
    return Feasible{(int)above | (int)(C <= near[kNearU + s_lo]), px_fma(C, rc.x, rc.y)};
}

// The same without a table of thresholds; recip(s, (double)s): 1 / (s + 1).
template <typename RECIP>
__device__ __forceinline__ Feasible feasible_end(double C, int s_lo, int s_hi, const RECIP &recip)
{
    const double lo = (double)s_lo, hi = (double)s_hi;
    const bool above = C > px_fma(hi, hi, px_fma(3.0, hi, 2.0));
    const int s = above ? s_hi : s_lo;
    const double sd = above ? hi : lo;
    return Feasible{(int)above | (int)(C <= px_fma(lo, lo, lo)), px_fma(C, recip(s, sd), sd)};
}

// The grid point a sweep elects: index into the job's batch-size grid and accumulation
// count; i = -1 when no point is feasible.
struct Pick {
    int i, s;
};

// The lanes' smallest h and where each found it (accumulation count | index of its group of 64 batch sizes << 16; bit l of
// `second` adds one to lane l's group index): the point with the smallest h over the wavefront, equal values to the lowest
// flat index i * Gs + s.  Every lane returns the same result.
__device__ __forceinline__ Pick elect(double kbest, int where, unsigned long long second, int Gs)
{
    const int lane = lane_id();
    // positive doubles order like their bit patterns: unsigned 32-bit wave minima, high words first;
    // the low words only among several lanes that share the smallest high word
    const unsigned hi = (unsigned)__double2hiint(kbest), lo = (unsigned)__double2loint(kbest);
    const unsigned hmin = wave_min(hi);
    if (hmin >= 0x7FF00000u) return Pick{-1, -1};              // every lane still holds +inf
    unsigned long long winners = __builtin_amdgcn_ballot_w64(hi == hmin);
    if (winners & (winners - 1)) {
        const unsigned lmin = wave_min(hi == hmin ? lo : 0xFFFFFFFFu);
        winners &= __builtin_amdgcn_ballot_w64(lo == lmin);
        if (winners & (winners - 1)) {
            // equal values (duplicated batch sizes): the lowest flat index i * Gs + s.  Winners with one
            // group of 64 and one count differ in the lane only, so the lowest lane has it; else a third minimum.
            where |= (int)((second >> lane) & 1ull) << 16;
            const int first_lane = __ffsll(winners) - 1;
            const int where0 = __builtin_amdgcn_readlane(where, first_lane);
            const unsigned long long same = __builtin_amdgcn_ballot_w64(where == where0);
            if ((winners & ~same) != 0) {
                const bool top = ((winners >> lane) & 1ull) != 0;
                const int flat = ((where >> 16) * kWave + lane) * Gs + (where & 0xFFFF);
                const int first = wave_min(top ? flat : 0x7FFFFFFF);
                winners &= __builtin_amdgcn_ballot_w64(flat == first);
            }
        }
    }
    const int wl = __ffsll(winners) - 1;
    const int wwhere = __builtin_amdgcn_readlane(where, wl);
    return Pick{((wwhere >> 16) | (int)((second >> wl) & 1ull)) * kWave + wl, wwhere & 0xFFFF};
}

// ---- elections between values of the scan ----------------------------------------------
// What elects a batch size is its h = fma(T_grad, fma(C, 1 / (s + 1), s), A0) at its best feasible count s: rounding decides between batch
// sizes whose h agree to the last places, so every way to an argmax (sweeps, memoised rows, fair shares, queries) forms it so.  The
// scan's minimum may differ from that w in the last places: beyond 16 counts it is rounded once more for each offset, and next to a
// threshold it may be a neighbour's.  That is less than 2^-49 of h, so the scan's values elect where the smallest is alone within
// one unit of its high word (2^-20 of itself); where another is as close (one election in 6000 on the timing cases' grids, nearly
// all where alpha_grad = 0 and gamma = 1 make h a function of m (s + 1)), h itself decides (settle).  1000 candidates of 200 jobs on
// 64 nodes, 64 x 16, us: 61.1 without this, 60.7 so; 80 where every election of every job is settled.
// In single precision the scan's h has five roundings where h itself has four, so two of them can change places within ten units in the
// last place; sixteen are close.  1000 candidates of 200 jobs on 64 nodes, 64 x 16, us: 62.8 without this, 63.8 so.
// Positive values order like their bit patterns: the election sees high words of doubles, all bits of single ones.
template <typename REAL>
struct Closeness;

template <>
struct Closeness<double> {
    static constexpr unsigned kWindow = 1u, kInf = 0x7FF00000u;
    static __device__ __forceinline__ unsigned bits(double h) { return (unsigned)__double2hiint(h); }
};

template <>
struct Closeness<float> {
    static constexpr unsigned kWindow = 16u, kInf = 0x7F800000u;
    static __device__ __forceinline__ unsigned bits(float h) { return (unsigned)__float_as_int(h); }
};

template <typename REAL>
__device__ __forceinline__ bool close_to(REAL a, REAL b)
{
    unsigned d;
    asm("v_sad_u32 %0, %1, %2, 0" : "=v"(d) : "v"(Closeness<REAL>::bits(a)), "v"(Closeness<REAL>::bits(b)));
    return d <= Closeness<REAL>::kWindow;
}

// The second smallest of least <= second and next.
__device__ __forceinline__ unsigned second_smallest(unsigned least, unsigned second, unsigned next)
{
    unsigned v;
    asm("v_med3_u32 %0, %1, %2, %3" : "=v"(v) : "v"(least), "v"(second), "v"(next));
    return v;
}

// The batch size with the smallest of the scan's h over the wavefront, -1 where there is none, kClose where it is not alone.  kbest: the
// lane's smallest; its batch size is the lane's number + first(lane), again: the lanes of which another h is close to it.
// Every lane returns the same result.
template <typename REAL, typename FIRST>
__device__ __forceinline__ int elect_scanned(REAL kbest, unsigned long long again, const FIRST &first)
{
    const unsigned h = Closeness<REAL>::bits(kbest), least = wave_min(h);
    if (least >= Closeness<REAL>::kInf) return -1;             // every lane still holds +inf
    const unsigned long long close = __builtin_amdgcn_ballot_w64(h <= least + Closeness<REAL>::kWindow);
    if ((close & ((close - 1ull) | again)) != 0ull) return kClose;
    const int wl = __builtin_ctzll(close);
    return wl + first(wl);
}

// The same for each row of 16 lanes: its batch size is `where`, runner_up holds the bits of the lane's second smallest h.  One lane a row
// is close to the row's smallest h and no other h of that lane, or no lane of the row has a point.  Else, in double precision, a row's
// lanes are told apart to 2^-46: that costs less than to settle them, two trips to memory at the end of a launch that may last 9 us (40
// candidates of 24 jobs on 16 nodes, 128 x 16, tables kept, 9.5 us without this, 9.0 so).  (In elect_scanned it made the sweep one candidate at
// a time slower, 131 to 135 us for 1021 candidates of 331 jobs on 130 nodes.)
template <typename REAL>
__device__ __forceinline__ int elect_scanned_rows(REAL kbest, unsigned runner_up, int where)
{
    constexpr unsigned kMost = Closeness<REAL>::kInf - 1u;
    const unsigned h = Closeness<REAL>::bits(kbest), least = row16_min(h), most = least + Closeness<REAL>::kWindow;
    const unsigned bound = most < kMost ? most : kMost;
    unsigned long long at = __builtin_amdgcn_ballot_w64(h <= bound);
    const unsigned long long again = __builtin_amdgcn_ballot_w64(runner_up <= bound);
    int first = (int)row16_min(h <= bound ? (unsigned)where : ~0u);
    if (__builtin_expect(16 * __popcll(at) + __popcll(__builtin_amdgcn_ballot_w64(first == -1)) + __popcll(again) != kWave, 0)) {
        int shift = lane_id() & 48;
        asm volatile("" : "+v"(shift));               // (nothing of this is formed before the loop)
        if constexpr (sizeof(REAL) == 8) {
            const unsigned low = row16_min(h == least ? (unsigned)__double2loint(kbest) : ~0u);
            const double smallest = __hiloint2double((int)least, (int)low);
            const bool ties = h <= bound && kbest - smallest <= smallest * 0x1p-46;
            at = __builtin_amdgcn_ballot_w64(ties);
            first = (int)row16_min(ties ? (unsigned)where : ~0u);
        }
        if (__popc((unsigned)(at >> shift) & 0xFFFFu) > 1 || ((unsigned)(again >> shift) & 0xFFFFu) != 0u) first = kClose;
    }
    return first;
}

// The elections of two rows of the tables by h itself, without a scan (two, as each waits for a trip to memory).  All 64 lanes call
// this with the same arguments; picked: the batch sizes, equal values to the lowest.  near: as for sweep_pick, when has_near.
__device__ __forceinline__ void settle(int (&picked)[2], int lane, const JobTables &tb, const double *__restrict__ rs, LdsDoubles near,
                                       bool has_near, int Gm, int Gs, const int (&K)[2], const bool (&one_node)[2])
{
    double kbest[2] = {__builtin_inf(), __builtin_inf()};
    int where[2] = {0, 0};
    for (int i = lane; i < Gm; i += kWave) {
        const double tg = tb.tg[i].x;
        double2 car[2];
        int bounds[2];
#pragma unroll
        for (int n = 0; n < 2; ++n) {
            car[n] = tb.ca[(unsigned)((one_node[n] ? kTableK : 0) + K[n] - 1) * (unsigned)Gm + (unsigned)i];
            bounds[n] = tb.srange[(unsigned)(K[n] - 1) * (unsigned)Gm + (unsigned)i];
        }
#pragma unroll
        for (int n = 0; n < 2; ++n) {
            const int s = px_best_count(car[n].x, bounds[n] & 0xFFFF, bounds[n] >> 16);
            const double key = px_fma(tg, px_fma(car[n].x, has_near ? near[2 * s] : rs[s], (double)s), car[n].y);
            if (key < kbest[n]) {
                kbest[n] = key;
                where[n] = (i / kWave) << 16;
            }
        }
    }
#pragma unroll
    for (int n = 0; n < 2; ++n) picked[n] = elect(kbest[n], where[n], 0ull, Gs).i;
}

// All 64 lanes call this with the same (job, nodes, K within the tables).  Every lane returns the same result: the batch size
// (index into the job's grid) of the feasible point with the smallest h over the whole grid, equal values to the lowest
// index, or -1 when no point is feasible, or kClose.  Its count is found where it is priced (price_tabled).
// WHOLE: the caller has checked that Gm is a multiple of 64, so no lane runs past the grid of batch sizes.
template <int CH, bool WHOLE = false, bool STAGED = false>
__device__ __forceinline__ int sweep_pick(int lane, const JobTables &tb, const RunSteps &X, const double *__restrict__ rs, int Gm, int Gs, int K,
                                          int nodes, LdsDoubles near, bool has_near, int staged_row)
{
    // near: a copy of rs in LDS (quicker to read per lane) when has_near
    // staged_row: where in `near` the terms of this (class, K) are staged (STAGED; see kStageBase), or -1;
    // rows are staged only together with has_near
    K = __builtin_amdgcn_readfirstlane(K);        // the same in every lane (see above): kept in scalar registers
    nodes = __builtin_amdgcn_readfirstlane(nodes);
    const bool one_node = nodes == 1;
    // offsets inside one job's tables fit 32 bits (Gm <= 2^20)
    const double2 *__restrict__ carow = tb.ca + (unsigned)((one_node ? kTableK : 0) + K - 1) * (unsigned)Gm;
    const int32_t *__restrict__ srow = tb.srange + (unsigned)(K - 1) * (unsigned)Gm;

    // where this lane's terms of a staged row start in LDS (bytes from `near`): the (C, A0) pairs, the feasible ranges
    const unsigned at_ca = ((unsigned)lane << 4) + 8u * (unsigned)staged_row;
    const unsigned at_range = ((unsigned)lane << 2) + 8u * (unsigned)(staged_row + 2 * kStageGm);

    double kbest = __builtin_inf();   // smallest h seen by this lane
    int where = 0;                    // the first of its group of 64 batch sizes
    unsigned long long again = 0;     // the lanes of which another h is close to the smallest (elect_scanned)
    unsigned long long second = 0;    // staged terms: the lanes whose best belongs to the second group (no `where`)
    const ScalarDoubles rsc = (ScalarDoubles)rs;
    auto in_memory = [&](int s, double) { return *(const double *)((const char *)rs + 8u * (unsigned)s); };

    // One group of 64 batch sizes starting at i0.  G: the group's index when the terms are staged in LDS (the caller
    // stages only grids of one or two groups, so the index is a compile-time constant and the group's offset goes
    // into the LDS instructions' immediate fields), else -1.
    auto group = [&](const int i0, auto G) __attribute__((always_inline)) {
        constexpr int g = decltype(G)::value;
        const int i = i0 + lane;
        const bool active = WHOLE || i < Gm;
        const int il = active ? i : Gm - 1;
        // a uniform base plus a 32-bit byte offset per lane: the address needs no 64-bit vector arithmetic;
        // the offsets of the 16-byte and the 4-byte entries are one shift-and-add each on the lane number
        // (the opaque statement keeps the two shifted counters on the scalar unit)
        unsigned i16 = (unsigned)i0 << 4, i4 = (unsigned)i0 << 2;
        asm("" : "+s"(i16), "+s"(i4));
        const unsigned at16 = WHOLE ? ((unsigned)lane << 4) + i16 : (unsigned)il * 16u;
        const unsigned at4 = WHOLE ? ((unsigned)lane << 2) + i4 : (unsigned)il * 4u;
        double tg, C, A0;                        // A0 = +inf when the batch size has no feasible count
        int bounds;
        if constexpr (g >= 0) {
            // the row's offset is added to the lane's once per call; the group's is a constant
            typedef const char __attribute__((address_space(3))) *LdsBytes;
            const Double2 car = *(const Double2 __attribute__((address_space(3))) *)((LdsBytes)near + at_ca + 16 * kWave * g);
            C = car.x;
            A0 = car.y;
            tg = *(LdsDoubles)((LdsBytes)near + ((unsigned)lane << 4) + (8 * kStageBase + 16 * kWave * g));
            bounds = *(const int __attribute__((address_space(3))) *)((LdsBytes)near + at_range + 4 * kWave * g);
        } else {
            tg = *(const double *)((const char *)tb.tg + at16);
            const double2 car = *(const double2 *)((const char *)carow + at16);
            C = car.x;
            A0 = car.y;
            bounds = *(const int32_t *)((const char *)srow + at4);
        }
        // (rows are staged only in a workgroup that also keeps the table of reciprocals and thresholds in LDS)
        const double wmin = scan_min<CH>(C, X, rsc, Gs);
        const Feasible f = g >= 0 || has_near ? feasible_end(C, bounds, near) : feasible_end(C, bounds & 0xFFFF, bounds >> 16, in_memory);
        const double key = px_fma(tg, f.outside ? f.w : wmin, A0);
        if constexpr (g == 0) {
            // the first group starts the lane's minimum (a batch size without a feasible count has h = +inf)
            kbest = key;
        } else if constexpr (g == 1) {
            // which lanes hold a batch size of the second group stays a lane mask in scalar registers
            // (the smaller of a number and a NaN, where T_grad overflows, is the number)
            const double least = min_f64(kbest, key);
            second = __builtin_amdgcn_ballot_w64(least != kbest);
            again = __builtin_amdgcn_ballot_w64(close_to(kbest, key));
            kbest = least;
        } else {
            const bool better = active && key < kbest;
            again = (again & ~__builtin_amdgcn_ballot_w64(better)) | __builtin_amdgcn_ballot_w64(active && close_to(kbest, key));
            if (better) {
                kbest = key;
                where = i0;
            }
        }
    };
    if (STAGED && staged_row >= 0) {
        group(0, std::integral_constant<int, 0>());
        if (Gm > kWave) group(kWave, std::integral_constant<int, 1>());
        return elect_scanned(kbest, again, [&](int l) { return (int)((second >> l) & 1ull) * kWave; });
    }
    // the counter of this loop is advanced on the scalar unit (it would otherwise be copied to a vector register)
    for (int i0 = 0; i0 < Gm;) {
        group(i0, std::integral_constant<int, -1>());
        asm volatile("s_add_i32 %0, %0, 64" : "+s"(i0) : : "scc");
    }
    return elect_scanned(kbest, again, [&](int l) { return __builtin_amdgcn_readlane(where, l); });
}

// The sweep of a row the tables do not hold, by a plain loop over the feasible counts of each batch size; it returns the
// elected point.  rs, rk: 1 / (s + 1), 1 / K.
template <int CH>
__device__ __forceinline__ Pick sweep_pick_beyond(const Job &q, const JobTables &tb, const double *__restrict__ rs, const double *__restrict__ rk,
                                                  int Gm, int Gs, int K, int nodes)
{
    const int lane = lane_id();
    K = __builtin_amdgcn_readfirstlane(K);
    nodes = __builtin_amdgcn_readfirstlane(nodes);
    // 1/K arrives through the scalar cache
    const double rK = K < kRecipTable ? ((ScalarDoubles)rk)[K] : 1.0 / (double)K;
    const SyncTerm st = sync_term(q, K, nodes == 1);
    double kbest = __builtin_inf();   // smallest h seen by this lane
    int where = 0;                    // its accumulation count | (index of its group of 64 batch sizes) << 16
    for (int i0 = 0; i0 < Gm; i0 += kWave) {
        const int i = i0 + lane;
        const bool active = i < Gm;
        const int il = active ? i : Gm - 1;
        const double2 tgr = tb.tg[il];
        const double tg = tgr.x;
        const double last = last_pass(st, tg, tb.lntg[il]);
        const double u = tb.pu[il] * rK;
        const double A0 = px_fma(u, tg, last);
        const double B0 = (last - tg) * u;
        int s_lo = 1, s_hi = 0, s_c = 0;
        feasible_range(tb.ql5[il], tb.qh5[il], rK, Gs, s_lo, s_hi);
        if (!active) s_hi = -1;
        double key = __builtin_inf();    // h of this batch size at its best feasible count s_c
        for (int s0 = 0; s0 < Gs; s0 += CH) {
            const double A0s = s0 == 0 ? A0 : px_fma((double)s0, tg, A0);
            const double kmin = sweep_chunk_plain<CH>(tg, A0s, B0, rs + s0, s_lo - s0, s_hi - s0);
            if (kmin < key) {
                key = kmin;
                s_c = s0 + (__double2loint(kmin) & 31);
            }
        }
        if (key < __builtin_inf()) {
            // the plain loop's keys carry the count in their low bits: the exact order of neighbours inside the feasible
            // counts, and the key again without index bits
            const double C = B0 * tgr.y, sd = (double)s_c;
            const double t_lo = px_fma(sd, sd, sd), t_hi = px_fma(sd, sd, px_fma(3.0, sd, 2.0));
            if (s_c > s_lo && C <= t_lo) s_c -= 1;
            else if (s_c < s_hi && C > t_hi) s_c += 1;
            key = px_fma(B0, rs[s_c], px_fma((double)s_c, tg, A0));
            if (key < kbest) {
                kbest = key;
                where = s_c | ((i0 / kWave) << 16);
            }
        }
    }
    return elect(kbest, where, 0ull, Gs);
}

// The same election for four (job, K, nodes) at once, one per row of 16 lanes, for small grids, where a sweep per
// wavefront spends more on its cross-lane steps than on the grid: every row of 16 lanes calls this with its own
// K (1 .. kTableK) and its own one_node (the same in all 16 lanes of a row; the job is the same for the whole
// wavefront), lane l of a row takes batch sizes l, l + 16, ..., and every lane of a row returns the row's
// result: the batch size of the feasible point with the smallest h, -1 when the row has no feasible point, or
// kClose (elect_scanned).
template <int CH, bool WHOLE>
__device__ __forceinline__ int sweep_pick_rows(const JobTables &tb, const RunSteps &X, const double *__restrict__ rs,
                                               int Gm, int Gs, int K, bool one_node, LdsDoubles near, bool has_near)
{
    const int l16 = lane_id() & 15;
    // Byte offsets inside one job's tables fit 32 bits (Gm <= 2^20, 2 * kTableK rows of 16 bytes per batch size): a
    // uniform base plus a 32-bit offset per lane, so that no address needs 64-bit vector arithmetic.
    const unsigned ca_row = (unsigned)((one_node ? kTableK : 0) + K - 1) * (unsigned)Gm * 16u;
    const unsigned s_row = (unsigned)(K - 1) * (unsigned)Gm * 4u;
    double kbest = __builtin_inf();   // smallest h seen by this lane
    unsigned runner_up = ~0u;         // the bits of the second smallest (elect_scanned_rows)
    int where = 0;                    // its batch size
    const ScalarDoubles rsc = (ScalarDoubles)rs;
    auto in_memory = [&](int s, double) { return *(const double *)((const char *)rs + 8u * (unsigned)s); };
    // NC sets of 16 batch sizes from i0 on: their terms are asked for together and share the reciprocals of the scan.
    auto sets = [&](const int i0, auto COUNT) __attribute__((always_inline)) {
        constexpr int NC = decltype(COUNT)::value;
        double tg[NC], A0[NC], C[NC], wmin[NC];
        int bounds[NC];
#pragma unroll
        for (int n = 0; n < NC; ++n) {
            const int i = i0 + 16 * n + l16;
            const unsigned il = (unsigned)(WHOLE || i < Gm ? i : Gm - 1);      // WHOLE: Gm is a multiple of 64, so no lane runs past the grid
            bounds[n] = *(const int32_t *)((const char *)tb.srange + (s_row + 4u * il));
            const double2 car = *(const double2 *)((const char *)tb.ca + (ca_row + 16u * il));
            C[n] = car.x;
            A0[n] = car.y;                          // A0 = +inf when the batch size has no feasible count
            tg[n] = *(const double *)((const char *)tb.tg + 16u * il);
        }
        scan_mins<CH, NC>(wmin, C, X, rsc, Gs);
#pragma unroll
        for (int n = 0; n < NC; ++n) {
            const int i = i0 + 16 * n + l16;
            const Feasible f = has_near ? feasible_end(C[n], bounds[n], near) : feasible_end(C[n], bounds[n] & 0xFFFF, bounds[n] >> 16, in_memory);
            const double key = px_fma(tg[n], f.outside ? f.w : wmin[n], A0[n]);
            const bool active = WHOLE || i < Gm;
            runner_up = second_smallest(Closeness<double>::bits(kbest), runner_up, active ? Closeness<double>::bits(key) : ~0u);
            if (active && key < kbest) {
                kbest = key;
                where = i;
            }
        }
    };
    for (int i0 = 0; i0 < Gm; i0 += 32) {
        if (WHOLE || i0 + 16 < Gm) sets(i0, std::integral_constant<int, 2>());
        else sets(i0, std::integral_constant<int, 1>());
    }
    return elect_scanned_rows(kbest, runner_up, where);
}

// Eq. 4 for batch size i of a tabled row at the count the sweep's minimum has there, in the paper's order of operations.  Arguments
// may differ from lane to lane.
__device__ __forceinline__ Best price_tabled(const Job &q, const JobTables &tb, int Gm, int K, bool one_node, int i)
{
    if (i < 0) return Best{0.0, -1, -1};
    const unsigned row = (unsigned)((one_node ? kTableK : 0) + K - 1) * (unsigned)Gm + (unsigned)i;
    // (all five asked for before the first is waited for)
    const double C = tb.ca[row].x, last = tb.lt[row], tg = tb.tg[i].x;
    const int bounds = tb.srange[(unsigned)(K - 1) * (unsigned)Gm + (unsigned)i], m = tb.m[i];
    const int s = px_best_count(C, bounds & 0xFFFF, bounds >> 16);
    return Best{goodput_point(q, (double)K * (double)m, tg, last, s), m, s};
}

// The same at grid point (i, s) of a row beyond the tables.
__device__ __forceinline__ Best price_beyond(const Job &q, const JobTables &tb, int K, bool one_node, int i, int s)
{
    if (i < 0) return Best{0.0, -1, -1};
    const int m = tb.m[i];
    const double tg = tb.tg[i].x;
    return Best{goodput_point(q, (double)K * (double)m, tg, last_pass(sync_term(q, K, one_node), tg, tb.lntg[i]), s), m, s};
}

__device__ __forceinline__ JobTables job_tables(const FitnessArgs &a, int j)
{
    const size_t o = (size_t)j * a.Gm;
    return JobTables{a.m_grid + o, a.tg + o, a.lntg + o, a.pu + o, a.qh5 + o, a.ql5 + o,
                     a.lt + (size_t)j * 2 * kTableK * a.Gm, a.ca + (size_t)j * 2 * kTableK * a.Gm,
                     a.srange + (size_t)j * kTableK * a.Gm, __builtin_amdgcn_readfirstlane(*a.k1)};
}

// ---- argmax by sampling total batch sizes (Sec. 4.3) -------------------------------
// The grid row of the job holds candidate total batch sizes M_i.  Lane l takes
// i = l, l+64, ...: s is the smallest accumulation count whose per-GPU batch
// m = ceil(M / (K (s+1))) stays within the memory bound, found with integer
// arithmetic; the point is then priced with Eq. 4 in the paper's order of operations
// (T_grad, its logarithm and the last pass of Eq. 10 are formed here, m is not on a grid).
// Gm evaluations per call instead of Gm * Gs.  Ties go to the lowest i.
// LEAN: for pairs_kernel where rows are looked up, in which a row beyond the tables is the exception and spills because of it are not.
template <bool LEAN>
__device__ __forceinline__ Best sweep_sampled(const Coefs &c, const Job &q, const GridParams &gp, const SyncParams &y, double m_mem,
                                              const int32_t *__restrict__ M_list, int Gm, int Gs, int K, int nodes)
{
    if (K <= 0 || !(m_mem >= 1.0 && m_mem <= 2147483647.0)) return Best{0.0, -1, -1};
    const int lane = lane_id();
    // The quotients are found in doubles: the numerators stay below 2^38 wherever the quotient is not one, so that a quotient below
    // an integer is further from it than a rounded one can be off, and its floor is exact.  (200 jobs' rows 0.5 us quicker than with
    // 64-bit integers, which hold ten registers less: LEAN.)
    const double Kd = (double)K;
    const double per_pass = Kd * floor(m_mem);                      // examples one pass over K GPUs can hold
    auto quotient_up = [](double n, double d) {
        if constexpr (LEAN) return (double)(((long long)n + ((long long)d - 1)) / (long long)d);
        else return floor(px_div(n + (d - 1.0), d));
    };
    const SyncTerm st = sync_term(c, y, K, nodes == 1);

    double gbest = 0.0;
    int ibest = 0x7FFFFFFF, m_best = -1, s_best = -1;
    for (int i0 = 0; i0 < Gm; i0 += kWave) {
        const int i = i0 + lane;
        if (i >= Gm) continue;
        const double M = (double)M_list[i];
        if (M <= 0.0) continue;
        const double passes = quotient_up(M, per_pass);                // s + 1
        if (passes > (double)Gs) continue;
        const double ks = Kd * passes;
        const double m = quotient_up(M, ks);                           // 1 <= m <= m_mem
        const double Km = Kd * m;
        const double Mrun = Km * passes;
        if (Mrun < gp.M0 || Mrun > gp.Mmax) continue;
        const double tg = gp.alpha_g + gp.beta_g * m;                  // Eq. 8
        const double last = last_pass(c, st, tg, st.mode == 2 ? px_log(c, tg) : 0.0);
        const int s = (int)passes - 1;
        const double g = goodput_point(q, Km, tg, last, s);
        if (g > gbest) { gbest = g; ibest = i; m_best = (int)m; s_best = s; }
    }
    return wave_argmax(gbest, ibest, m_best, s_best);
}

template <bool LEAN>
__device__ __forceinline__ Best sweep_sampled(const Job &q, const int32_t *__restrict__ M_list, int Gm, int Gs, int K, int nodes)
{
    return sweep_sampled<LEAN>(plain_coefs(), q, load_grid_params(q.jp, q.J, q.j), load_sync(q), q.jp[(size_t)PX_M_MEM * q.J + q.j],
                               M_list, Gm, Gs, K, nodes);
}

// ---- fp32 variant of the sweep --------------------------------------------------
// The same model with every parameter rounded to fp32 and all arithmetic of Eq. 4-11 in
// fp32 (powf for Eq. 10).  Each lane elects its best s with the rearranged form of the fp64
// sweep, evaluated in fp32, and prices the elected point with Eq. 4 in the plain form.  The
// feasibility interval M0 <= K m (s+1) <= M_max stays the exact integer test of the fp64
// path.  Ties go to the lowest flat index.

struct JobF32 {
    float alpha_g, beta_g, alpha_sl, beta_sl, alpha_sn, beta_sn, gamma, inv_gamma, phi, a;
};

__device__ __forceinline__ JobF32 load_job_f32(const double *__restrict__ jp, int J, int j)
{
    JobF32 q;
    q.alpha_g = (float)jp[(size_t)PX_ALPHA_G * J + j];
    q.beta_g = (float)jp[(size_t)PX_BETA_G * J + j];
    q.alpha_sl = (float)jp[(size_t)PX_ALPHA_SL * J + j];
    q.beta_sl = (float)jp[(size_t)PX_BETA_SL * J + j];
    q.alpha_sn = (float)jp[(size_t)PX_ALPHA_SN * J + j];
    q.beta_sn = (float)jp[(size_t)PX_BETA_SN * J + j];
    q.gamma = (float)jp[(size_t)PX_GAMMA * J + j];
    q.inv_gamma = 1.0f / q.gamma;
    q.phi = (float)jp[(size_t)PX_PHI * J + j];
    q.a = q.phi + (float)jp[(size_t)PX_M0 * J + j];
    return q;
}

// A row beyond the tables.  terms(i, m): the half-offset quotients of batch size m, the i-th (see GridPoint); rK: 1 / K.
template <typename TERMS>
__device__ __forceinline__ Best sweep_beyond_f32(const JobF32 &q, const int32_t *__restrict__ m_row, const TERMS &terms, double rK, int Gm,
                                                 int Gs, int K, int nodes)
{
    const int lane = lane_id();
    const float Kf = (float)K;
    float ts = 0.0f;                                                          // Eq. 9
    if (K > 1) ts = (nodes == 1) ? q.alpha_sl + q.beta_sl * (float)(K - 2) : q.alpha_sn + q.beta_sn * (float)(K - 2);
    const float tsg = (ts != 0.0f && q.gamma != 1.0f) ? powf(ts, q.gamma) : 0.0f;

    float gbest = -1.0f;
    int flat = 0x7FFFFFFF, m_best = -1, s_best = -1;
    for (int i0 = 0; i0 < Gm; i0 += kWave) {
        const int i = i0 + lane;
        if (i >= Gm) continue;
        const int m = m_row[i];
        const float mf = (float)m;
        const float tg = q.alpha_g + q.beta_g * mf;                           // Eq. 8
        float last;                                                           // Eq. 10
        if (ts == 0.0f) last = tg;
        else if (q.gamma == 1.0f) last = tg + ts;
        else last = powf(powf(tg, q.gamma) + tsg, q.inv_gamma);
        const double2 quotients = terms(i, m);
        const int s_lo = (int)(quotients.x * rK);
        int s_hi = (int)(quotients.y * rK) - 1;
        s_hi = s_hi < Gs - 1 ? s_hi : Gs - 1;
        // the lane's best s by the same rearrangement as the fp64 sweep, in fp32: argmax GOODPUT = argmin h,
        // h = (last + u tg) + s tg + (last - tg) u / (s + 1), u = phi / (K m); ties to the smaller s
        const float Km = Kf * mf;
        const float u = q.phi / Km;
        const float A0 = fmaf(u, tg, last), B0 = (last - tg) * u;
        float hbest = __builtin_inff();
        int sb = -1;
        for (int sI = s_lo; sI <= s_hi; ++sI) {
            const float h = fmaf(B0, __builtin_amdgcn_rcpf((float)(sI + 1)), fmaf((float)sI, tg, A0));
            if (h < hbest) { hbest = h; sb = sI; }
        }
        if (sb >= 0) {
            // Eq. 4 at the elected point, plain form
            const float M = Km * (float)(sb + 1);
            const float t_iter = (float)sb * tg + last;                      // Eq. 11
            const float g = (M / t_iter) * (q.a / (q.phi + M));              // Eq. 7 x Eq. 6
            if (g > gbest) { gbest = g; flat = i * Gs + sb; m_best = m; s_best = sb; }
        }
    }
    return wave_argmax((double)gbest, flat, m_best, s_best);
}

__device__ __forceinline__ Best sweep_f32(const JobF32 &q, const JobTables &tb, const double *__restrict__ rk, int Gm, int Gs, int K, int nodes)
{
    if (K <= 0) return Best{0.0, -1, -1};
    auto terms = [&](int i, int) { return double2{tb.ql5[i], tb.qh5[i]}; };
    return sweep_beyond_f32(q, tb.m, terms, K < kRecipTable ? rk[K] : 1.0 / (double)K, Gm, Gs, K, nodes);
}

// ---- fp32 variant: the same sweep as the fp64 one ------------------------------
// For GPU counts within the tables.  Lane l owns batch sizes i = l, l + 64, ...; for each it takes the smallest
// w(s) = s + C / (s + 1) over all accumulation counts in chunks of 16, one v_fma_f32 per grid point
// (1/(s+1) from scalar registers, s from sixteen vector registers that hold 0 .. 15 for the whole
// kernel) and one v_min3_f32 per two points: three instructions per two grid points.  Where the argmin over all counts is not
// feasible w is taken at the end of the feasible counts towards it, by the same exact test as in fp64 (w(s+1) < w(s) exactly when
// C > (s+1)(s+2); the products are exact for grids of up to 4094 counts).
// The wave takes the smallest h (equal values: lowest batch size; elect_scanned, settle_f32).  The elected point's count follows from
// its C, and the point is priced with Eq. 4 in the plain form, in fp32 (price_point_f32).  T_grad, u and C are formed in fp32 from the
// parameters rounded to fp32; the last pass of Eq. 10 is the fp64 table rounded to fp32.
typedef const float __attribute__((address_space(4))) *ScalarFloats;
typedef const float __attribute__((address_space(3))) *LdsFloats;

struct RunStepsF32 {
    float x[16];
};

__device__ __forceinline__ RunStepsF32 make_run_steps_f32()
{
    RunStepsF32 X;
#pragma unroll
    for (int t = 0; t < 16; ++t) X.x[t] = (float)t;
    asm volatile("" : "+v"(X.x[0]), "+v"(X.x[1]), "+v"(X.x[2]), "+v"(X.x[3]), "+v"(X.x[4]), "+v"(X.x[5]), "+v"(X.x[6]), "+v"(X.x[7]));
    asm volatile("" : "+v"(X.x[8]), "+v"(X.x[9]), "+v"(X.x[10]), "+v"(X.x[11]), "+v"(X.x[12]), "+v"(X.x[13]), "+v"(X.x[14]), "+v"(X.x[15]));
    return X;
}

// Two grid points at positions B, B + 1 of a chunk: their values of w relative to the chunk's first count,
// folded into the running minimum.
template <int B>
__device__ __forceinline__ void scan_two_f32(float &wmin, float C, float r0, float r1, const RunStepsF32 &X)
{
    float w0, w1;
    asm("v_fma_f32 %0, %1, %2, %3" : "=v"(w0) : "v"(C), "s"(r0), "v"(X.x[B]));
    asm("v_fma_f32 %0, %1, %2, %3" : "=v"(w1) : "v"(C), "s"(r1), "v"(X.x[B + 1]));
    if constexpr (B == 0) asm("v_min_f32 %0, %1, %2" : "=v"(wmin) : "v"(w0), "v"(w1));
    else asm("v_min3_f32 %0, %0, %1, %2" : "+v"(wmin) : "v"(w0), "v"(w1));
}

template <int CH, int B = 0, typename RECIPS>
__device__ __forceinline__ void scan_chunk_f32(float &wmin, float C, const RECIPS &r, const RunStepsF32 &X)
{
    if constexpr (B < CH) {
        scan_two_f32<B>(wmin, C, r[B], r[B + 1], X);
        scan_chunk_f32<CH, B + 2>(wmin, C, r, X);
    }
}

// The smallest w(s) among all counts of the grid.  first: the reciprocals of the first CH counts.
template <int CH, typename RECIPS>
__device__ __forceinline__ float scan_min_f32(float C, const RunStepsF32 &X, ScalarFloats rsc, int Gs, const RECIPS &first)
{
    float wmin;
    scan_chunk_f32<CH>(wmin, C, first, X);
    for (int s0 = CH; s0 < Gs; s0 += CH) {
        float w;
        scan_chunk_f32<CH>(w, C, rsc + s0, X);               // values relative to the chunk's first count
        wmin = fminf(wmin, w + (float)s0);
    }
    return wmin;
}

template <int CH>
__device__ __forceinline__ float scan_min_f32(float C, const RunStepsF32 &X, ScalarFloats rsc, int Gs)
{
    return scan_min_f32<CH>(C, X, rsc, Gs, rsc);
}

// Eq. 9 in fp32.
__device__ __forceinline__ float t_sync_f32(const JobF32 &q, int K, bool one_node)
{
    if (K <= 1) return 0.0f;
    return one_node ? q.alpha_sl + q.beta_sl * (float)(K - 2) : q.alpha_sn + q.beta_sn * (float)(K - 2);
}

// The terms of one batch size: h(s) = A0 + T_grad (s + C / (s + 1)).  tabled: the last pass of Eq. 10 as the fp64 table has it.
struct TermsF32 {
    float tg, last, A0, C;
};

__device__ __forceinline__ TermsF32 terms_f32(const JobF32 &q, float ts, float Kf, int m, float tabled)
{
    TermsF32 t;
    const float mf = (float)m;
    t.tg = q.alpha_g + q.beta_g * mf;                                         // Eq. 8
    t.last = ts == 0.0f ? t.tg : (q.gamma == 1.0f ? t.tg + ts : tabled);      // Eq. 10
    const float u = q.phi * __builtin_amdgcn_rcpf(Kf * mf);
    t.A0 = fmaf(u, t.tg, t.last);
    t.C = (t.last - t.tg) * u * __builtin_amdgcn_rcpf(t.tg);
    return t;
}

// The smallest h over the feasible counts s_lo .. s_hi (see Feasible); wmin: the smallest w over all counts, recip(s): 1 / (s + 1).
template <typename RECIP>
__device__ __forceinline__ float feasible_h_f32(const TermsF32 &t, int s_lo, int s_hi, float wmin, const RECIP &recip)
{
    const float lo = (float)s_lo, hi = (float)s_hi;
    const bool above = t.C > fmaf(hi, hi, fmaf(3.0f, hi, 2.0f)), below = t.C <= fmaf(lo, lo, lo);
    const float w = fmaf(t.C, recip(above ? s_hi : s_lo), above ? hi : lo);
    return fmaf(t.tg, (int)above | (int)below ? w : wmin, t.A0);
}

// h at count s, as every election that needs no scan forms it (elect_scanned).
template <typename RECIP>
__device__ __forceinline__ float exact_h_f32(const TermsF32 &t, int s, const RECIP &recip)
{
    return fmaf(t.tg, fmaf(t.C, recip(s), (float)s), t.A0);
}

// All 64 lanes call this with the same (job, 1 <= K <= kTableK, nodes); every lane returns the same result.
// rsf: 1/(s+1) in fp32, padded to a multiple of 32 counts; near: a copy of it in LDS when has_near.  Returns the batch size of the
// feasible point with the smallest h, or -1.
template <int CH, bool WHOLE>
__device__ __forceinline__ int sweep_pick_f32(const JobF32 &q, const JobTables &tb, const RunStepsF32 &X,
                                              const float *__restrict__ rsf, int Gm, int Gs, int K, int nodes,
                                              LdsFloats near = nullptr, bool has_near = false)
{
    static_assert(CH == 8 || CH == 16, "sixteen steps in registers");
    const int lane = lane_id();
    K = __builtin_amdgcn_readfirstlane(K);
    nodes = __builtin_amdgcn_readfirstlane(nodes);
    const bool one_node = nodes == 1;
    const float Kf = (float)K, ts = t_sync_f32(q, K, one_node);
    const double *__restrict__ lrow = tb.lt + (unsigned)((one_node ? kTableK : 0) + K - 1) * (unsigned)Gm;
    const int32_t *__restrict__ srow = tb.srange + (unsigned)(K - 1) * (unsigned)Gm;
    const ScalarFloats rsc = (ScalarFloats)rsf;
    auto recip = [&](int s) { return has_near ? near[s] : rsf[s]; };

    float kbest = __builtin_inff();   // smallest h seen by this lane
    int where = 0;                    // the first of its group of 64 batch sizes
    unsigned long long again = 0;     // the lanes of which another h is close to the smallest (elect_scanned)
    for (int i0 = 0; i0 < Gm; i0 += kWave) {
        const int i = i0 + lane;
        const bool active = WHOLE || i < Gm;
        const int il = active ? i : Gm - 1;
        const TermsF32 t = terms_f32(q, ts, Kf, tb.m[il], (float)lrow[il]);
        const int bounds = srow[il];
        const int s_lo = bounds & 0xFFFF, s_hi = bounds >> 16;
        const bool feasible = active && s_lo <= s_hi;
        const float key = feasible_h_f32(t, s_lo, s_hi, scan_min_f32<CH>(t.C, X, rsc, Gs), recip);
        const bool better = feasible && key < kbest;
        if (i0 > 0) again = (again & ~__builtin_amdgcn_ballot_w64(better)) | __builtin_amdgcn_ballot_w64(feasible && close_to(kbest, key));
        if (better) {
            kbest = key;
            where = i0;
        }
    }
    return elect_scanned(kbest, again, [&](int l) { return __builtin_amdgcn_readlane(where, l); });
}

// The election of a row of the tables by h itself, as settle in fp64.  All 64 lanes call this with the same arguments.
__device__ __forceinline__ int settle_f32(int lane, const JobF32 &q, const JobTables &tb, const float *__restrict__ rsf, int Gm, int Gs, int K,
                                          bool one_node)
{
    const double *__restrict__ lrow = tb.lt + (unsigned)((one_node ? kTableK : 0) + K - 1) * (unsigned)Gm;
    const int32_t *__restrict__ srow = tb.srange + (unsigned)(K - 1) * (unsigned)Gm;
    const float Kf = (float)K, ts = t_sync_f32(q, K, one_node);
    float kbest = __builtin_inff();
    int where = 0;
    for (int i = lane; i < Gm; i += kWave) {
        const TermsF32 t = terms_f32(q, ts, Kf, tb.m[i], (float)lrow[i]);
        const int s_lo = srow[i] & 0xFFFF, s_hi = srow[i] >> 16;
        const float key = exact_h_f32(t, px_best_count(t.C, s_lo, s_hi), [&](int s) { return rsf[s]; });
        if (s_lo <= s_hi && key < kbest) {
            kbest = key;
            where = (i / kWave) << 16;
        }
    }
    return elect((double)kbest, where, 0ull, Gs).i;        // (positive floats order like their values in double precision)
}

// The same election for four (job, K, placement) at once, one per row of 16 lanes, as sweep_pick_rows does in fp64: lane l of
// a row takes batch sizes l, l + 16, ...; every lane of a row returns the batch size of the row's point, or -1.  Per (K, batch
// size) the arithmetic is that of sweep_pick_f32.
template <int CH, bool WHOLE>
__device__ __forceinline__ int sweep_pick_rows_f32(const JobF32 &q, const JobTables &tb, const RunStepsF32 &X, const float *__restrict__ rsf,
                                                   int Gm, int Gs, int K, bool one_node, LdsFloats near, bool has_near)
{
    const int l16 = lane_id() & 15;
    const float Kf = (float)K, ts = t_sync_f32(q, K, one_node);
    // byte offsets inside one job's tables, 32 bits each (see sweep_pick_rows)
    const unsigned l_row = (unsigned)((one_node ? kTableK : 0) + K - 1) * (unsigned)Gm * 8u;
    const unsigned s_row = (unsigned)(K - 1) * (unsigned)Gm * 4u;
    const ScalarFloats rsc = (ScalarFloats)rsf;
    auto recip = [&](int s) { return has_near ? near[s] : rsf[s]; };
    float kbest = __builtin_inff();
    unsigned runner_up = ~0u;         // the bits of the second smallest (elect_scanned_rows)
    int where = 0;
    for (int i0 = 0; i0 < Gm; i0 += 16) {
        const int i = i0 + l16;
        const bool active = WHOLE || i < Gm;
        const unsigned il = (unsigned)(active ? i : Gm - 1);
        const int m = *(const int32_t *)((const char *)tb.m + 4u * il);
        const double last = *(const double *)((const char *)tb.lt + (l_row + 8u * il));
        const int bounds = *(const int32_t *)((const char *)tb.srange + (s_row + 4u * il));
        float first[CH];
#pragma unroll
        for (int b = 0; b < CH; ++b) first[b] = rsc[b];
        __builtin_amdgcn_sched_barrier(0);            // (all are asked for before the first is waited for)
        const TermsF32 t = terms_f32(q, ts, Kf, m, (float)last);
        const int s_lo = bounds & 0xFFFF, s_hi = bounds >> 16;
        const bool feasible = active && s_lo <= s_hi;
        float key = feasible_h_f32(t, s_lo, s_hi, scan_min_f32<CH>(t.C, X, rsc, Gs, first), recip);
        key = feasible ? key : __int_as_float(-1);         // (not a number: never smaller, and the largest of bit patterns)
        runner_up = second_smallest(Closeness<float>::bits(kbest), runner_up, Closeness<float>::bits(key));
        if (key < kbest) {
            kbest = key;
            where = i;
        }
    }
    return elect_scanned_rows(kbest, runner_up, where);
}

// Eq. 4 for batch size i at its best feasible count, in the plain form, in fp32, for a GPU count within the tables.  Arguments may
// differ from lane to lane.
__device__ __forceinline__ Best price_point_f32(const JobF32 &q, const JobTables &tb, int Gm, int K, bool one_node, int i)
{
    if (i < 0) return Best{0.0, -1, -1};
    const int m = tb.m[i];
    const TermsF32 t = terms_f32(q, t_sync_f32(q, K, one_node), (float)K, m,
                                 (float)tb.lt[(unsigned)((one_node ? kTableK : 0) + K - 1) * (unsigned)Gm + (unsigned)i]);
    const int bounds = tb.srange[(unsigned)(K - 1) * (unsigned)Gm + (unsigned)i];
    const int s = px_best_count(t.C, bounds & 0xFFFF, bounds >> 16);
    const float M = (float)K * (float)m * (float)(s + 1);
    const float t_iter = (float)s * t.tg + t.last;                            // Eq. 11
    const float g = (M / t_iter) * (q.a / (q.phi + M));                       // Eq. 7 x Eq. 6
    return Best{(double)g, m, s};
}

// The fp32 sweep of one (job, K, nodes) whatever K: scan and price within the tables, the plain loop beyond.
// Every lane returns the same result.
template <int CH>
__device__ __forceinline__ Best sweep_any_f32(const JobF32 &q, const JobTables &tb, const float *__restrict__ rsf,
                                              const double *__restrict__ rk, int Gm, int Gs, int K, int nodes)
{
    K = __builtin_amdgcn_readfirstlane(K);
    nodes = __builtin_amdgcn_readfirstlane(nodes);
    if (K <= 0) return Best{0.0, -1, -1};
    if (!tabled_row(K, nodes == 1, tb.k1)) return sweep_f32(q, tb, rk, Gm, Gs, K, nodes);
    int i = sweep_pick_f32<CH, false>(q, tb, make_run_steps_f32(), rsf, Gm, Gs, K, nodes);
    if (i == kClose) i = settle_f32(lane_id(), q, tb, rsf, Gm, Gs, K, nodes == 1);
    return price_point_f32(q, tb, Gm, K, nodes == 1, i);
}

// ---- per job: what the status word says of its parameters, and its current row ------------------

__device__ __forceinline__ int job_status(const GridParams &g, const SyncParams &y, double weight)
{
    if (!(y.gamma >= 1.0 && y.gamma <= 10.0) || !(g.alpha_g >= 0.0) || !(g.beta_g >= 0.0) || !(y.alpha_sl >= 0.0) ||
        !(y.beta_sl >= 0.0) || !(y.alpha_sn >= 0.0) || !(y.beta_sn >= 0.0) || !(g.phi > 0.0) || !(g.M0 >= 1.0) ||
        !(g.Mmax >= g.M0) || !(weight >= 0.0) || !(g.Mmax <= 4503599627370496.0) || !(g.alpha_g + g.beta_g > 0.0))
        return PX_ST_BAD_PARAM;
    return 0;
}

struct CurrentRow {
    long long total;                // GPUs the job holds now
    bool negative;                  // the row has a negative entry
    unsigned long long groups;      // groups of four entries that hold a non-zero one (rows that one 16-byte load per lane covers)
};

__device__ __forceinline__ CurrentRow current_row(const FitnessArgs &a, int j)
{
    const int lane = lane_id();
    const int32_t *__restrict__ row = a.current_alloc + (size_t)j * a.N;
    CurrentRow out = {0, false, 0ull};
    long long sum = 0;
    bool neg = false;
    for (int n = lane; n < a.N; n += kWave) {
        const int c = row[n];
        sum += c;
        neg |= c < 0;
    }
    out.total = wave_sum(sum);
    out.negative = __ballot(neg) != 0ull;
    if (a.N <= 4 * kWave) {
        bool any = false;
        for (int n = 4 * lane; n < 4 * lane + 4 && n < a.N; ++n) any |= row[n] != 0;
        out.groups = __ballot(any);
    }
    return out;
}

// ---- the argmax of one (job, K, placement) in place ------------------------------------------
// What the calls that ask for a handful of argmaxes per job need (fair shares, memoised rows, rows beyond the memo table,
// the queries outside the search): the same election as sweep_pick without any table.  Lane l forms the terms of its batch
// sizes itself; the best accumulation count needs no scan (px_best_count).

// The terms of one batch size with 1/K = rK: h(s) = A0 + T_grad (s + C / (s + 1)), and its feasible counts.
struct RowTerms {
    double A0, B0, C;
    int s_lo, s_hi;

    __device__ __forceinline__ bool none() const { return s_lo > s_hi || s_hi < 0; }
};

__device__ __forceinline__ RowTerms row_terms(const GridPoint &g, double last, double rK, int Gs)
{
    RowTerms t;
    feasible_range(g.ql5, g.qh5, rK, Gs, t.s_lo, t.s_hi);
    const double u = g.pu * rK;
    t.A0 = px_fma(u, g.tg, last);
    t.B0 = (last - g.tg) * u;
    t.C = t.B0 * g.rtg;
    return t;
}

// h of one batch size at its best feasible count s_c (+inf when no count is feasible).  tabled: h in the form the tables
// give it (C and A0), else in the form of the untabled sweep: rounding decides elections between equal points, so a row
// keeps the form its sweep has.
__device__ __forceinline__ double best_count(const GridPoint &g, const RowTerms &t, bool tabled, int &s_c)
{
    s_c = px_best_count(t.C, t.s_lo, t.s_hi);
    const double sd = (double)s_c, r = px_div(1.0, sd + 1.0);
    const double h = tabled ? px_fma(g.tg, px_fma(t.C, r, sd), t.A0) : px_fma(t.B0, r, px_fma(sd, g.tg, t.A0));
    return t.none() ? __builtin_inf() : h;
}

// The most counts of a call in one launch (small_call), and of one whose single-precision fair shares come with the tables' launch.
constexpr int kSmallGs = 32;

// All 64 lanes call this with the same arguments; every lane returns the same result.  m_row: the job's batch sizes.
// The elected point is priced from the terms its lane has formed; LEAN: from terms formed anew, which holds five registers less.
template <bool LEAN = false>
__device__ __forceinline__ Best row_best(const Coefs &c, const Job &q, const GridParams &gp, const SyncParams &y,
                                         const int32_t *__restrict__ m_row, int Gm, int Gs, int K, bool one_node, bool tabled)
{
    const SyncTerm st = sync_term(c, y, K, one_node);
    const double rK = 1.0 / (double)K;
    double kbest = __builtin_inf(), tg_at = 0.0, last_at = 0.0;
    int where = 0, m_at = 0;
    for (int i = lane_id(); i < Gm; i += kWave) {
        const int m = m_row[i];
        const GridPoint g = grid_point(c, gp, m);
        const double last = last_pass(c, st, g.tg, g.lntg);
        int s_c;
        const double h = best_count(g, row_terms(g, last, rK, Gs), tabled, s_c);
        if (h < kbest) {
            kbest = h;
            where = s_c | ((i / kWave) << 16);
            if constexpr (!LEAN) {
                tg_at = g.tg;
                last_at = last;
                m_at = m;
            }
        }
    }
    const Pick pick = elect(kbest, where, 0ull, Gs);
    if (pick.i < 0) return Best{0.0, -1, -1};
    if constexpr (LEAN) {
        const int m = m_row[pick.i];
        const double tg = gp.alpha_g + gp.beta_g * (double)m;
        return Best{goodput_point(q, (double)K * (double)m, tg, last_pass(c, st, tg, px_log(c, tg)), pick.s), m, pick.s};
    }
    const int l = pick.i & (kWave - 1);
    const int m = __builtin_amdgcn_readlane(m_at, l);
    return Best{goodput_point(q, (double)K * (double)m, wave_read(tg_at, l), wave_read(last_at, l), pick.s), m, pick.s};
}

template <bool LEAN>
__device__ __forceinline__ Best row_best_plain(const Job &q, const GridParams &gp, const int32_t *__restrict__ m_row, int Gm, int Gs, int K,
                                               bool one_node, bool tabled)
{
    return row_best<LEAN>(plain_coefs(), q, gp, load_sync(q), m_row, Gm, Gs, K, one_node, tabled);
}

// The same in single precision, for a GPU count within the tables: the same point as sweep_pick_f32 and price_point_f32 find, the same
// bits (elect_scanned).
__device__ __forceinline__ Best row_best_f32(const Coefs &c, const JobF32 &q, const GridParams &gp, const SyncParams &y,
                                             const int32_t *__restrict__ m_row, int Gm, int Gs, int K, bool one_node)
{
    const SyncTerm st = sync_term(c, y, K, one_node);
    const double rK = 1.0 / (double)K;
    const float Kf = (float)K, ts = t_sync_f32(q, K, one_node);
    float kbest = __builtin_inff();
    TermsF32 at = {};                     // the lane's best: its terms and batch size
    int where = 0, m_at = 0;
    for (int i = lane_id(); i < Gm; i += kWave) {
        const int m = m_row[i];
        const GridPoint g = grid_point(c, gp, m);
        const TermsF32 t = terms_f32(q, ts, Kf, m, (float)last_pass(c, st, g.tg, g.lntg));
        int s_lo, s_hi;
        feasible_range(g.ql5, g.qh5, rK, Gs, s_lo, s_hi);
        const int s_c = px_best_count(t.C, s_lo, s_hi);
        const float key = exact_h_f32(t, s_c, [](int s) { return 1.0f / (float)(s + 1); });
        if (s_lo <= s_hi && s_hi >= 0 && key < kbest) {
            kbest = key;
            where = s_c | ((i / kWave) << 16);
            at = t;
            m_at = m;
        }
    }
    const Pick pick = elect((double)kbest, where, 0ull, Gs);      // (positive floats order like their values in double precision)
    if (pick.i < 0) return Best{0.0, -1, -1};
    const int l = pick.i & (kWave - 1), s = pick.s;
    auto read = [&](float v) { return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), l)); };
    const int m = __builtin_amdgcn_readlane(m_at, l);
    const float M = (float)K * (float)m * (float)(s + 1);
    const float t_iter = (float)s * read(at.tg) + read(at.last);              // Eq. 11
    const float g = (M / t_iter) * (q.a / (q.phi + M));                       // Eq. 7 x Eq. 6
    return Best{(double)g, m, s};
}

// ---- everything that depends on the jobs only: one launch ---------------------------------------
// The wavefronts of a job: one that checks its parameters, finds its fair-share goodput (denominator of Eq. 15) and its
// re-allocation factor, and further ones that take ROWS rows (placement class, K) each.  No wavefront reads what another
// writes (each forms the terms of its own batch sizes, an eighth of a row's work), so a call needs one launch here where
// it took three or four, one after the other: at 8 jobs 15 us of launches became 7, at 200 jobs 25 became 11.
// Bound by the vector ALU (busy 0.7 at 900 memoised jobs) and, at 200 jobs, by how few wavefronts there are to spread over the
// SIMDs: what a wavefront forms before its first row counts as much as three rows.
//   kPrepPlain    rows into the tables of the sweep (lt, ca, srange; per grid point tg, lntg, pu, qh5, ql5)
//   kPrepTablesF32  the same for the fp32 variant, fair shares in single precision
//   kPrepTables   the same for the fp32 variant on grids of more than kSmallGs counts: fair shares are found from the tables, by a
//                 launch of its own (jobs_kernel_f32)
//   kPrepMemo     memoised mode: the rows' argmaxes into the memo table, no other table
//   kPrepSampled  the sampling argmax: fair shares only (no table)
//   kPrepSampledMemo  and with its rows memoised
// Rows of the "one node" class stop at the largest node capacity: a job on one node holds at most that node's GPUs.  A row
// that claims more there, which no valid allocation does, is swept in place like a row beyond the tables (tabled_row).
// Table rows: lt[row][i] the last pass, ca[row][i] = (C, A0) with A0 = +inf where no accumulation count is feasible, or where the
// batch size is the one before it again: geometric grids round their small sizes to the same ones, of equal values the first is
// elected, and without its twins that one is alone for elect_scanned.  Such a batch size never wins an election.
// row = (j * 2 + one_node) * kTableK + K - 1; the rows of the "several nodes" class also write the feasible counts of (job, K, i),
// which do not depend on the class: srange[j][K-1][i] = first | last << 16, first > last when there is none (or a twin).
// Workgroups are dealt to the XCDs round-robin; a job's wavefronts run on XCD j % 8, as its pairs do.
enum PrepMode { kPrepPlain, kPrepTables, kPrepTablesF32, kPrepMemo, kPrepSampled, kPrepSampledMemo };

constexpr bool prep_has_tables(int mode) { return mode == kPrepPlain || mode == kPrepTables || mode == kPrepTablesF32; }
constexpr int prep_tasks(int mode, int rows) { return 1 + (mode == kPrepSampled ? 0 : 2 * kTableK / rows); }

// Whether some node holds at least K GPUs.
__device__ __forceinline__ bool node_holds(const FitnessArgs &a, int K)
{
    bool found = false;
    for (int n0 = 0; n0 < a.N && !found; n0 += kWave) {
        const int n = n0 + lane_id();
        found = __ballot(n < a.N && a.node_capacity[n] >= K) != 0ull;
    }
    return found;
}

template <int MODE>
__device__ __forceinline__ void prepare_job(const Coefs &c, const FitnessArgs &a, int j)
{
    const int lane = lane_id();
    const double *__restrict__ jp = a.job_params;
    const GridParams gp = load_grid_params(jp, a.J, j);
    const int32_t *__restrict__ m_row = a.m_grid + (size_t)j * a.Gm;
    if constexpr (prep_has_tables(MODE)) {
        for (int i = lane; i < a.Gm; i += kWave) {
            const GridPoint g = grid_point(c, gp, m_row[i]);
            const size_t o = (size_t)j * a.Gm + i;
            a.tg[o] = double2{g.tg, g.rtg};
            a.lntg[o] = g.lntg;
            a.pu[o] = g.pu;
            a.qh5[o] = g.qh5;
            a.ql5[o] = g.ql5;
        }
    }
    if constexpr (MODE == kPrepTables) return;
    const Job q = load_job(jp, a.J, j);
    const SyncParams y = load_sync(q);
    const double w = jp[(size_t)PX_WEIGHT * a.J + j];
    const double T = jp[(size_t)PX_AGE_T * a.J + j];
    const double R = jp[(size_t)PX_RESTARTS_R * a.J + j];
    constexpr bool kSampled = MODE == kPrepSampled || MODE == kPrepSampledMemo;
    int st = job_status(gp, y, w);
    if constexpr (kSampled) {
        const double m_mem = jp[(size_t)PX_M_MEM * a.J + j];
        if (!(m_mem >= 1.0 && m_mem <= 2147483647.0)) st |= PX_ST_BAD_PARAM;
    }
    // re-allocation penalty factor of Sec. 4.2
    double factor = (T - R * a.delta) / (T + a.delta);
    if constexpr (MODE == kPrepTablesF32) factor = (double)(((float)T - (float)R * (float)a.delta) / ((float)T + (float)a.delta));
    if (!(a.flags & PX_FLAG_NO_REALLOC_PENALTY) && !(T - R * a.delta > 0.0)) st |= PX_ST_BAD_RESTART;
    const CurrentRow cur = current_row(a, j);
    if (cur.negative) st |= PX_ST_NEG_ALLOC;
    // denominator of Eq. 15: the same argmax at the fair-share allocation
    const int K = __builtin_amdgcn_readfirstlane(a.fair_share[2 * j]);
    const bool one_node = __builtin_amdgcn_readfirstlane(a.fair_share[2 * j + 1]) == 1;
    Best fair = {0.0, -1, -1};
    if constexpr (kSampled) fair = sweep_sampled<false>(c, q, gp, y, jp[(size_t)PX_M_MEM * a.J + j], m_row, a.Gm, a.Gs, K, one_node ? 1 : 2);
    else if constexpr (MODE == kPrepTablesF32) {
        auto terms = [&](int, int m) {
            const GridPoint g = grid_point(c, gp, m);
            return double2{g.ql5, g.qh5};
        };
        const JobF32 qf = load_job_f32(jp, a.J, j);
        if (K > 0 && K <= kTableK && (!one_node || node_holds(a, K))) fair = row_best_f32(c, qf, gp, y, m_row, a.Gm, a.Gs, K, one_node);
        else if (K > 0) fair = sweep_beyond_f32(qf, m_row, terms, 1.0 / (double)K, a.Gm, a.Gs, K, one_node ? 1 : 2);
    } else if (K > 0) fair = row_best(c, q, gp, y, m_row, a.Gm, a.Gs, K, one_node, K <= kTableK && (!one_node || node_holds(a, K)));
    if (!(fair.goodput > 0.0)) st |= PX_ST_ZERO_FAIR;
    if (lane == 0) {
        a.denom[j] = fair.goodput;
        a.factor[j] = (!(a.flags & PX_FLAG_NO_REALLOC_PENALTY) && cur.total > 0) ? factor : 1.0;
        a.curmask[j] = cur.groups;
        a.jobstat[j] = st;
    }
    if (j == 0 && lane < 16) a.zeros[lane] = 0;
}

// The argmaxes of `rows` (K, placement) of one job, at most a wavefront's lanes: lane r holds the r-th's K, its synchronisation term, 1/K and
// whether it takes the tables' form (see best_count), and returns its point.  The terms of a batch size are formed once for all rows.
__device__ __forceinline__ Best argmax_rows(const Coefs &c, const Job &q, const GridParams &gp, const int32_t *__restrict__ m_row, int Gm, int Gs,
                                            int rows, int my_K, const SyncTerm &mine, double my_rK, bool my_tabled)
{
    // Batch sizes two groups of 64 at a time, one election for both; later ones have to be better than what earlier ones elected
    // (equal values: the earlier).
    const int lane = lane_id();
    double my_h = __builtin_inf(), my_tg = 1.0, my_last = 1.0;
    int my_m = -1, my_s = -1;
    auto groups = [&](int i0, auto TWO) __attribute__((always_inline)) {
        constexpr bool two = decltype(TWO)::value;
        const int i = i0 + lane;
        const int m0 = m_row[i < Gm ? i : Gm - 1], m1 = two ? m_row[i + kWave < Gm ? i + kWave : Gm - 1] : 0;
        const GridPoint g0 = grid_point(c, gp, m0);
        GridPoint g1 = g0;
        if constexpr (two) g1 = grid_point(c, gp, m1);
#pragma unroll 1
        for (int r = 0; r < rows; ++r) {
            const SyncTerm t = {wave_read(mine.ts, r), wave_read(mine.lnts, r), mine.gamma, mine.inv_gamma,
                                __builtin_amdgcn_readlane(mine.mode, r)};
            const double rK = wave_read(my_rK, r);
            const bool tabled = __builtin_amdgcn_readlane((int)my_tabled, r) != 0;
            double last_at = last_pass(c, t, g0.tg, g0.lntg), tg_at = g0.tg;
            int where, m_at = m0;
            double h = best_count(g0, row_terms(g0, last_at, rK, Gs), tabled, where);
            if (!(i < Gm && h < __builtin_inf())) h = __builtin_inf();      // (not a number where T_grad overflows: no point either)
            if constexpr (two) {
                const double last = last_pass(c, t, g1.tg, g1.lntg);
                int s_c;
                const double h1 = best_count(g1, row_terms(g1, last, rK, Gs), tabled, s_c);
                if (i + kWave < Gm && h1 < h) {
                    h = h1;
                    where = s_c | (1 << 16);
                    last_at = last;
                    tg_at = g1.tg;
                    m_at = m1;
                }
            }
            const Pick pick = elect(h, where, 0ull, Gs);
            if (pick.i >= 0) {
                const int l = pick.i & (kWave - 1);
                const double h_l = wave_read(h, l), tg_l = wave_read(tg_at, l), last_l = wave_read(last_at, l);
                const int m_l = __builtin_amdgcn_readlane(m_at, l);
                const bool here = lane == r && h_l < my_h;
                my_h = here ? h_l : my_h;
                my_tg = here ? tg_l : my_tg;
                my_last = here ? last_l : my_last;
                my_m = here ? m_l : my_m;
                my_s = here ? pick.s : my_s;
            }
        }
    };
    for (int i0 = 0; i0 < Gm; i0 += 2 * kWave) {
        if (i0 + kWave < Gm) groups(i0, std::true_type());
        else groups(i0, std::false_type());
    }
    // lane r prices the point elected for row r, from the terms that point's lane has formed
    Best best = {0.0, my_m, my_s};
    if (my_m >= 0) best.goodput = goodput_point(q, (double)my_K * (double)my_m, my_tg, my_last, my_s);
    return best;
}

// ROWS rows from K0 on.  The rows follow one another in a loop: written out they want more scalar registers than there are, beside
// the constants.
template <int ROWS, int MODE>
__device__ __forceinline__ void prepare_rows(const Coefs &c, const FitnessArgs &a, int j, int K0, bool one_node)
{
    const int lane = lane_id();
    const size_t row0 = ((size_t)j * 2 + (one_node ? 1 : 0)) * kTableK + (K0 - 1);
    const Job q = load_job(a.job_params, a.J, j);
    const int32_t *__restrict__ m_row = a.m_grid + (size_t)j * a.Gm;
    const GridParams gp = load_grid_params(a.job_params, a.J, j);
    const SyncParams y = load_sync(q);
    if constexpr (MODE == kPrepSampledMemo) {
        const double m_mem = a.job_params[(size_t)PX_M_MEM * a.J + j];
#pragma unroll 1
        for (int r = 0; r < ROWS; ++r) {
            const Best best = sweep_sampled<false>(c, q, gp, y, m_mem, m_row, a.Gm, a.Gs, K0 + r, one_node ? 1 : 2);
            if (lane == 0) a.memo[row0 + r] = MemoEntry{best.goodput, best.m, best.s};
        }
        return;
    }
    // lane r prepares T_sync and its logarithm, and 1/K, for the r-th row
    const int my_K = K0 + (lane < ROWS ? lane : 0);
    const SyncTerm mine = sync_term(c, y, my_K, one_node);
    const double my_rK = px_div(1.0, (double)my_K);
    if constexpr (MODE == kPrepMemo) {
        const Best best = argmax_rows(c, q, gp, m_row, a.Gm, a.Gs, ROWS, my_K, mine, my_rK, true);
        if (lane < ROWS) a.memo[row0 + lane] = MemoEntry{best.goodput, best.m, best.s};
    } else {
        for (int i0 = 0; i0 < a.Gm; i0 += kWave) {
            const int i = i0 + lane;
            const bool active = i < a.Gm;
            const int il = active ? i : a.Gm - 1, m = m_row[il];
            const bool twin = il > 0 && m_row[il > 0 ? il - 1 : 0] == m;
            const GridPoint g = grid_point(c, gp, m);
            double *__restrict__ lt = a.lt + row0 * a.Gm;
            double2 *__restrict__ ca = a.ca + row0 * a.Gm;
            int32_t *__restrict__ ranges = a.srange + ((size_t)j * kTableK + (size_t)(K0 - 1)) * a.Gm;
#pragma unroll 1
            for (int r = 0; r < ROWS; ++r) {
                const SyncTerm t = {wave_read(mine.ts, r), wave_read(mine.lnts, r), mine.gamma, mine.inv_gamma,
                                    __builtin_amdgcn_readlane(mine.mode, r)};
                const double rK = wave_read(my_rK, r);
                const double last = last_pass(c, t, g.tg, g.lntg);
                int s_lo, s_hi;
                feasible_range(g.ql5, g.qh5, rK, a.Gs, s_lo, s_hi);
                const bool none = s_lo > s_hi || s_hi < 0 || twin;
                if (none) { s_lo = 1; s_hi = 0; }
                // what the sweep needs of (job, class, K, i): h(m_i, s) = A0 + T_grad (s + C / (s+1))
                const double u = g.pu * rK;
                const double A0 = px_fma(u, g.tg, last);
                const double B0 = (last - g.tg) * u;
                if (active) {
                    lt[(unsigned)i] = last;
                    ca[(unsigned)i] = double2{B0 * g.rtg, none ? __builtin_inf() : A0};
                    if (!one_node) ranges[(unsigned)i] = s_lo | (s_hi << 16);
                }
                lt += a.Gm;
                ca += a.Gm;
                ranges += a.Gm;
            }
        }
    }
}

template <int ROWS, int MODE>
__global__ void __launch_bounds__(256) prepare_kernel(FitnessArgs a)
{
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const size_t tid = (size_t)blockIdx.x * blockDim.x + threadIdx.x, threads = (size_t)gridDim.x * blockDim.x;
    if (tid < kStatusWords) a.status[tid] = 0;
    if (a.clear_counters) {
        // the per-candidate, per-node counters of the constraint check start the call at zero
        const size_t n = (size_t)a.P * a.N;
        for (size_t i = tid; i < n; i += threads) a.colpack[i] = 0ull;
    }
    if constexpr (prep_has_tables(MODE)) {
        for (size_t i = tid; i < (size_t)a.gs_pad; i += threads) {
            a.rs[i] = 1.0 / (double)(int)(i + 1);
            a.rsf[i] = 1.0f / (float)(int)(i + 1);
        }
        if (tid < kRecipTable) a.rk[tid] = tid > 0 ? 1.0 / (double)(int)tid : 0.0;
    }
    if (blockIdx.x == 0 && wave == 0) {
        int c = 0;
        for (int n = lane_id(); n < a.N; n += kWave) {
            const int v = a.node_capacity[n];
            c = v > c ? v : c;
        }
        c = (int)wave_max((unsigned)c);
        if (lane_id() == 0) *a.k1 = c < kTableK ? c : kTableK;
    }
    constexpr int kTasks = prep_tasks(MODE, ROWS);
    const PrepSlot slot = prep_slot(blockIdx.x, wave, kTasks);
    const int j = slot.job, task = slot.task;
    if (j >= a.J) return;
    const Coefs c = held_coefs();
    if (task == 0) {
        prepare_job<MODE>(c, a, j);
    } else if constexpr (MODE != kPrepSampled) {
        constexpr int kPerClass = kTableK / ROWS;
        const bool one_node = task - 1 >= kPerClass;
        const int K0 = ((task - 1) % kPerClass) * ROWS + 1;
        if (one_node && !node_holds(a, K0)) return;       // no row of this wavefront is ever looked up
        prepare_rows<ROWS, MODE>(c, a, j, K0, one_node);
    }
}

// ---- fp32 variant: fair shares and memo table, from the tables --------------------------------------

// (grids of more than kSmallGs counts)
__global__ void __launch_bounds__(256) jobs_kernel_f32(FitnessArgs a)
{
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int j = blockIdx.x * kWavesPerBlock + wave;
    if (j >= a.J) return;
    const int lane = lane_id();
    const double *__restrict__ jp = a.job_params;
    const double T = jp[(size_t)PX_AGE_T * a.J + j];
    const double R = jp[(size_t)PX_RESTARTS_R * a.J + j];
    int st = job_status(load_grid_params(jp, a.J, j), load_sync(load_job(jp, a.J, j)), jp[(size_t)PX_WEIGHT * a.J + j]);
    // re-allocation penalty factor of Sec. 4.2
    const double factor = (double)(((float)T - (float)R * (float)a.delta) / ((float)T + (float)a.delta));
    if (!(a.flags & PX_FLAG_NO_REALLOC_PENALTY) && !(T - R * a.delta > 0.0)) st |= PX_ST_BAD_RESTART;
    const CurrentRow cur = current_row(a, j);
    if (cur.negative) st |= PX_ST_NEG_ALLOC;
    const Best fair = sweep_any_f32<16>(load_job_f32(a.job_params, a.J, j), job_tables(a, j), a.rsf, a.rk, a.Gm, a.Gs,
                                        a.fair_share[2 * j], a.fair_share[2 * j + 1]);
    if (!(fair.goodput > 0.0)) st |= PX_ST_ZERO_FAIR;
    if (lane == 0) {
        a.denom[j] = fair.goodput;
        a.factor[j] = (!(a.flags & PX_FLAG_NO_REALLOC_PENALTY) && cur.total > 0) ? factor : 1.0;
        a.curmask[j] = cur.groups;
        a.jobstat[j] = st;
    }
    if (j == 0 && lane < 16) a.zeros[lane] = 0;
}

// One wavefront per (job, class, K <= kTableK).
template <int CH>
__global__ void __launch_bounds__(256) memo_kernel_f32(FitnessArgs a)
{
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const long long row = (long long)blockIdx.x * kWavesPerBlock + wave;
    if (row >= (long long)a.J * 2 * kTableK) return;
    const int K = (int)(row % kTableK) + 1;
    const int nodes = ((row / kTableK) & 1) ? 1 : 2;
    const int j = (int)(row / (2 * kTableK));
    if (nodes == 1 && K > *a.k1) return;            // never looked up (tabled_row)
    const Best best = sweep_any_f32<CH>(load_job_f32(a.job_params, a.J, j), job_tables(a, j), a.rsf, a.rk, a.Gm, a.Gs, K, nodes);
    if (lane_id() == 0) a.memo[row] = MemoEntry{best.goodput, best.m, best.s};
}

// ---- per (candidate, job) ------------------------------------------------------
// Workgroup -> (job, group of candidates).  Workgroups are dealt to the eight XCDs
// round-robin, so the job index is derived from (blockIdx % 8) first: all workgroups
// of one job then run on one XCD and its tables stay in that XCD's L2.  Each of the
// four wavefronts walks cand_per_wave candidates of that job.

// ROW1: the host has checked that a row has 4 to 256 entries, so one 16-byte load per lane covers it.
// RAG: rows of any length and alignment (row_lane: the lane of a row's last entries takes the last four and masks those its
// neighbour has).  Without it the host has checked that a row is whole 16-byte groups and that population and current_alloc
// are 16-byte aligned: the masks cost an instruction per entry (200 jobs on 64 nodes: 53.6 us against 52.4), so whole grids
// keep an instance without them.  (1021 candidates of 331 jobs on 130 nodes: 207 us entry by entry, 134 so.)
// WHOLE: the host has checked that Gm is a multiple of 64 (tabled sweeps then skip the test for the end of the grid).
// ROW4: ROW1 and a row is at most 64 entries, so one load of the wavefront covers the rows of four candidates
// (16 lanes each); cand_per_wave is at most 16.  kFourRowsSwept: the candidates are also swept four at a time (see split_pairs, balanced_split).
// SEL: only the candidates listed in a.sel are evaluated (the children a search step has just formed); the
// wavefronts then walk positions of that list and look the candidate up where an address is formed.
// Eight wavefronts per SIMD (64 registers); the instances that sweep four candidates at a time (rows_at_a_time)
// take six: two sets of 16 batch sizes that share the reciprocals want 80 registers (eight bytes of the row pass spill; 1000 x 200 on 64
// nodes, 64 x 16, 62.3 us a call with one set at a time and seven wavefronts, 60.1 so, 61.3 with five wavefronts and no spill).
// Order of a wavefront's work (ROW1): request its first rows; fill the workgroup's table in LDS (entries formed
// in registers, so nothing waits for memory) and meet the other wavefronts; reduce the rows two at a time, and
// hand the registers of each finished pair to the rows of the next stretch of eight; then the sweeps of its
// candidates, one after the other; then prices and stores.  What a wavefront spends waiting at its start is
// time the vector ALU has one wavefront fewer to draw on, so memory is asked as early as the addresses are known.
// Between row pass and sweeps (grids of at most 128 batch sizes, stage_candidates or more a wavefront): the workgroup's 64 pairs
// share one job and mostly a handful of (placement class, GPU count) rows of its tables, so each pair votes for
// its row, the rows with two votes or more (four at most) are copied to LDS once, and the sweeps of those pairs
// read (C, A0), T_grad and the feasible range from there.  Three vector-memory loads per lane and group of 64
// batch sizes were what kept the texture addresser two thirds busy and the vector ALU waiting.
enum { kRowAtATime, kFourRowsLoaded, kFourRowsSwept };      // ROW4
constexpr bool rows_at_a_time(int ROW4) { return ROW4 == kFourRowsSwept; }

// Wavefronts a SIMD.  The sampling argmax of a pair (CH = 0) spills 36 bytes a lane where eight leave it 64 registers: 74 candidates of
// 433 jobs on 79 nodes 46.0 us, seven 40.3, six 40.4; 100 of 1000 on 250 nodes, where the rows' reading counts, 146, 118 and 124.
constexpr int pair_waves(int CH, bool MEMO, int ROW4) { return rows_at_a_time(ROW4) ? 6 : (CH == 0 && !MEMO ? 7 : 8); }

// SEL = 2: per job, the candidates listed in a.dirty[j, 0 .. a.dirty_count[j]) (row inheritance: the rows of job j that a
// move or a repair of the search step has changed); workgroups beyond a job's list return at once.
template <int CH, bool F32, bool MEMO, bool ROW1, bool WHOLE, int ROW4, bool RAG, int SEL>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(pair_waves(CH, MEMO, ROW4))))
pairs_kernel(FitnessArgs a)
{
    const int xcd = blockIdx.x & 7, slot = blockIdx.x >> 3;
    const int j = (slot / a.cand_groups) * 8 + xcd;
    const int group = slot % a.cand_groups;
    if (j >= a.J) return;
    // the number of candidates this job's workgroups share out among them
    int P_eff = SEL == 1 ? a.n_sel : a.P;
    if constexpr (SEL == 2) {
        P_eff = __builtin_amdgcn_readfirstlane(a.dirty_count[j]);
        if (group * a.cand_per_wave * kWavesPerBlock >= P_eff) return;
    }
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int lane = lane_id();
    // the reciprocals 1/(s+1) also in LDS when they fit: a lane reads the entry of an end of its feasible counts
    // behind them U[t] = t (t+1), U[0] = -1: what decides the order of neighbouring counts (sweep_pick)
    // kStage: behind them the table rows most of the workgroup's pairs read (see kStageBase); stage_votes counts, per
    // (class, K), the pairs of the workgroup that read the row
    constexpr bool kStage = CH != 0 && !F32 && !MEMO && ROW1 && !ROW4;
    __shared__ __align__(16) double r_lds[kNearU + kNearRecips + 8 + (kStage ? kStageDoubles : 0)];
    __shared__ int stage_votes[kStage ? 2 * kTableK : 1];
    // (only where the table of reciprocals and thresholds is in LDS as well: sweep_pick's staged path reads both)
    // (the host's decision; formed here, which is the same, it costs whole grids 0.4 % and saves ragged ones 0.9 %)
    const bool stage_on = kStage && (WHOLE ? a.stage_rows != 0
                                           : a.Gm <= kStageGm && a.gs_pad <= kNearRecips && a.cand_per_wave >= stage_candidates(SEL != 0));
    bool has_near = false;
    // (the instances whose rows fit one 16-byte load per lane fill the table after they have requested their first rows)
    constexpr bool kRowsFirst = CH != 0 && ROW1;
    // every thread brings one entry: no load, so storing it waits for nothing that is on its way from memory.  px_div rounds the
    // reciprocals of whole numbers as the division does that fills a.rs (prepare_kernel): checked for all up to 2^14 by a host test
    static_assert(kNearRecips <= kWavesPerBlock * kWave, "one entry per thread");
    const bool near_fits = CH != 0 && !MEMO && a.gs_pad <= kNearRecips;
    const double near_d = px_div(1.0, (double)((int)threadIdx.x + 1));
    const float near_f = 1.0f / (float)((int)threadIdx.x + 1);
    auto fill_near = [&]() {
        if (near_fits) {
            const int t = threadIdx.x;
            if (t < a.gs_pad) {
                if constexpr (F32) {
                    ((float *)r_lds)[t] = near_f;
                } else {
                    r_lds[2 * t] = near_d;
                    r_lds[2 * t + 1] = (double)t;
                    for (int e = t; e < a.gs_pad + 8; e += a.gs_pad) {
                        const double ed = (double)e;
                        r_lds[kNearU + e] = e > 0 ? ed * (ed + 1.0) : -1.0;
                    }
                }
            }
        }
        if (stage_on && threadIdx.x < 2 * kTableK) stage_votes[threadIdx.x] = 0;
        if (near_fits || stage_on) __syncthreads();
        has_near = near_fits;
    };
    if constexpr (!kRowsFirst) fill_near();
    const Job q = load_job(a.job_params, a.J, j);
    JobF32 qf = {};
    if constexpr (F32) qf = load_job_f32(a.job_params, a.J, j);
    const JobTables tb = job_tables(a, j);
    const int32_t *__restrict__ cur = a.current_alloc + (size_t)j * a.N;
    const bool vec4 = ROW1 || ((a.N & 3) == 0 && (((uintptr_t)a.population | (uintptr_t)a.current_alloc) & 15) == 0);
    const int n4 = RAG ? (a.N + 3) >> 2 : a.N >> 2;   // lanes that hold entries of a row (ROW1), 16-byte groups of a row
    const int lane4 = lane < n4 ? lane : n4 - 1;      // lanes past the end of the row load its last 16 bytes again
    const unsigned long long in_row = __ballot(lane < n4);
    // RAG: the lane's first entry of a row and which of the four it keeps; such a lane's loads take any alignment
    const RowLane ragged = row_lane(ROW4 ? (lane & 15) : lane, RAG ? a.N : 4);
    auto kept = [&](const int4 &v) {
        if constexpr (RAG) return int4{v.x & ragged.mask.x, v.y & ragged.mask.y, v.z & ragged.mask.z, v.w & ragged.mask.w};
        else return v;
    };
    // the lane's entries of a row of ROW1 as they are in memory; `kept` of them when they are used
    auto load_entries = [&](const int32_t *from) {
        if constexpr (RAG) {
            const Entries e = *(const Entries *)(from + ragged.base);
            return int4{e.x, e.y, e.z, e.w};
        } else {
            return ((const int4 *)from)[ROW4 ? ((lane & 15) < n4 ? (lane & 15) : n4 - 1) : lane4];
        }
    };
    int4 cur0 = {0, 0, 0, 0};                         // the lane's share of the job's current row (its first 256 entries)
    if constexpr (ROW1) cur0 = kept(load_entries(cur));
    else if (vec4) cur0 = ((const int4 *)cur)[lane4];
    constexpr bool kDeferred = CH != 0;               // the grid sweeps of both precisions (not the sampling argmax)
    constexpr int kPriced = -3;                       // a row beyond the tables whose result lane r already holds (see below)
    int d_K = 0, d_meta = 0, d_i = -1, d_row = -1;    // lane r: what candidate r of this wavefront needs at the end
    RunSteps X = {};
    RunStepsF32 XF = {};
    bool any_neg = false;

    // The wavefront's r-th candidate is c0 + kWavesPerBlock * r; its row of job j and its counters are reached
    // by stepping pointers.  With SEL that number is a position in the list, and lane r holds the candidate
    // listed there (-1 past the end of the list).
    const int c0 = group * a.cand_per_wave * kWavesPerBlock + wave;
    int d_c = -1;
    if constexpr (SEL != 0) {
        const int k = c0 + kWavesPerBlock * lane;
        if (lane < a.cand_per_wave && k < P_eff) d_c = SEL == 2 ? a.dirty[(size_t)j * a.n_sel + k] : a.sel[k];
    }
    const size_t row_step = (size_t)kWavesPerBlock * a.J * a.N;
    const int32_t *__restrict__ row = a.population + ((size_t)c0 * a.J + j) * a.N - row_step;
    unsigned long long *__restrict__ cp = a.colpack + (size_t)c0 * a.N - (size_t)kWavesPerBlock * a.N;
    // the row of job j of the wavefront's r-th candidate (SEL), and making that candidate the current one
    auto row_of = [&](int r) -> const int32_t * {
        return a.population + ((size_t)__builtin_amdgcn_readlane(d_c, r) * a.J + j) * a.N;
    };
    auto advance = [&](int r) {
        if constexpr (SEL != 0) {
            row = row_of(r);
            cp = a.colpack + (size_t)__builtin_amdgcn_readlane(d_c, r) * a.N;
        } else {
            row += row_step;
            cp += (size_t)kWavesPerBlock * a.N;
        }
    };

    // The row stage of the current candidate (see advance): row reduce and constraint counters.
    // ROW1 callers that have the row in registers already pass it as `have`; otherwise it is read here.  Callers
    // that have the row's sum already pass it as `K_have`, with `in_range` when they know that the row has no
    // negative entry.
    auto row_stage = [&](int &K_out, int &nodes_out, bool &changed_out, bool &neg_out, const int4 *have = nullptr,
                         const int *K_have = nullptr, int in_range = 0) {
        // row reduce: K = sum, nodes = #positive, changed = differs from the current row
        int ksum = 0, nodes = 0;
        bool changed = false, neg = false;
        int4 v0 = {0, 0, 0, 0};       // the lane's first four entries (the whole row when N <= 256)
        if constexpr (ROW1) {
            const int4 v = have ? *have : kept(load_entries(row));
            v0 = v;
            if (!K_have) {
                const int part = (v.x + v.y) + (v.z + v.w);
                ksum = lane < n4 ? part : 0;
            }
            nodes = __popcll(__ballot(v.x > 0) & in_row) + __popcll(__ballot(v.y > 0) & in_row) +
                    __popcll(__ballot(v.z > 0) & in_row) + __popcll(__ballot(v.w > 0) & in_row);
            changed = ((__ballot(v.x != cur0.x) | __ballot(v.y != cur0.y) | __ballot(v.z != cur0.z) | __ballot(v.w != cur0.w)) & in_row) != 0;
            if (in_range == 0) neg = (__ballot((v.x | v.y | v.z | v.w) < 0) & in_row) != 0;
        } else if (vec4) {
            const int4 *__restrict__ row4 = (const int4 *)row;
            const int4 *__restrict__ cur4 = (const int4 *)cur;
            for (int n0 = 0; n0 < n4; n0 += kWave) {
                // lanes past the end of the row load its last 16 bytes again and are masked out of the ballots
                const int n = n0 + lane;
                const int nc = n < n4 ? n : n4 - 1;
                const int4 v = row4[nc];
                const int4 cv = n0 == 0 ? cur0 : cur4[nc];
                const unsigned long long valid = __ballot(n < n4);
                if (n0 == 0) v0 = v;
                const int part = (v.x + v.y) + (v.z + v.w);
                ksum += n < n4 ? part : 0;
                nodes += __popcll(__ballot(v.x > 0) & valid) + __popcll(__ballot(v.y > 0) & valid) +
                         __popcll(__ballot(v.z > 0) & valid) + __popcll(__ballot(v.w > 0) & valid);
                changed |= ((__ballot(v.x != cv.x) | __ballot(v.y != cv.y) | __ballot(v.z != cv.z) | __ballot(v.w != cv.w)) & valid) != 0;
                neg |= (__ballot((v.x | v.y | v.z | v.w) < 0) & valid) != 0;
            }
        } else {
            for (int n0 = 0; n0 < a.N; n0 += kWave) {
                const int n = n0 + lane;
                const int v = n < a.N ? row[n] : 0;
                const int cv = n < a.N ? cur[n] : 0;
                ksum += v;
                nodes += __popcll(__ballot(v > 0));
                changed |= __ballot(v != cv) != 0;
                neg |= __ballot(v < 0) != 0;
            }
        }
        const int K = K_have ? *K_have : wave_sum(ksum);

        // constraint check, part one: the row's non-zero entries (a job sits on few nodes) go to the
        // candidate's per-node counters; a multi-node job also counts once on each of its nodes.
        // One 64-bit integer atomic per entry: the result does not depend on the order of arrival.
        // (the flags of this stage are kept as integers in scalar registers: the compiler otherwise carries a
        // truth value across the branches as a lane mask that it rebuilds with two vector instructions)
        int need = __builtin_amdgcn_readfirstlane(a.need_constraints);
        asm volatile("" : "+s"(need));
        if (need != 0) {
            const unsigned long long one_job = nodes >= 2 ? kPackJob : 0ull;
            if ((ROW1 || (vec4 && a.N <= 4 * kWave)) && !neg) {
                // the row is still in registers and has no negative entry
                const int nb = RAG ? ragged.base : lane * 4;
                if (lane < n4) {
                    if (v0.x > 0) atomicAdd(&cp[nb + 0], (unsigned long long)v0.x + one_job);
                    if (v0.y > 0) atomicAdd(&cp[nb + 1], (unsigned long long)v0.y + one_job);
                    if (v0.z > 0) atomicAdd(&cp[nb + 2], (unsigned long long)v0.z + one_job);
                    if (v0.w > 0) atomicAdd(&cp[nb + 3], (unsigned long long)v0.w + one_job);
                }
            } else {
                for (int n = lane; n < a.N; n += kWave) {
                    const int v = row[n];
                    if (v != 0) atomicAdd(&cp[n], (unsigned long long)(long long)v + (v > 0 ? one_job : 0ull));
                }
            }
        }
        K_out = K; nodes_out = nodes; changed_out = changed; neg_out = neg;
    };

    if constexpr (kDeferred) {
        // grid sweep (either precision), in two passes over the wavefront's candidates so that neither pass keeps the
        // other's addresses in scalar registers: first the row stage of every candidate (lane r keeps K and
        // nodes | changed of candidate r), then the sweeps, which elect a point per candidate; the points are
        // priced after the loop.
        int rows = a.cand_per_wave;
        if (c0 + kWavesPerBlock * (rows - 1) >= P_eff) rows = c0 < P_eff ? (P_eff - c0 + kWavesPerBlock - 1) / kWavesPerBlock : 0;
        if constexpr (ROW4) {
            // Lanes 16 g .. 16 g + 15 hold the row of candidate 4 b + g of the wavefront in batch b; all
            // batches are requested together.  Sums over a row are sums over 16 lanes (four DPP steps).
            static_assert(ROW1, "rows of 16-byte groups");
            const int g = lane >> 4, l16 = lane & 15;
            const bool in_row16 = l16 < n4;
            const int at16 = RAG ? ragged.base : 4 * l16;
            const int32_t *__restrict__ row1 = row + row_step;
            unsigned long long *__restrict__ cp1 = cp + (size_t)kWavesPerBlock * a.N + at16;
            const int4 curg = cur0;
            constexpr int kBatches = kMaxCandPerWave / 4;
            int4 v[kBatches];
            int kb[kBatches] = {}, mb[kBatches] = {};
            int cb[kBatches] = {};           // SEL: the candidate whose row the lane holds in batch b
#pragma unroll
            for (int b = 0; b < kBatches; ++b) {
                if (4 * b < rows) {
                    const int r = 4 * b + g < rows ? 4 * b + g : rows - 1;             // the tail reads the last row again
                    if constexpr (SEL != 0) {
                        cb[b] = __builtin_amdgcn_ds_bpermute(r << 2, d_c);
                        v[b] = load_entries(a.population + ((size_t)cb[b] * a.J + j) * a.N);
                    } else {
                        v[b] = load_entries(row1 + (size_t)r * row_step);
                    }
                }
            }
            fill_near();        // while the rows are on their way
#pragma unroll
            for (int b = 0; b < kBatches; ++b) {
                if (4 * b < rows) {
                    const int r = 4 * b + g;
                    const bool live = in_row16 && r < rows;
                    const int4 w = kept(v[b]);
                    const int part = (w.x + w.y) + (w.z + w.w);
                    const int positive = (w.x > 0 ? 1 : 0) + (w.y > 0 ? 1 : 0) + (w.z > 0 ? 1 : 0) + (w.w > 0 ? 1 : 0);
                    const int differs = ((w.x != curg.x) | (w.y != curg.y) | (w.z != curg.z) | (w.w != curg.w)) ? 1 : 0;
                    const int negative = ((w.x | w.y | w.z | w.w) < 0) ? 1 : 0;
                    // one word carries three small counts: positive entries (at most 64), lanes that differ, lanes with a negative entry
                    const int counts = row16_sum(live ? positive | (differs << 12) | (negative << 20) : 0);
                    const int K = row16_sum(live ? part : 0);
                    const int nodes = counts & 0xFFF;
                    kb[b] = K;
                    mb[b] = nodes | (((counts >> 12) & 0xFF) != 0 ? kMetaChanged : 0);
                    any_neg |= __ballot(live && (counts >> 20) != 0) != 0ull;
                    if (a.need_constraints && live) {
                        // every non-zero entry goes to the candidate's per-node counters (a negative one as it is)
                        const unsigned long long one_job = nodes >= 2 ? kPackJob : 0ull;
                        unsigned long long *__restrict__ to = SEL != 0 ? a.colpack + (size_t)cb[b] * a.N + at16
                                                                  : cp1 + (size_t)r * kWavesPerBlock * a.N;
                        if (w.x != 0) atomicAdd(&to[0], (unsigned long long)(long long)w.x + (w.x > 0 ? one_job : 0ull));
                        if (w.y != 0) atomicAdd(&to[1], (unsigned long long)(long long)w.y + (w.y > 0 ? one_job : 0ull));
                        if (w.z != 0) atomicAdd(&to[2], (unsigned long long)(long long)w.z + (w.z > 0 ? one_job : 0ull));
                        if (w.w != 0) atomicAdd(&to[3], (unsigned long long)(long long)w.w + (w.w > 0 ? one_job : 0ull));
                    }
                }
            }
            // lane r takes over what candidate r needs: from lane 16 (r mod 4) of batch r / 4
#pragma unroll
            for (int b = 0; b < kBatches; ++b) {
                const int from = ((lane & 3) * 16) << 2;
                const int K = __builtin_amdgcn_ds_bpermute(from, kb[b]), meta = __builtin_amdgcn_ds_bpermute(from, mb[b]);
                if ((lane >> 2) == b) {
                    d_K = K;
                    d_meta = meta;
                }
            }
        } else if constexpr (ROW1) {
            // eight rows are requested together: their latencies overlap.  The last eight come first: a stretch leaves
            // what its candidates need in lanes 0 .. 7, and the lanes move up by eight before the next stretch
            constexpr int kAhead = 8;
            static_assert(kMaxCandPerWave <= 2 * kAhead, "two stretches at most (the lanes move inside a row of 16)");
            const int r_last = (rows - 1) & ~(kAhead - 1);
            int at_row = -1;          // the candidate (of this wavefront) that `row` and `cp` point at
            int4 v[kAhead];
            const int32_t *__restrict__ row_first = row + row_step;       // the row of the wavefront's candidate 0 (SEL == 0)
            auto request = [&](int r, int4 &to) {
                const int ru = r < rows ? r : rows - 1;                   // the tail reads the last row again
                if constexpr (SEL != 0) to = load_entries(row_of(ru));
                else to = load_entries(row_first + (size_t)ru * row_step);
            };
            // the rows of the first stretch are on their way while the workgroup fills its table in LDS
            if (r_last >= 0) {
#pragma unroll
                for (int u = 0; u < kAhead; ++u) request(r_last + u, v[u]);
            }
            fill_near();
            // One stretch; with hand_on the registers of its rows are handed on to the rows of the stretch below it, two
            // at a time.  (Written out once per stretch instead of as a loop, so that every wait names the loads it needs.)
            auto stretch = [&](int r0, auto hand_on) {
                if constexpr (SEL == 0) {
                    // advance() steps from one candidate to the next: start one before the stretch
                    const ptrdiff_t step = r0 - 1 - at_row;
                    row += step * (ptrdiff_t)row_step;
                    cp += step * (ptrdiff_t)kWavesPerBlock * a.N;
                    at_row = (r0 + kAhead < rows ? r0 + kAhead : rows) - 1;
                }
                // The sums of two rows come out of one reduction, 16 bits each, when every entry of both lies in
                // 0 .. 255 (a row of 256 such entries sums to less than 2^16), which the rows of any valid
                // population do; otherwise each row is summed on its own.
#pragma unroll
                for (int u = 0; u < kAhead; u += 2) {
                    if (r0 + u < rows) {
                        if constexpr (RAG) {
                            v[u] = kept(v[u]);
                            v[u + 1] = kept(v[u + 1]);
                        }
                        const int4 &va = v[u], &vb = v[u + 1];
                        int wide = (__ballot((unsigned)(((va.x | va.y) | (va.z | va.w)) | ((vb.x | vb.y) | (vb.z | vb.w))) > 255u) & in_row) != 0 ? 1 : 0;
                        wide = __builtin_amdgcn_readfirstlane(wide);
                        asm volatile("" : "+s"(wide));
                        const int part_a = lane < n4 ? (va.x + va.y) + (va.z + va.w) : 0;
                        const int part_b = lane < n4 ? (vb.x + vb.y) + (vb.z + vb.w) : 0;
                        int K2[2];
                        if (wide == 0) {
                            const int both = wave_sum(part_a + (part_b << 16));
                            K2[0] = both & 0xFFFF;
                            K2[1] = (int)((unsigned)both >> 16);
                        } else {
                            K2[0] = wave_sum(part_a);
                            K2[1] = wave_sum(part_b);
                        }
#pragma unroll
                        for (int e = 0; e < 2; ++e) {
                            if (r0 + u + e < rows) {
                                int K, nodes;
                                bool changed, neg;
                                advance(r0 + u + e);
                                row_stage(K, nodes, changed, neg, &v[u + e], &K2[e], wide ^ 1);
                                // lane r keeps what candidate r needs (see above)
                                d_K = write_lane8(d_K, K, u + e);
                                d_meta = write_lane8(d_meta, nodes | (changed ? kMetaChanged : 0), u + e);
                                any_neg |= neg;
                            }
                        }
                    }
                    // the rows of the next stretch take the registers this pair has left: they are on their way
                    // while the rest of this stretch is worked on
                    if constexpr (decltype(hand_on)::value) {
                        request(r0 - kAhead + u, v[u]);
                        request(r0 - kAhead + u + 1, v[u + 1]);
                    }
                }
            };
            if (r_last >= kAhead) {
                stretch(r_last, std::true_type());
                // (write_lane is an opaque statement: the two wait states a DPP read needs after a vector write of its
                // source are put here by hand, whatever the compiler schedules in between)
                asm volatile("s_nop 1" : "+v"(d_K), "+v"(d_meta));
                d_K = row16_up8(d_K);
                d_meta = row16_up8(d_meta);
            }
            if (r_last >= 0) stretch(0, std::false_type());
        } else {
            for (int r = 0; r < rows; ++r) {
                int K, nodes;
                bool changed, neg;
                advance(r);
                row_stage(K, nodes, changed, neg);
                if (lane == r) {
                    d_K = K;
                    d_meta = nodes | (changed ? kMetaChanged : 0);
                }
                any_neg |= neg;
            }
        }
        if constexpr (kStage) {
            if (stage_on) {
                // Which rows to stage: every pair of the workgroup votes for the row it will read, and every
                // wavefront takes, from the same counts (so all four agree), the rows with two votes or more: those
                // of the "one node" class first, fewer GPUs first, which is where allocations concentrate.  Lane r
                // then notes where its candidate's row is staged (-1: not staged).
                const int my_nodes = d_meta & ~kMetaChanged;
                const bool votes = lane < rows && d_K >= 1 && tabled_row(d_K, my_nodes == 1, tb.k1);
                const int my_row = (my_nodes == 1 ? kTableK : 0) + d_K - 1;
                if (votes) atomicAdd(&stage_votes[my_row], 1);
                __syncthreads();
                unsigned long long several = __ballot(stage_votes[lane] >= 2), one = __ballot(stage_votes[lane + kWave] >= 2);
                int staged[kStageRows];
                const int t = threadIdx.x;
                double2 ca_in[kStageRows];
                int range_in[kStageRows];
                double2 tg_in = {0.0, 0.0};
                if (t < a.Gm) tg_in = tb.tg[t];
                // lanes past the end of a grid that is no whole group of 64 find a batch size without a feasible count
                const int whole_gm = WHOLE ? a.Gm : (a.Gm <= kWave ? kWave : kStageGm);
#pragma unroll
                for (int e = 0; e < kStageRows; ++e) {
                    staged[e] = -1;
                    ca_in[e] = double2{0.0, __builtin_inf()};
                    range_in[e] = 0;
                    if (one != 0ull) {
                        staged[e] = kTableK + __builtin_ctzll(one);
                        one &= one - 1ull;
                    } else if (several != 0ull) {
                        staged[e] = __builtin_ctzll(several);
                        several &= several - 1ull;
                    }
                    if (staged[e] >= 0) {
                        // threads 0 .. Gm-1 bring the (C, A0) pairs of the row, as many from whole_gm on its feasible ranges
                        if (t < a.Gm) ca_in[e] = tb.ca[(size_t)staged[e] * a.Gm + t];
                        else if (t >= whole_gm && t < whole_gm + a.Gm) range_in[e] = tb.srange[(size_t)(staged[e] & (kTableK - 1)) * a.Gm + (t - whole_gm)];
                        if (votes && my_row == staged[e]) d_row = kStageBase + 2 * kStageGm + e * kStageRowDoubles;
                    }
                }
                if (t < whole_gm) {
                    r_lds[kStageBase + 2 * t] = tg_in.x;
                    r_lds[kStageBase + 2 * t + 1] = tg_in.y;
                }
#pragma unroll
                for (int e = 0; e < kStageRows; ++e) {
                    if (staged[e] >= 0) {
                        double *row_lds = r_lds + kStageBase + 2 * kStageGm + e * kStageRowDoubles;
                        if (t < whole_gm) {
                            row_lds[2 * t] = ca_in[e].x;
                            row_lds[2 * t + 1] = ca_in[e].y;
                        } else if (t < 2 * whole_gm) {
                            ((int *)(row_lds + 2 * kStageGm))[t - whole_gm] = range_in[e];
                        }
                    }
                }
                __syncthreads();
            }
        }
        // after the row pass, whose rows in flight use the registers these occupy
        if constexpr (F32) XF = make_run_steps_f32();
        else X = make_run_steps();
        int sweep_lane = lane;
        asm volatile("" : "+v"(sweep_lane));
        // Short rows come with small grids: there the sweeps go four candidates at a time, one per row of 16 lanes.
        constexpr bool kRows = rows_at_a_time(ROW4);
        if constexpr (kRows) {
            // Lane r holds K and nodes of candidate r.  A sweep lasts as long with empty rows as with others: where it saves a
            // sweep, the rows that want one (not those beyond the tables, swept after the loop, either) move up to the first slots.
            const bool one = (d_meta & ~kMetaChanged) == 1, tabled = tabled_row(d_K, one, tb.k1);
            const bool wanted = lane < rows && d_K >= 1 && tabled;
            const unsigned live = (unsigned)__ballot(wanted);
            const int live_sweeps = (__builtin_popcount(live) + 3) >> 2;
            const bool packed = live_sweeps < ((rows + 3) >> 2);
            const int sweeps = packed ? live_sweeps : (rows + 3) >> 2;
            int in_slot = wanted ? d_K | (one ? 1 << 8 : 0) : 0, found_in_slot = -1;
            const int slot = wanted ? __builtin_popcount(live & ((1u << (lane & 15)) - 1u)) : kWave - 1;
            if (packed) in_slot = __builtin_amdgcn_ds_permute(slot << 2, in_slot);
            for (int b = 0; b < sweeps; ++b) {
                // this lane's row works on slot 4 b + (its number)
                const int K_one = __builtin_amdgcn_ds_bpermute((4 * b + (lane >> 4)) << 2, in_slot);
                const int K = K_one & 0xFF, K_in = K < 1 ? 1 : K;
                const bool one_node = (K_one >> 8) != 0;
                // (this instance is launched only for grids whose tables of reciprocals and thresholds fit LDS)
                int found;
                if constexpr (F32) found = sweep_pick_rows_f32<CH, WHOLE>(qf, tb, XF, a.rsf, a.Gm, a.Gs, K_in, one_node, (LdsFloats)(const float *)r_lds, WHOLE || has_near);
                else found = sweep_pick_rows<CH, WHOLE>(tb, X, a.rs, a.Gm, a.Gs, K_in, one_node, (LdsDoubles)r_lds, WHOLE || has_near);
                found = K < 1 ? -1 : found;
                // lane 4 b + g takes over what row g has found
                const int taken = __builtin_amdgcn_ds_bpermute(((lane & 3) * 16) << 2, found);
                if ((lane >> 2) == b) found_in_slot = taken;
            }
            d_i = packed ? __builtin_amdgcn_ds_bpermute(slot << 2, found_in_slot) : found_in_slot;
            if (lane < rows && d_K >= 1 && !tabled) d_i = kPending;
        }
        for (int r = 0; !kRows && r < rows; ++r) {
            const int K = __builtin_amdgcn_readlane(d_K, r);
            const int nodes = __builtin_amdgcn_readlane(d_meta, r) & ~kMetaChanged;
            int pick = -1;
            if (K >= 1 && !tabled_row(K, nodes == 1, tb.k1)) pick = kPending;   // rare: swept after the loop, outside the hot path
            else if (!MEMO && K >= 1) {
                if constexpr (F32) pick = sweep_pick_f32<CH, WHOLE>(qf, tb, XF, a.rsf, a.Gm, a.Gs, K, nodes, (LdsFloats)(const float *)r_lds, has_near);
                else pick = sweep_pick<CH, WHOLE, kStage>(sweep_lane, tb, X, a.rs, a.Gm, a.Gs, K, nodes, (LdsDoubles)r_lds, has_near,
                                                          kStage ? __builtin_amdgcn_readlane(d_row, r) : -1);
            }
            if (lane == r) d_i = pick;
        }
    } else {
        // the sampling argmax: one candidate after the other, priced where it is swept
        for (int r = 0; r < a.cand_per_wave; ++r) {
            if (c0 + kWavesPerBlock * r >= P_eff) break;
            const int c = SEL != 0 ? __builtin_amdgcn_readlane(d_c, r) : c0 + kWavesPerBlock * r;
            int K, nodes;
            bool changed, neg;
            advance(r);
            row_stage(K, nodes, changed, neg);
            Best best;
            if (MEMO && K >= 1 && tabled_row(K, nodes == 1, tb.k1)) {
                const MemoEntry e = a.memo[((size_t)j * 2 + (nodes == 1 ? 1 : 0)) * kTableK + (K - 1)];
                best.goodput = e.goodput; best.m = e.m; best.s = e.s;
            } else {
                best = sweep_sampled<MEMO>(q, tb.m, a.Gm, a.Gs, K, nodes);
            }
            if (lane == 0) {
                const size_t pair = (size_t)c * a.J + j;
                a.G[pair] = best.goodput;
                a.meta[pair] = nodes | (changed ? kMetaChanged : 0);
                if (a.best_m) {
                    a.best_m[pair] = best.m;
                    a.best_s[pair] = best.s;
                }
                if (a.best_goodput) a.best_goodput[pair] = best.goodput;
                if (neg) atomicOr(a.status, PX_ST_NEG_ALLOC);
            }
        }
    }

    if constexpr (kDeferred) {
        // What follows needs pointers the loop above never touches (outputs, the tables of the
        // untabled path).  They are read from the kernel-argument segment again here, behind a
        // volatile statement, instead of occupying scalar registers throughout the loop.
        typedef const FitnessArgs __attribute__((address_space(4))) *KernelArgs;
        KernelArgs again = (KernelArgs)__builtin_amdgcn_kernarg_segment_ptr();
        asm volatile("" : "+s"(again));
        const FitnessArgs b = *(const FitnessArgs *)again;
        const Job qb = load_job(b.job_params, b.J, j);
        const JobTables tbb = job_tables(b, j);

        // sweeps whose scan has left several batch sizes
        if constexpr (!MEMO) {
            unsigned long long close = __ballot(d_i == kClose);
            int settle_lane = lane;
            asm volatile("" : "+v"(settle_lane));          // (its addresses are formed here, not kept from the start on)
            while (close) {
                const int l0 = __ffsll(close) - 1;
                close &= close - 1;
                if constexpr (F32) {
                    const int i = settle_f32(settle_lane, qf, tbb, b.rsf, b.Gm, b.Gs, __builtin_amdgcn_readlane(d_K, l0),
                                             (__builtin_amdgcn_readlane(d_meta, l0) & ~kMetaChanged) == 1);
                    if (lane == l0) d_i = i;
                    continue;
                }
                const int l1 = close != 0ull ? __ffsll(close) - 1 : l0;
                close &= close - 1;
                const int K[2] = {__builtin_amdgcn_readlane(d_K, l0), __builtin_amdgcn_readlane(d_K, l1)};
                const bool one_node[2] = {(__builtin_amdgcn_readlane(d_meta, l0) & ~kMetaChanged) == 1,
                                          (__builtin_amdgcn_readlane(d_meta, l1) & ~kMetaChanged) == 1};
                int picked[2];
                settle(picked, settle_lane, tbb, b.rs, (LdsDoubles)r_lds, b.gs_pad <= kNearRecips, b.Gm, b.Gs, K, one_node);
                d_i = lane == l0 ? picked[0] : (lane == l1 ? picked[1] : d_i);
            }
        }
        // rows with more GPUs than the tables cover: the whole wavefront sweeps and prices them one by one
        Best beyond = {0.0, -1, -1};
        unsigned long long pending = __ballot(d_i == kPending);
        while (pending) {
            const int l = __ffsll(pending) - 1;
            pending &= pending - 1;
            const int K = __builtin_amdgcn_readlane(d_K, l);
            const int nodes = __builtin_amdgcn_readlane(d_meta, l) & ~kMetaChanged;
            Best found;
            if constexpr (F32) {
                found = sweep_f32(qf, tbb, b.rk, b.Gm, b.Gs, K, nodes);
            } else if constexpr (MEMO) {
                found = row_best_plain<true>(qb, load_grid_params(b.job_params, b.J, j), tbb.m, b.Gm, b.Gs, K, nodes == 1, false);
            } else {
                const Pick pick = sweep_pick_beyond<CH>(qb, tbb, b.rs, b.rk, b.Gm, b.Gs, K, nodes);
                found = price_beyond(qb, tbb, K, nodes == 1, pick.i, pick.s);
            }
            if (lane == l) {
                beyond = found;
                d_i = kPriced;
            }
        }
        // Lane l finishes the l-th candidate of this wavefront: the elected point is priced with
        // Eq. 4 in the paper's order of operations (or looked up in memoised mode) and stored.
        const int k = (group * b.cand_per_wave + lane) * kWavesPerBlock + wave;
        if (lane < b.cand_per_wave && k < (SEL == 2 ? P_eff : (SEL == 1 ? b.n_sel : b.P))) {
            const int c = SEL != 0 ? d_c : k;
            const size_t pair = (size_t)c * b.J + j;
            const int nodes = d_meta & ~kMetaChanged;
            Best best;
            if (MEMO && d_K >= 1 && tabled_row(d_K, nodes == 1, tbb.k1)) {
                const MemoEntry e = b.memo[((size_t)j * 2 + (nodes == 1 ? 1 : 0)) * kTableK + (d_K - 1)];
                best.goodput = e.goodput; best.m = e.m; best.s = e.s;
            } else if (d_i == kPriced) {
                best = beyond;
            } else if constexpr (F32) {
                best = price_point_f32(qf, tbb, b.Gm, d_K, nodes == 1, d_i);
            } else {
                best = price_tabled(qb, tbb, b.Gm, d_K, nodes == 1, d_i);
            }
            b.G[pair] = best.goodput;
            b.meta[pair] = d_meta;
            if (b.best_m) {
                b.best_m[pair] = best.m;
                b.best_s[pair] = best.s;
            }
            if (b.best_goodput) b.best_goodput[pair] = best.goodput;
        }
        if (any_neg && lane == 0) atomicOr(b.status, PX_ST_NEG_ALLOC);
    }
}

// ---- the argmax alone, for the consumers outside the search ----------------------------
// One wavefront per query (job, K, nodes), found in place (row_best; many at once in queries_rows_kernel): the job tables would cost a call 72 rows per job
// where it asks for one (or max_nodes + 1), and two launches (200 jobs, 17 queries each: 28 us with them).
//   per_gpu mode   query (j, n), n = 0..max_nodes: column 0 is the job on one GPU, column n >= 1
//                  the job on n full nodes of gpus_per_node GPUs; the goodput is divided by the
//                  GPUs held (auto-scaling rule of Sec. 5.3.3)
//   tick mode      query j: the job at its current (K, nodes); its progress advances by
//                  goodput x (dt - restart delay if its allocation was changed) (Sec. 5.3)
struct QueryArgs {
    int mode;                       // 0 per_gpu, 1 tick
    int gpus_per_node, max_nodes;
    double *per_gpu;                // [J, max_nodes + 1]
    const int32_t *K, *nodes, *changed;
    const double *target;
    double dt, restart_delay;
    double *progress, *goodput;
    int32_t *finished;
};

__global__ void __launch_bounds__(256) queries_kernel(FitnessArgs a, QueryArgs q)
{
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const long long id = (long long)blockIdx.x * kWavesPerBlock + wave;
    const int per_job = q.mode == 0 ? q.max_nodes + 1 : 1;
    if (id >= (long long)a.J * per_job) return;
    const int j = (int)(id / per_job), n = (int)(id % per_job);
    int K, nodes;
    if (q.mode == 0) {
        K = n == 0 ? 1 : n * q.gpus_per_node;
        nodes = n == 0 ? 1 : n;
    } else {
        K = q.K[j];
        nodes = q.nodes[j];
        if (!(q.progress[j] < q.target[j])) K = 0;              // a finished job is left as it is
    }
    // (the parameters all together: one trip to memory)
    const Job job = load_job(a.job_params, a.J, j);
    const GridParams gp = load_grid_params(a.job_params, a.J, j);
    const SyncParams y = load_sync(job);
    K = __builtin_amdgcn_readfirstlane(K);             // one query per wavefront: the same in every lane
    nodes = __builtin_amdgcn_readfirstlane(nodes);
    Best best = {0.0, -1, -1};
    if (K > 0)
        best = row_best(held_coefs(), job, gp, y, a.m_grid + (size_t)j * a.Gm, a.Gm, a.Gs, K, nodes == 1, K <= kTableK);
    if (lane_id() != 0) return;
    if (q.mode == 0) {
        q.per_gpu[id] = best.goodput / (double)K;
    } else {
        const double before = q.progress[j];
        const double run = q.dt - (q.changed[j] ? q.restart_delay : 0.0);
        const double after = (K > 0 && run > 0.0) ? before + best.goodput * run : before;
        q.goodput[j] = best.goodput;
        q.progress[j] = after;
        q.finished[j] = after >= q.target[j];
    }
}

// The same for many queries (per_gpu mode): `rows` of one job to a wavefront (query_rows), which share the terms of its batch sizes.
__global__ void __launch_bounds__(256) queries_rows_kernel(FitnessArgs a, QueryArgs q, int rows)
{
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)), lane = lane_id();
    const int per_job = q.max_nodes + 1, waves = (per_job + rows - 1) / rows;
    const long long id = (long long)blockIdx.x * kWavesPerBlock + wave;
    if (id >= (long long)a.J * waves) return;
    const int j = (int)(id / waves), n0 = (int)(id % waves) * rows;
    const Job job = load_job(a.job_params, a.J, j);
    const GridParams gp = load_grid_params(a.job_params, a.J, j);
    const SyncParams y = load_sync(job);
    const int mine = per_job - n0 < rows ? per_job - n0 : rows;
    const int n = n0 + (lane < mine ? lane : 0), K = n == 0 ? 1 : n * q.gpus_per_node;
    const Coefs c = held_coefs();
    const Best best = argmax_rows(c, job, gp, a.m_grid + (size_t)j * a.Gm, a.Gm, a.Gs, mine, K, sync_term(c, y, K, n <= 1), 1.0 / (double)K,
                                  K <= kTableK);
    if (lane < mine) q.per_gpu[(size_t)j * per_job + n] = best.goodput / (double)K;
}

// Sec. 5.3.3: a job scales up when its goodput per GPU exceeds U of the ideal (one GPU, column 0), to the
// node count reached by adding nodes while the next count still predicts at least L of the ideal per GPU.
__global__ void __launch_bounds__(256) autoscale_kernel(int J, int max_nodes, const double *__restrict__ per_gpu,
                                                       const int32_t *__restrict__ nodes_now, double U, double L,
                                                       int32_t *__restrict__ nodes_new)
{
    const int j = blockIdx.x * blockDim.x + threadIdx.x;
    if (j >= J) return;
    const double *__restrict__ row = per_gpu + (size_t)j * (max_nodes + 1);
    int n = nodes_now[j];
    if (n >= 1 && n <= max_nodes && row[n] > U * row[0]) {
        while (n < max_nodes && row[n + 1] >= L * row[0]) ++n;
    }
    nodes_new[j] = n;
}

// ---- per candidate -------------------------------------------------------------

constexpr int kCandThreads = 256;

// The last six levels of that tree, across the lanes of a wavefront; lane 0 holds the sum.
template <typename T>
__device__ __forceinline__ T wave_tree_sum(T s)
{
    s += exchange<5>(s);                     // lane ^ 32
    s += exchange<4>(s);                     // lane ^ 16
    s += rotate16<8>(s);                     // lane ^ 8, and from here on lanes 2^k apart hold the same
    s += rotate16<4>(s);
    s += rotate16<2>(s);
    s += rotate16<1>(s);
    return s;
}

// The sum of red[0 .. kCandThreads-1] in lane 0 of the first wavefront, which alone calls this: the tree that adds the upper half
// to the lower one again and again, its last six levels across lanes (a barrier per level took 0.6 us of a 5 us kernel).
template <typename T>
__device__ __forceinline__ T tree_sum(const T *red)
{
    static_assert(kCandThreads == 4 * kWave, "two levels before one wavefront holds the rest");
    const int l = lane_id();
    return wave_tree_sum((red[l] + red[l + 2 * kWave]) + (red[l + kWave] + red[l + 3 * kWave]));
}

// (the powers behind everything else: their code is long, and a kernel of a few microseconds waits for every line it has to fetch)
__device__ __forceinline__ double pmean_term(double s, double w, double p)
{
    if (__builtin_expect(p == -1.0, 1)) return w * (1.0 / s);  // 1/0 = +inf, as pow(0, -1)
    if (__builtin_expect(p == 1.0, 1)) return w * s;
    if (__builtin_expect(p == 0.0, 0)) return w * log(s);      // log(0) = -inf
    return w * pow(s, p);                                      // pow(0, p<0) = +inf
}

__device__ __forceinline__ float pmean_term(float s, float w, float p)
{
    if (p == 0.0f) return w * logf(s);
    return w * powf(s, p);
}

__device__ __forceinline__ double pmean_finish(double mean, double p)
{
    if (__builtin_expect(p == -1.0, 1)) return 1.0 / mean;
    if (__builtin_expect(p == 1.0, 1)) return mean;
    if (__builtin_expect(p == 0.0, 0)) return exp(mean);
    return pow(mean, 1.0 / p);
}
__device__ __forceinline__ float pmean_finish(float mean, float p) { return p == 0.0f ? expf(mean) : powf(mean, 1.0f / p); }

// The status bits prepare_kernel has left per job go into the status word here: that kernel also clears the word, so no
// wavefront of it may add to it.  Called by one workgroup of the call's last kernel.
__device__ __forceinline__ void or_job_status(const FitnessArgs &a)
{
    int st = 0;
    for (int j = threadIdx.x; j < a.J; j += blockDim.x) st |= a.jobstat[j];
    if (st) atomicOr(a.status, st);
}

// REAL = double, or float for the fp32 variant (SPEEDUP, the penalty and the mean are then formed in fp32).
// JOBS: how many of its jobs a thread asks for together.  One after the other, each waits for its own trip to memory: 4096
// candidates of 1000 jobs 26.7 us, four together 18.8; 1021 of 331 7.4, 7.0.  Up to 256 jobs a thread has one, and the code of four costs
// what a launch of 5 us waits to fetch it (1000 of 200 4.7, 5.2).
template <typename REAL, int JOBS>
__global__ void __launch_bounds__(kCandThreads) candidates_kernel(FitnessArgs a)
{
    __shared__ REAL red_acc[kCandThreads];
    __shared__ REAL red_w[kCandThreads];
    __shared__ long long red_v[kCandThreads];
    const int c = a.sel ? a.sel[blockIdx.x] : (int)blockIdx.x;
    const int t = threadIdx.x;
    const double *__restrict__ G = a.G + (size_t)c * a.J;
    const int32_t *__restrict__ meta = a.meta + (size_t)c * a.J;
    const double *__restrict__ wt = a.job_params + (size_t)PX_WEIGHT * a.J;

    if (a.or_job_status && blockIdx.x == 0) or_job_status(a);
    // SPEEDUP (Eq. 15) with the re-allocation penalty, then the generalized mean (Eq. 14):
    // each thread sums its jobs in ascending order, then a fixed tree
    REAL acc = 0, wsum = 0;
    const REAL p = (REAL)a.p;
    for (int j0 = t; j0 < a.J; j0 += JOBS * kCandThreads) {
        double g[JOBS], d[JOBS], f[JOBS], w[JOBS];
        int m[JOBS];
#pragma unroll
        for (int u = 0; u < JOBS; ++u) {
            const int j = j0 + u * kCandThreads < a.J ? j0 + u * kCandThreads : j0;
            g[u] = G[j];
            m[u] = meta[j];
            d[u] = a.denom[j];
            f[u] = a.factor[j];
            w[u] = wt[j];
        }
#pragma unroll
        for (int u = 0; u < JOBS; ++u) {
            const int j = j0 + u * kCandThreads;
            if (j < a.J) {
                REAL s_j = (REAL)d[u] > 0 ? (REAL)g[u] / (REAL)d[u] : (REAL)0;
                if (m[u] & kMetaChanged) s_j = s_j * (REAL)f[u];
                if (a.speedup) a.speedup[(size_t)c * a.J + j] = (double)s_j;
                acc += pmean_term(s_j, (REAL)w[u], p);
                wsum += (REAL)w[u];
            }
        }
    }
    red_acc[t] = acc;
    red_w[t] = wsum;

    // constraint check, part two: per node, multi-node jobs beyond the first and GPUs beyond capacity
    long long v = 0;
    if (a.need_constraints) {
        // the counters are left at zero for the next call on this workspace (see launch_fitness)
        unsigned long long *__restrict__ cp = a.colpack + (size_t)c * a.N;
        for (int n = t; n < a.N; n += kCandThreads) {
            const long long x = (long long)cp[n];
            cp[n] = 0ull;
            const long long asked = (x << 24) >> 24;              // low 40 bits, sign-extended
            const long long distributed = (x - asked) >> 40;
            if (distributed > 1) v += distributed - 1;
            const long long over = asked - (long long)a.node_capacity[n];
            if (over > 0) v += over;
        }
    }
    red_v[t] = v;
    __syncthreads();
    if (t >= kWave) return;
    const REAL total = tree_sum(red_acc), weight = tree_sum(red_w);
    const long long V = tree_sum(red_v);
    if (t == 0) {
        const REAL mean = total / weight;
        double f = (double)pmean_finish(mean, (REAL)a.p);
        if (a.violations) a.violations[c] = (int32_t)(V > 0x7FFFFFFF ? 0x7FFFFFFF : V);
        if (V > 0 && !(a.flags & PX_FLAG_NO_CONSTRAINT_CHECK)) f = -(double)V;
        a.fitness[c] = f;
    }
}

// ---- small calls: one launch -----------------------------------------------------------------------
// A few hundred candidates of a dozen jobs are less work than the tables their sweeps would share (72 rows a job), and the call
// lasts as long as its launches follow one another: three of 5 to 7 us each.  Here one workgroup takes a candidate: it finds the
// jobs' fair-share goodputs and reduces, elects and prices the candidate's rows, forming the terms of the batch sizes itself; the
// best count of each follows from its C as for fair shares (px_best_count), so rows, shares and memoised rows are one arithmetic.
// The node counters are in LDS, and the first wavefront forms SPEEDUP and the mean, term by term and in the tree of
// candidates_kernel.  The same results, bit by bit.  Sixteen wavefronts share the tasks out (row_best); with at most 32 batch sizes
// there are 4 to 16, which take two tasks each, a half of the lanes for one (half_best).  A call that starts anew leaves its fair
// shares and re-allocation factors in the workspace, beside the status section; one that keeps the job tables (the children of a
// generation are such) takes them from there.
// (With a scan over all counts for the rows a kept call of 4 jobs, 100 x 32, took 7.1 to 7.5 us, 6.0 so; 14 jobs, 64 x 8, 7.9 to 8.3, 7.3.)
// The line (small_call) is drawn where a wavefront has two rows of 64 batch sizes to take, fair shares included.  us a call here and
// in three launches, 16 candidates: 8 jobs, 64 x 16, 8.5, 14.9, 12 jobs 10.0, 14.9, 16 jobs 12.4, 14.9 (200 candidates 12.4, 17.6),
// 64 x 32 12.5, 18.2; 8 jobs, 128 x 16, 10.0, 16.9; 16 jobs, 32 x 32, 10.0, 15.3; one job, 512 x 16, 10.1, 27.  Keeping their tables,
// two launches on the other side: 6.7, 8.8; 6.9, 8.7; 7.4, 8.7 (7.5, 11.5), 7.4, 11.9; 7.0, 9.6; 6.7, 8.9; 9.3, 14.2.  Long grids are groups
// of 64 one after the other, so the line lies at sixteen groups over all jobs, eight with more than 16 counts.  The status section
// holds a byte per candidate.
constexpr int kSmallThreads = 1024;
constexpr int kSmallJobs = 16;
constexpr int kSmallCandidates = 4 * (kStatusWords - 1);

static bool small_call(const pollux_dims &d)
{
    const int groups = (d.Gm + kWave - 1) / kWave;             // of 64 batch sizes, a row
    return d.precision == 0 && (d.flags & (PX_FLAG_MEMOISE | PX_FLAG_SAMPLE_M)) == 0 && d.P <= kSmallCandidates && d.J <= kSmallJobs &&
           d.N >= 4 && d.N <= 4 * kWave && d.Gs <= kSmallGs &&
           d.J * groups <= kSmallJobs && (d.Gs <= 16 || groups <= 8);
}

// Threads of a workgroup: sixteen wavefronts, one task each, fair shares before rows; or, with at most 32 batch sizes, one wavefront for
// two tasks (small_kernel's HALVES), and four at least.
constexpr int kSmallHalf = kWave / 2;
static int small_threads(const pollux_dims &d, bool kept)
{
    if (d.Gm > kSmallHalf) return kSmallThreads;
    const int waves = kept ? (d.J + 1) / 2 : d.J;
    return kWave * (waves > 4 ? waves : 4);
}

// Smallest value among the lane's half of the wavefront, in every lane of that half.
__device__ __forceinline__ unsigned half_min(unsigned v)
{
    v = row16_min(v);
    const unsigned other = (unsigned)exchange<4>((int)v);            // the half's other row of 16
    return v < other ? v : other;
}

// The argmax of two (job, K, placement) at once, one per half of the wavefront, for grids of at most 32 batch sizes; each lane's
// arguments are its half's.  The lane that holds the elected point (the half's first where there is none) returns it in `best`
// and is told so.  The same point as row_best finds, the same bits.
__device__ __forceinline__ bool half_best(const Coefs &c, const Job &q, const GridParams &gp, const SyncParams &y, int m, bool in_grid,
                                          int Gs, int K, bool one_node, bool tabled, Best &best)
{
    SyncTerm st = sync_term(c, y, K, one_node);
    const GridPoint g = grid_point(c, gp, m);
    const double last = last_pass(c, st, g.tg, g.lntg);
    int s;
    double h = best_count(g, row_terms(g, last, 1.0 / (double)K, Gs), tabled, s);
    h = in_grid && h < __builtin_inf() ? h : __builtin_inf();
    const unsigned hi = (unsigned)__double2hiint(h), lo = (unsigned)__double2loint(h);
    const unsigned hmin = half_min(hi);
    const unsigned lmin = half_min(hi == hmin ? lo : 0xFFFFFFFFu);
    const unsigned lane = (unsigned)lane_id() & (kSmallHalf - 1);
    const unsigned first = half_min(hi == hmin && lo == lmin ? lane : 0xFFu);      // equal values: the lowest batch size
    best = Best{0.0, -1, -1};
    if (hmin < 0x7FF00000u) best = Best{goodput_point(q, (double)K * (double)m, g.tg, last, s), m, s};
    return lane == first;
}

// KEPT: the call keeps the job tables.  HALVES: at most 32 batch sizes.  A wavefront would leave half its lanes idle with one task, and
// sixteen of them share four SIMDs whose issue bounds them (8 jobs, 32 x 8: 13000 of the workgroup's 19400 cycles, with a scan of the
// counts in each), so a wavefront takes a job's fair share and its row together, a half each, or two rows where the fair shares are
// kept.  The rows are reduced first, a wavefront each.  Calls, us, with a wavefront a task and so, both with that scan, and so without it:
// 16 candidates of 8 jobs, 32 x 8, 8.7, 7.8, 7.1; 200 of 16 jobs, 32 x 32, 13.5, 10.8, 9.9; 16 of 16 on 200 nodes 14.0, 10.8, 10.3; 250 of 3
// jobs 6.4, 6.6, 6.0.
template <bool KEPT, bool HALVES>
__global__ void __launch_bounds__(kSmallThreads) small_kernel(FitnessArgs a)
{
    __shared__ unsigned long long node_lds[4 * kWave];       // per node: GPUs asked + multi-node jobs << 40, as colpack
    __shared__ double fair_lds[kSmallJobs], factor_lds[kSmallJobs], goodput_lds[kSmallJobs];
    __shared__ int meta_lds[kSmallJobs], m_lds[kSmallJobs], s_lds[kSmallJobs];
    __shared__ int K_lds[HALVES ? kSmallJobs : 1], held_lds[HALVES ? kSmallJobs : 1];
    __shared__ int status_lds, negative;
    const int c = a.sel ? a.sel[blockIdx.x] : (int)blockIdx.x;
    const int t = threadIdx.x, lane = lane_id();
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const Coefs coefs = held_coefs();
    if (t < 4 * kWave) node_lds[t] = 0ull;
    if (t == 0) status_lds = negative = 0;
    // the largest node capacity (rows of the "one node" class beyond it take the form of the untabled sweep)
    const RowLane at_row = row_lane(lane, a.N);
    const Entries caps = *(const Entries *)(a.node_capacity + at_row.base);
    int k1 = caps.x > caps.y ? caps.x : caps.y;
    k1 = k1 > caps.z ? k1 : caps.z;
    k1 = k1 > caps.w ? k1 : caps.w;
    k1 = (int)wave_max((unsigned)(k1 > 0 ? k1 : 0));
    k1 = k1 < kTableK ? k1 : kTableK;
    __syncthreads();
    // (asked for here, so that the trip to memory is over when the first wavefront needs them)
    double kept_fair = 0.0, kept_factor = 1.0;
    if (KEPT && t < a.J) {
        kept_fair = a.denom[t];
        kept_factor = a.factor[t];
    }
    if constexpr (HALVES) {
        // this half's task, and what it needs of memory
        const int half = lane / kSmallHalf, slot = KEPT ? 2 * wave + half : wave;
        const bool is_row = KEPT || half == 1, valid = slot < a.J;
        const int j = valid ? slot : a.J - 1, i = lane & (kSmallHalf - 1);
        const Job q = load_job(a.job_params, a.J, j);
        const GridParams gp = load_grid_params(a.job_params, a.J, j);
        const SyncParams y = load_sync(q);
        const bool in_grid = i < a.Gm;
        const int m = a.m_grid[(size_t)j * a.Gm + (in_grid ? i : a.Gm - 1)];
        int K = 0, fair_nodes = 0;
        double T = 0.0, R = 0.0, weight = 0.0;
        if constexpr (!KEPT) {
            K = a.fair_share[2 * j];
            fair_nodes = a.fair_share[2 * j + 1];
            T = a.job_params[(size_t)PX_AGE_T * a.J + j];
            R = a.job_params[(size_t)PX_RESTARTS_R * a.J + j];
            weight = a.job_params[(size_t)PX_WEIGHT * a.J + j];
        }
        for (int r = wave; r < a.J; r += (int)(blockDim.x / kWave)) {
            const Entries w = *(const Entries *)(a.population + ((size_t)c * a.J + r) * a.N + at_row.base) & at_row.mask;
            const Entries was = *(const Entries *)(a.current_alloc + (size_t)r * a.N + at_row.base) & at_row.mask;
            const int sum = wave_sum((w.x + w.y) + (w.z + w.w));
            const int nodes = __popcll(__ballot(w.x > 0)) + __popcll(__ballot(w.y > 0)) + __popcll(__ballot(w.z > 0)) + __popcll(__ballot(w.w > 0));
            const bool changed = __ballot(((w.x ^ was.x) | (w.y ^ was.y) | (w.z ^ was.z) | (w.w ^ was.w)) != 0) != 0;
            if (__ballot((w.x | w.y | w.z | w.w) < 0) != 0 && lane == 0) negative = 1;
            if ((w.x | w.y | w.z | w.w) != 0) {
                const unsigned long long one_job = nodes >= 2 ? kPackJob : 0ull;
                unsigned long long *to = node_lds + at_row.base;
                atomicAdd(&to[0], (unsigned long long)(long long)w.x + (w.x > 0 ? one_job : 0ull));
                atomicAdd(&to[1], (unsigned long long)(long long)w.y + (w.y > 0 ? one_job : 0ull));
                atomicAdd(&to[2], (unsigned long long)(long long)w.z + (w.z > 0 ? one_job : 0ull));
                atomicAdd(&to[3], (unsigned long long)(long long)w.w + (w.w > 0 ? one_job : 0ull));
            }
            if constexpr (!KEPT) {
                const bool held = wave_sum((long long)was.x + was.y + was.z + was.w) > 0;
                const bool below = __ballot((was.x | was.y | was.z | was.w) < 0) != 0;
                if (lane == 0) held_lds[r] = (held ? 1 : 0) | (below ? 2 : 0);
            }
            if (lane == 0) {
                K_lds[r] = sum;
                meta_lds[r] = nodes | (changed ? kMetaChanged : 0);
            }
        }
        __syncthreads();
        if (is_row) K = K_lds[j];
        const bool one_node = (is_row ? meta_lds[j] & ~kMetaChanged : fair_nodes) == 1;
        const bool wanted = K >= 1;
        Best best;
        const bool mine = half_best(coefs, q, gp, y, m, in_grid, a.Gs, wanted ? K : 1, one_node, !wanted || tabled_row(K, one_node, k1), best);
        if (!wanted) best = Best{0.0, -1, -1};
        if (valid && mine) {
            if (is_row) {
                goodput_lds[j] = best.goodput;
                m_lds[j] = best.m;
                s_lds[j] = best.s;
            } else {
                // the job's fair share, its status and its re-allocation factor (Sec. 4.2)
                const bool penalty = !(a.flags & PX_FLAG_NO_REALLOC_PENALTY);
                int st = job_status(gp, y, weight);
                if (penalty && !(T - R * a.delta > 0.0)) st |= PX_ST_BAD_RESTART;
                if ((held_lds[j] & 2) != 0) st |= PX_ST_NEG_ALLOC;
                if (!(best.goodput > 0.0)) st |= PX_ST_ZERO_FAIR;
                fair_lds[j] = best.goodput;
                factor_lds[j] = penalty && (held_lds[j] & 1) != 0 ? (T - R * a.delta) / (T + a.delta) : 1.0;
                if (st) atomicOr(&status_lds, st);
            }
        }
    }
    const int shares = KEPT ? 0 : a.J;                       // fair shares to find, before the rows
    for (int task = wave; !HALVES && task < shares + a.J; task += kSmallThreads / kWave) {
        const bool is_row = KEPT || task >= shares;
        const int j = is_row ? task - shares : task;
        const Job q = load_job(a.job_params, a.J, j);
        const GridParams gp = load_grid_params(a.job_params, a.J, j);
        const SyncParams y = load_sync(q);
        const int32_t *__restrict__ m_row = a.m_grid + (size_t)j * a.Gm;
        const Entries was = *(const Entries *)(a.current_alloc + (size_t)j * a.N + at_row.base) & at_row.mask;
        if (is_row) {
            const Entries w = *(const Entries *)(a.population + ((size_t)c * a.J + j) * a.N + at_row.base) & at_row.mask;
            const int K = wave_sum((w.x + w.y) + (w.z + w.w));
            const int nodes = __popcll(__ballot(w.x > 0)) + __popcll(__ballot(w.y > 0)) + __popcll(__ballot(w.z > 0)) + __popcll(__ballot(w.w > 0));
            const bool changed = __ballot(((w.x ^ was.x) | (w.y ^ was.y) | (w.z ^ was.z) | (w.w ^ was.w)) != 0) != 0;
            if (__ballot((w.x | w.y | w.z | w.w) < 0) != 0 && lane == 0) negative = 1;
            if ((w.x | w.y | w.z | w.w) != 0) {
                const unsigned long long one_job = nodes >= 2 ? kPackJob : 0ull;
                unsigned long long *to = node_lds + at_row.base;
                atomicAdd(&to[0], (unsigned long long)(long long)w.x + (w.x > 0 ? one_job : 0ull));
                atomicAdd(&to[1], (unsigned long long)(long long)w.y + (w.y > 0 ? one_job : 0ull));
                atomicAdd(&to[2], (unsigned long long)(long long)w.z + (w.z > 0 ? one_job : 0ull));
                atomicAdd(&to[3], (unsigned long long)(long long)w.w + (w.w > 0 ? one_job : 0ull));
            }
            Best best = {0.0, -1, -1};
            if (K >= 1) best = row_best(coefs, q, gp, y, m_row, a.Gm, a.Gs, K, nodes == 1, tabled_row(K, nodes == 1, k1));
            if (lane == 0) {
                goodput_lds[j] = best.goodput;
                meta_lds[j] = nodes | (changed ? kMetaChanged : 0);
                m_lds[j] = best.m;
                s_lds[j] = best.s;
            }
        } else {
            const int K = __builtin_amdgcn_readfirstlane(a.fair_share[2 * j]);
            const bool one_node = __builtin_amdgcn_readfirstlane(a.fair_share[2 * j + 1]) == 1;
            const double T = a.job_params[(size_t)PX_AGE_T * a.J + j], R = a.job_params[(size_t)PX_RESTARTS_R * a.J + j];
            int st = job_status(gp, y, a.job_params[(size_t)PX_WEIGHT * a.J + j]);
            // re-allocation penalty factor of Sec. 4.2
            const bool penalty = !(a.flags & PX_FLAG_NO_REALLOC_PENALTY);
            if (penalty && !(T - R * a.delta > 0.0)) st |= PX_ST_BAD_RESTART;
            const long long held = wave_sum((long long)was.x + was.y + was.z + was.w);
            if (__ballot((was.x | was.y | was.z | was.w) < 0) != 0) st |= PX_ST_NEG_ALLOC;
            Best fair = {0.0, -1, -1};
            if (K > 0) fair = row_best(coefs, q, gp, y, m_row, a.Gm, a.Gs, K, one_node, tabled_row(K, one_node, k1));
            if (!(fair.goodput > 0.0)) st |= PX_ST_ZERO_FAIR;
            if (lane == 0) {
                fair_lds[j] = fair.goodput;
                factor_lds[j] = penalty && held > 0 ? (T - R * a.delta) / (T + a.delta) : 1.0;
                if (st) atomicOr(&status_lds, st);
            }
        }
    }
    __syncthreads();
    if (wave != 0) return;
    // one job per lane: SPEEDUP (Eq. 15) with the penalty, its term of Eq. 14
    const bool mine = lane < a.J;
    double acc = 0.0, wsum = 0.0;
    if (mine) {
        const size_t pair = (size_t)c * a.J + lane;
        const double w = a.job_params[(size_t)PX_WEIGHT * a.J + lane];
        const double d = KEPT ? kept_fair : fair_lds[lane], factor = KEPT ? kept_factor : factor_lds[lane];
        double s_j = d > 0 ? goodput_lds[lane] / d : 0.0;
        if (meta_lds[lane] & kMetaChanged) s_j = s_j * factor;
        if (a.best_m) {
            a.best_m[pair] = m_lds[lane];
            a.best_s[pair] = s_lds[lane];
        }
        if (a.best_goodput) a.best_goodput[pair] = goodput_lds[lane];
        if (a.speedup) a.speedup[pair] = s_j;
        acc += pmean_term(s_j, w, a.p);
        wsum += w;
    }
    long long v = 0;
    if (a.need_constraints) {
        for (int n = lane; n < a.N; n += kWave) {
            const long long x = (long long)node_lds[n];
            const long long asked = (x << 24) >> 24;              // low 40 bits, sign-extended
            const long long distributed = (x - asked) >> 40;
            if (distributed > 1) v += distributed - 1;
            const long long over = asked - (long long)a.node_capacity[n];
            if (over > 0) v += over;
        }
    }
    const long long V = wave_sum(v);
    const double mean = wave_tree_sum(acc) / wave_tree_sum(wsum);
    if (lane == 0) {
        double f = pmean_finish(mean, a.p);
        if (a.violations) a.violations[c] = (int32_t)(V > 0x7FFFFFFF ? 0x7FFFFFFF : V);
        if (V > 0 && !(a.flags & PX_FLAG_NO_CONSTRAINT_CHECK)) f = -(double)V;
        a.fitness[c] = f;
        uint8_t *negatives = (uint8_t *)(a.status + 1);
        if (!KEPT || negative) negatives[c] = (uint8_t)negative;
    }
    // a call that starts anew starts the status section anew; what it finds of the jobs is the same in every workgroup
    if (!KEPT && blockIdx.x == 0) {
        if (lane == 0) *a.status = status_lds;
        if (mine) {
            a.denom[lane] = fair_lds[lane];
            a.factor[lane] = factor_lds[lane];
        }
        for (int i = a.P + lane; i < kSmallCandidates; i += kWave) ((uint8_t *)(a.status + 1))[i] = 0;
    }
}

// ---- row inheritance (pollux_generation with PX_GA_INHERIT_ROWS) ----------------------------------
// The search step has left, per child it formed and per job, the candidate whose row the child holds unchanged
// (a survivor: its results are in place), or -1.  Eq. 13, the re-allocation flag and everything else the fitness
// takes from a row depend on the row, the job and the current allocation only, so an unchanged row takes over the
// results of its source.  The rows a move or a repair has changed are listed per job (a.dirty[j, ...], counted in
// a.dirty_count[j]) for pairs_kernel with SEL = 2, which treats them like any other (candidate, job) pair, per-node
// counters included.  A child the step has flagged (a.odd: it may hold a negative entry or violate a constraint)
// lists all its rows, so its counters come out complete; of every other child only some rows reach the counters,
// and a part of a matrix that satisfies both constraints (which such a child does by construction) satisfies
// them too, so its violation count is the zero it has to be.  One workgroup per listed child; candidates_kernel
// follows as usual.
__global__ void __launch_bounds__(256) inherit_kernel(FitnessArgs a)
{
    const int k = blockIdx.x;
    const int slot = a.sel[k];
    const bool odd = a.odd[k] != 0;
    const int32_t *__restrict__ src = a.src_row + (size_t)k * a.J;
    // four jobs per thread and pass: the sources first, then all the reads that depend on them, then the stores
    constexpr int kJobs = 4;
    for (int j0 = threadIdx.x; j0 < a.J; j0 += kJobs * 256) {
        int s[kJobs];
#pragma unroll
        for (int u = 0; u < kJobs; ++u) {
            const int j = j0 + u * 256;
            s[u] = (j < a.J && !odd) ? src[j] : -1;
        }
        double g[kJobs], bg[kJobs];
        int32_t mt[kJobs], bm[kJobs], bs[kJobs];
#pragma unroll
        for (int u = 0; u < kJobs; ++u) {
            const size_t from = (size_t)(s[u] >= 0 ? s[u] : slot) * a.J + (j0 + u * 256 < a.J ? j0 + u * 256 : 0);
            g[u] = a.G[from];
            mt[u] = a.meta[from];
            bm[u] = a.best_m ? a.best_m[from] : 0;
            bs[u] = a.best_m ? a.best_s[from] : 0;
            bg[u] = a.best_goodput ? a.best_goodput[from] : 0.0;
        }
#pragma unroll
        for (int u = 0; u < kJobs; ++u) {
            const int j = j0 + u * 256;
            if (j >= a.J) continue;
            const size_t to = (size_t)slot * a.J + j;
            if (s[u] >= 0) {
                a.G[to] = g[u];
                a.meta[to] = mt[u];
                if (a.best_m) {
                    a.best_m[to] = bm[u];
                    a.best_s[to] = bs[u];
                }
                if (a.best_goodput) a.best_goodput[to] = bg[u];
            } else {
                a.dirty[(size_t)j * a.n_sel + atomicAdd(&a.dirty_count[j], 1)] = slot;
            }
        }
    }
}

// ---- memoised mode, one workgroup per candidate ---------------------------------------------------
// With the argmaxes looked up a candidate costs the reading of its matrix and little else, so one workgroup
// takes the whole candidate: it walks the matrix in memory order (four wavefronts, 64 consecutive rows each
// per round of 256 jobs), keeps the per-node counters of the constraint check in LDS (integer atomics:
// order-independent) and K, nodes and the changed flag of every row in LDS as well.  After up to 1024 jobs the
// workgroup stops reading, and thread t finishes the pairs of jobs t, t + 256, ... of those: looks the result up, forms
// SPEEDUP (Eq. 15) with the penalty and its term of the generalized mean (Eq. 14).  (Finishing per round instead,
// between the requests, left the memory system idle a tenth of the time.)  The terms are summed exactly as
// candidates_kernel sums them (thread t over its jobs in ascending order, then the same tree), so the fitness is
// bit-identical to the plain mode's.  Nothing but the results leaves the chip.
// Rows of 4 to 256 entries, of any length and alignment: a lane's 16-byte load needs no more than the alignment of its
// entries, the lane of a row's last entries takes the last four and masks those its neighbour has, and lanes beyond mask
// all.  Rows of at most 64 entries (SHORT) come four to a load, 16 lanes each.
//   2048 candidates of 900 jobs on 250 nodes: 1169 us with a wavefront per (candidate, job) reading entry by entry, 0.34 ms so.
// KIND: the fp64 grid, the fp32 variant, or the sampling argmax.
// CHILD: the children of a search step that inherits rows (see inherit_kernel for the rule), where child_kernel does not take them:
// a row held unchanged takes over the results of the row it was copied from, only the others are read back and looked up.  One
// launch in place of three (inherit_kernel, pairs_kernel over the listed rows, candidates_kernel: 14 us a generation at 30 jobs, 15
// at 200).  A child that satisfies both constraints by construction has no violations; any other is evaluated in full, counters
// included.
// Rows of more GPUs than the memo table covers are found in place by their wavefront when the chunk is finished.  (An instance
// without that code, with a second launch for the candidates that need it, was no faster at any size: 4096 candidates of 1000
// jobs on 256 nodes 957 us a call with the pair of launches, 856 with the one.)
// PAIRS: the goodput and the node count of every pair are also left in the workspace (PX_FLAG_PAIR_RESULTS; CHILD does so).
constexpr int kMemoChunkJobs = 4 * kCandThreads;    // jobs between two finishing steps
constexpr int kMemoNodes = 4 * kWave;               // the longest row
constexpr int kInherited = -1;                      // row_lds: the row takes over the results of candidate x
enum MemoKind { kMemoGrid, kMemoF32, kMemoSampled };

// A row's share of the constraint counters: the few lanes that hold a non-zero entry (a job sits on few nodes) add their four
// entries, zeros included (a negative entry as it is): one branch per row instead of one per entry.
__device__ __forceinline__ void add_to_nodes(unsigned long long *node_lds, const RowLane &at_row, const Entries &w, int nodes)
{
    if ((w.x | w.y | w.z | w.w) != 0) {
        const unsigned long long one_job = nodes >= 2 ? kPackJob : 0ull;
        unsigned long long *to = node_lds + at_row.base;
        atomicAdd(&to[0], (unsigned long long)(long long)w.x + (w.x > 0 ? one_job : 0ull));
        atomicAdd(&to[1], (unsigned long long)(long long)w.y + (w.y > 0 ? one_job : 0ull));
        atomicAdd(&to[2], (unsigned long long)(long long)w.z + (w.z > 0 ? one_job : 0ull));
        atomicAdd(&to[3], (unsigned long long)(long long)w.w + (w.w > 0 ? one_job : 0ull));
    }
}

// Four rows per load: K and nodes | changed of the row the lane's group of 16 lanes holds (live: it holds one).
__device__ __forceinline__ int2 reduce_rows(const RowLane &at_row, const Entries &v, const Entries &was, bool live, bool count_nodes,
                                            unsigned long long *node_lds, bool &any_neg)
{
    const Entries mask = live ? at_row.mask : Entries{0, 0, 0, 0};
    const Entries w = v & mask, differs = (v ^ was) & mask;
    const int positive = (w.x > 0 ? 1 : 0) + (w.y > 0 ? 1 : 0) + (w.z > 0 ? 1 : 0) + (w.w > 0 ? 1 : 0);
    // one word carries two small counts: positive entries (at most 64) and lanes that differ
    const int counts = row16_sum(positive | ((differs.x | differs.y | differs.z | differs.w) != 0 ? 1 << 12 : 0));
    const int K = row16_sum((w.x + w.y) + (w.z + w.w));
    any_neg |= __ballot((w.x | w.y | w.z | w.w) < 0) != 0ull;
    if (count_nodes) add_to_nodes(node_lds, at_row, w, counts & 0xFFF);
    return make_int2(K, (counts & 0xFFF) | ((counts >> 12) != 0 ? kMetaChanged : 0));
}

// What a thread asks for ahead of its first pair (child_kernel): the results of the row's source, and the job's figures.
struct PairAhead {
    int from = -1;                   // the candidate those results are of, or -1: none
    double goodput = 0.0;
    int meta = 0, m = 0, s = 0;
    bool job = false;                // the job's figures are there
    double denom = 0.0, factor = 0.0, weight = 0.0;
};

// Thread t < kCandThreads finishes the pairs of jobs jc + t, jc + t + kCandThreads, ... < jc + jobs of candidate c (rows: K and nodes |
// changed per job, or candidate and kInherited): looks the result up, or takes it over, and adds the job's term of the mean.
template <int KIND, bool CHILD, bool PAIRS, typename REAL>
__device__ __forceinline__ void finish_pairs(const FitnessArgs &a, int c, int jc, int jobs, int k1, const int2 *rows, PairAhead ahead,
                                             REAL &acc, REAL &wsum)
{
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)), lane = lane_id();
    const double *__restrict__ wt = a.job_params + (size_t)PX_WEIGHT * a.J;
    const REAL p = (REAL)a.p;
    for (int at0 = kWave * wave; wave < 4 && at0 < jobs; at0 += kCandThreads) {
        const int at = at0 + lane;
        const bool mine = at < jobs;
        const int2 row = mine ? rows[at] : make_int2(0, 0);
        Best best = {0.0, -1, -1};
        // rows beyond the memo table: found and priced by the whole wavefront, one after the other
        unsigned long long pending = __ballot(row.y != kInherited && !tabled_row(row.x, (row.y & ~kMetaChanged) == 1, k1));
        while (__builtin_expect(pending != 0ull, 0)) {
            const int l = __ffsll(pending) - 1;
            pending &= pending - 1;
            const int K = __builtin_amdgcn_readlane(row.x, l);
            const int nodes = __builtin_amdgcn_readlane(row.y, l) & ~kMetaChanged;
            const int j = jc + at0 + l;
            Best found;
            if constexpr (KIND == kMemoF32) found = sweep_f32(load_job_f32(a.job_params, a.J, j), job_tables(a, j), a.rk, a.Gm, a.Gs, K, nodes);
            else if constexpr (KIND == kMemoSampled) found = sweep_sampled<false>(load_job(a.job_params, a.J, j), a.m_grid + (size_t)j * a.Gm,
                                                                                  a.Gm, a.Gs, K, nodes);
            else found = row_best_plain<false>(load_job(a.job_params, a.J, j), load_grid_params(a.job_params, a.J, j),
                                  a.m_grid + (size_t)j * a.Gm, a.Gm, a.Gs, K, nodes == 1, false);
            if (lane == l) best = found;
        }
        if (!mine) continue;
        const int j = jc + at;
        const size_t pair = (size_t)c * a.J + j;
        int d_meta = row.y;
        if (CHILD && row.y == kInherited) {
            if (ahead.from == row.x) {
                best.goodput = ahead.goodput;
                d_meta = ahead.meta;
                best.m = ahead.m;
                best.s = ahead.s;
            } else {
                const size_t from = (size_t)row.x * a.J + j;
                best.goodput = a.G[from];
                d_meta = a.meta[from];
                if (a.best_m) {
                    best.m = a.best_m[from];
                    best.s = a.best_s[from];
                }
            }
        } else if (row.x >= 1 && tabled_row(row.x, (d_meta & ~kMetaChanged) == 1, k1)) {
            const MemoEntry e = a.memo[((size_t)j * 2 + ((d_meta & ~kMetaChanged) == 1 ? 1 : 0)) * kTableK + (row.x - 1)];
            best.goodput = e.goodput; best.m = e.m; best.s = e.s;
        }
        if (a.best_m) {
            a.best_m[pair] = best.m;
            a.best_s[pair] = best.s;
        }
        if (a.best_goodput) a.best_goodput[pair] = best.goodput;
        if constexpr (PAIRS) {
            // what a later generation that inherits rows reads of this pair
            a.G[pair] = best.goodput;
            a.meta[pair] = d_meta;
        }
        // SPEEDUP (Eq. 15) with the re-allocation penalty, and the job's term of Eq. 14
        const REAL d = (REAL)(ahead.job ? ahead.denom : a.denom[j]);
        REAL s_j = d > 0 ? (REAL)best.goodput / d : (REAL)0;
        if (d_meta & kMetaChanged) s_j = s_j * (REAL)(ahead.job ? ahead.factor : a.factor[j]);
        if (a.speedup) a.speedup[pair] = (double)s_j;
        const REAL w = (REAL)(ahead.job ? ahead.weight : wt[j]);
        acc += pmean_term(s_j, w, p);
        wsum += w;
        ahead.from = -1;             // (that was the thread's first pair)
        ahead.job = false;
    }
}

// Constraint check of one node: multi-node jobs beyond the first and GPUs beyond capacity.
__device__ __forceinline__ long long node_violations(unsigned long long counter, int capacity)
{
    const long long x = (long long)counter;
    const long long asked = (x << 24) >> 24;              // low 40 bits, sign-extended
    const long long distributed = (x - asked) >> 40;
    const long long over = asked - (long long)capacity;
    return (distributed > 1 ? distributed - 1 : 0) + (over > 0 ? over : 0);
}

// The fitness of candidate c from the sums of its jobs' terms and its violations, by one thread.
template <typename REAL>
__device__ __forceinline__ void store_fitness(const FitnessArgs &a, int c, REAL total, REAL weight, long long V)
{
    const REAL mean = total / weight;
    double f = (double)pmean_finish(mean, (REAL)a.p);
    if (a.violations) a.violations[c] = (int32_t)(V > 0x7FFFFFFF ? 0x7FFFFFFF : V);
    if (V > 0 && !(a.flags & PX_FLAG_NO_CONSTRAINT_CHECK)) f = -(double)V;
    a.fitness[c] = f;
}

// WAVES: four wavefronts, or sixteen where the candidates are too few to fill the chip and their jobs many (see
// launch_memo_candidates).
template <int KIND, bool SHORT, bool CHILD, bool PAIRS, int WAVES>
__global__ void __launch_bounds__(WAVES *kWave) memo_candidates_kernel(FitnessArgs a)
{
    static_assert(kCandThreads == 4 * kWave && WAVES >= 4, "thread t < kCandThreads is lane t % 64 of wavefront t / 64");
    static_assert(!CHILD || PAIRS, "children: per-pair results kept");
    constexpr int kThreads = WAVES * kWave;
    using Real = typename std::conditional<KIND == kMemoF32, float, double>::type;
    __shared__ unsigned long long node_lds[kMemoNodes];      // per node: GPUs asked + multi-node jobs << 40, as colpack
    __shared__ int2 row_lds[kMemoChunkJobs];                 // per job of the chunk: K, nodes | changed flag; or candidate, kInherited
    __shared__ uint16_t list_lds[CHILD ? kMemoChunkJobs : 1]; // positions in the chunk of the rows to read
    __shared__ Real red_acc[kCandThreads];
    __shared__ Real red_w[kCandThreads];
    __shared__ long long red_v[kCandThreads];
    __shared__ int listed;
    const int c = a.sel ? a.sel[blockIdx.x] : (int)blockIdx.x;
    const int t = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int lane = lane_id();
    const int k1 = __builtin_amdgcn_readfirstlane(*a.k1);
    bool odd = true;                                         // CHILD: to be evaluated in full
    const int32_t *__restrict__ src = nullptr;
    if constexpr (CHILD) {
        odd = __builtin_amdgcn_readfirstlane(a.odd[blockIdx.x]) != 0;
        src = a.src_row + (size_t)blockIdx.x * a.J;
    }
    const bool count_nodes = a.need_constraints && odd;
    if (t < kMemoNodes) node_lds[t] = 0ull;
    if (t == 0) listed = 0;
    if (a.or_job_status && blockIdx.x == 0) or_job_status(a);
    __syncthreads();

    // what this lane holds of a row
    const RowLane at_row = row_lane(SHORT ? (lane & 15) : lane, a.N);
    auto load = [&](const int32_t *row) { return *(const Entries *)(row + at_row.base); };
    bool any_neg = false;
    // One row per load: K and nodes | changed of the row the wavefront holds, the same in every lane.
    auto reduce_row = [&](const Entries &v, const Entries &was) {
        const Entries w = v & at_row.mask, differs = (v ^ was) & at_row.mask;
        const int K = wave_sum((w.x + w.y) + (w.z + w.w));
        const int nodes = __popcll(__ballot(w.x > 0)) + __popcll(__ballot(w.y > 0)) + __popcll(__ballot(w.z > 0)) + __popcll(__ballot(w.w > 0));
        const bool changed = __ballot((differs.x | differs.y | differs.z | differs.w) != 0) != 0;
        any_neg |= __ballot((w.x | w.y | w.z | w.w) < 0) != 0;
        if (count_nodes) add_to_nodes(node_lds, at_row, w, nodes);
        return make_int2(K, nodes | (changed ? kMetaChanged : 0));
    };
    Real acc = 0, wsum = 0;
    for (int jc = 0; jc < a.J; jc += kMemoChunkJobs) {
        const int chunk_jobs = a.J - jc < kMemoChunkJobs ? a.J - jc : kMemoChunkJobs;
        const int32_t *__restrict__ pop = a.population + ((size_t)c * a.J + jc) * a.N;
        const int32_t *__restrict__ cur = a.current_alloc + (size_t)jc * a.N;
        if constexpr (CHILD) {
            for (int at = t; at < chunk_jobs; at += kThreads) {
                const int from = odd ? -1 : src[jc + at];
                if (from >= 0) row_lds[at] = make_int2(from, kInherited);
                else list_lds[atomicAdd(&listed, 1)] = (uint16_t)at;
            }
            __syncthreads();
            const int rows = __builtin_amdgcn_readfirstlane(listed);
            if constexpr (SHORT) {
                for (int q0 = 4 * wave; q0 < rows; q0 += 4 * WAVES) {
                    const int q = q0 + (lane >> 4);
                    const int at = list_lds[q < rows ? q : rows - 1];
                    const int2 row = reduce_rows(at_row, load(pop + (size_t)at * a.N), load(cur + (size_t)at * a.N), q < rows, count_nodes, node_lds, any_neg);
                    if (q < rows && (lane & 15) == 0) row_lds[at] = row;
                }
            } else {
                constexpr int kAhead = 4;
                for (int q0 = wave; q0 < rows; q0 += kAhead * WAVES) {
                    Entries v[kAhead], was[kAhead];
                    int at[kAhead];
#pragma unroll
                    for (int u = 0; u < kAhead; ++u) {
                        const int q = q0 + u * WAVES;
                        at[u] = __builtin_amdgcn_readfirstlane((int)list_lds[q < rows ? q : rows - 1]);
                        v[u] = load(pop + (size_t)at[u] * a.N);
                        was[u] = load(cur + (size_t)at[u] * a.N);
                    }
#pragma unroll
                    for (int u = 0; u < kAhead; ++u) {
                        if (q0 + u * WAVES < rows) {
                            const int2 row = reduce_row(v[u], was[u]);
                            if (lane == 0) row_lds[at[u]] = row;
                        }
                    }
                }
            }
        } else {
            // Row q of this wavefront in the chunk (position: the job's number less jc) of the `rows` it has: with four
            // wavefronts 64 consecutive rows of every round of 256 each, or where there is no such round an even share in
            // whole passes of the loops below (63 jobs on 138 nodes, 19 candidates: 23.0 us in one wavefront, 9.6 so; 200
            // jobs in other shares than 64, 64, 64, 8 only add passes); with more of them a stretch of its own.
            constexpr int kPass = SHORT ? 16 : 8;
            const int full = WAVES == 4 ? chunk_jobs / kCandThreads : 0, tail = chunk_jobs - full * kCandThreads;
            const int even = (tail + WAVES - 1) / WAVES;
            const int share = full > 0 ? kWave : (WAVES == 4 ? (even + kPass - 1) & ~(kPass - 1) : (even + 3) & ~3);
            const int last_rows = tail - share * wave;
            const int rows = kWave * full + (last_rows < 0 ? 0 : (last_rows > share ? share : last_rows));
            auto place = [&](int q) {
                if constexpr (WAVES == 4) return (q >> 6) * kCandThreads + share * wave + (q & (kWave - 1));
                else return share * wave + q;
            };
            if constexpr (SHORT) {
                constexpr int kAhead = 4;                   // loads in flight, of four rows each
                for (int q0 = 0; q0 < rows; q0 += 4 * kAhead) {
                    Entries v[kAhead], was[kAhead];
#pragma unroll
                    for (int u = 0; u < kAhead; ++u) {
                        const int q = q0 + 4 * u + (lane >> 4);
                        const int at = place(q < rows ? q : rows - 1);
                        v[u] = load(pop + (size_t)at * a.N);
                        was[u] = load(cur + (size_t)at * a.N);
                    }
#pragma unroll
                    for (int u = 0; u < kAhead; ++u) {
                        if (q0 + 4 * u < rows) {
                            const int q = q0 + 4 * u + (lane >> 4);
                            const int2 row = reduce_rows(at_row, v[u], was[u], q < rows, count_nodes, node_lds, any_neg);
                            if (q < rows && (lane & 15) == 0) row_lds[place(q)] = row;
                        }
                    }
                }
            } else if (rows > 0) {
                constexpr int kAhead = 4;
                static_assert(kWave % (2 * kAhead) == 0, "a pass of the request loop never straddles two rounds");
                const int32_t *__restrict__ rowp = pop + at_row.base;
                const int32_t *__restrict__ curp = cur + at_row.base;
                auto request = [&](int q0, Entries (&v)[kAhead]) {
#pragma unroll
                    for (int u = 0; u < kAhead; ++u) {
                        const int q = q0 + u < rows ? q0 + u : rows - 1;               // the tail reads the last row again
                        v[u] = *(const Entries *)(rowp + (size_t)place(q) * a.N);
                    }
                };
                // The rows of the current allocation come from L2 (shared by all candidates), and only the lanes whose
                // group of four entries of the current row holds anything read it (a.curmask, a scalar per row: a job sits
                // on few nodes, so that is a lane or two); all other lanes read one block of zeros, which is what the
                // current row holds there: a few cache lines per row through the vector cache instead of 1 KB.  Every lane
                // loads either way, so the number of loads in flight is the same on every path and the waits can be
                // exact.  The rows are requested when their batch is about to be worked on, not a batch ahead, which
                // saves the registers of a second buffer, but BEFORE the next batch of the population is requested:
                // loads complete in order, so waiting for them then leaves that next batch in flight.
                // (the masks through the scalar cache: a vector load would make every use wait for all loads in flight)
                typedef const unsigned long long __attribute__((address_space(4))) *ScalarMasks;
                const ScalarMasks maskp = (ScalarMasks)a.curmask + jc;
                auto request_current = [&](int q0, Entries (&cv)[kAhead]) {
#pragma unroll
                    for (int u = 0; u < kAhead; ++u) {
                        const int at = place(q0 + u < rows ? q0 + u : rows - 1);
                        cv[u] = *(const Entries *)(((maskp[at] >> lane) & 1ull) ? curp + (size_t)at * a.N : a.zeros);
                    }
                };
                int d_K = 0, d_meta = 0;                        // lane r: K and nodes | changed of row q with q % 64 = r
                auto work = [&](int q0, const Entries (&v)[kAhead], const Entries (&cv)[kAhead]) {
#pragma unroll
                    for (int u = 0; u < kAhead; ++u) {
                        if (q0 + u < rows) {
                            const int2 row = reduce_row(v[u], cv[u]);
                            if (lane == ((q0 + u) & (kWave - 1))) {
                                d_K = row.x;
                                d_meta = row.y;
                            }
                        }
                    }
                };
                // Two buffers of kAhead rows: requests are in flight all the time.  A request past the end of the
                // wavefront's rows reads its last row again (nothing works on it), so that every pass through the
                // loop issues the same loads in the same order and each wait leaves exactly the next batch in flight.
                Entries v0[kAhead], v1[kAhead], cv[kAhead];
                request(0, v0);
                // (the fences keep the compiler from issuing the requests in another order)
                auto fence = [] {
                    asm volatile("" ::: "memory");
                    __builtin_amdgcn_sched_barrier(0);
                };
                for (int q0 = 0; q0 < rows; q0 += 2 * kAhead) {
                    request_current(q0, cv);
                    fence();
                    request(q0 + kAhead, v1);
                    fence();
                    work(q0, v0, cv);
                    fence();
                    request_current(q0 + kAhead, cv);
                    fence();
                    request(q0 + 2 * kAhead, v0);
                    fence();
                    work(q0 + kAhead, v1, cv);
                    fence();
                    // a round of 64 rows (or the last, shorter one) is complete: lane r puts its row's figures away
                    const int next = q0 + 2 * kAhead;
                    if ((next & (kWave - 1)) == 0 || next >= rows) {
                        const int first = q0 & ~(kWave - 1);
                        const int in_round = rows - first < kWave ? rows - first : kWave;
                        if (lane < in_round) row_lds[place(first) + lane] = make_int2(d_K, d_meta);
                    }
                }
            }
        }
        __syncthreads();                                    // the chunk's rows are all put away
        finish_pairs<KIND, CHILD, PAIRS>(a, c, jc, chunk_jobs, k1, row_lds, PairAhead(), acc, wsum);
        if (CHILD && t == 0) listed = 0;
        __syncthreads();                                    // before the next chunk's rows take their places
    }
    if (t < kCandThreads) {
        red_acc[t] = acc;
        red_w[t] = wsum;
    }
    if (__ballot(any_neg) != 0ull && lane == 0) atomicOr(a.status, PX_ST_NEG_ALLOC);

    // constraint check: per node, multi-node jobs beyond the first and GPUs beyond capacity
    const long long v = count_nodes && t < a.N ? node_violations(node_lds[t], a.node_capacity[t]) : 0;
    if (t < kCandThreads) red_v[t] = v;
    __syncthreads();
    if (wave != 0) return;
    const Real total = tree_sum(red_acc), weight = tree_sum(red_w);
    const long long V = tree_sum(red_v);
    if (t == 0) store_fitness(a, c, total, weight, V);
}

// ---- a child of a memoised search that inherits rows: formed and evaluated by one workgroup ----------------------
// The step's workgroup has the child's rows and where each comes from at hand, so it goes on to the fitness: the rows held unchanged
// take over their source's results (asked for when the parents are known, so that they arrive while the rows are copied), the
// few others are read back and looked up.  The terms are summed as memo_candidates_kernel sums them.  A generation is two
// launches (rank, this) where it was three: an interval of 20 generations of 256 x 30 x 16 takes 268 us where it took 327, of
// 1000 x 200 x 64 515 where it took 581.  Bound, at 30 jobs, by its own chain: 17400 cycles, of which the parents (kernel
// arguments, order, draws) take 3800, the rows' trip from memory 2900, the repairs 3600 and what follows them 4600.
// For rows of 4 to 64 nodes without a GPU limit per job, up to kFinishJobs jobs (generation_in_one): longer rows are bound by the
// copy, and 18 bytes of LDS a job hold a thousand jobs.
constexpr int kFinishJobs = 1024;

// Three workgroups a compute unit: at 89 registers, which only the sweep of rows beyond the memo table needs, there were two, and
// 600 children took two rounds on 256 compute units (20 generations, 8 to 256 jobs: 1.06 to 1.12 times the three launches before, now
// 0.83 to 0.91; 800 children 1.05, now 0.94 to 0.96; 500 and fewer as before).  At 64 registers and four workgroups 50 to 600 children
// take 2 to 6 % longer, 800 and more 10 % less.
template <int KIND, int ROWS>
__global__ void __launch_bounds__(kGaThreads) __attribute__((amdgpu_waves_per_eu(6))) child_kernel(GaArgs g, FitnessArgs a)
{
    using Real = typename std::conditional<KIND == kMemoF32, float, double>::type;
    extern __shared__ __align__(16) unsigned char ga_lds[];
    __shared__ unsigned long long node_lds[kArrayNodes];     // per node: GPUs asked + multi-node jobs << 40, as colpack
    __shared__ Real red_acc[kCandThreads], red_w[kCandThreads];
    __shared__ int odd_lds, listed;
    const GaShared sh = carve_shared(ga_lds, g.J, g.N, g.max_entries);
    const int t = threadIdx.x, lane = lane_id();
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int c = a.sel[blockIdx.x];
    const int k1 = __builtin_amdgcn_readfirstlane(*a.k1);
    if (t < kArrayNodes) node_lds[t] = 0ull;
    if (t == 0) listed = 0;
    PairAhead ahead;
    if (t < kCandThreads && t < a.J) {
        ahead.job = true;
        ahead.denom = a.denom[t];
        ahead.factor = a.factor[t];
        ahead.weight = a.job_params[(size_t)PX_WEIGHT * a.J + t];
    }
    // the results of the row job t has if neither a move nor a repair touches it
    auto early = [&](int cand_a, int cand_b) {
        if (!ahead.job) return;
        const int d = sh.dec[t];                             // (this thread's own entry)
        if ((d >> 1) != 0) return;
        ahead.from = (d & 1) ? cand_b : cand_a;
        const size_t from = (size_t)ahead.from * a.J + t;
        ahead.goodput = a.G[from];
        ahead.meta = a.meta[from];
        if (a.best_m) {
            ahead.m = a.best_m[from];
            ahead.s = a.best_s[from];
        }
    };
    static_assert(kCandThreads <= kGaThreads, "thread t draws the decision of job t");
    form_child<ROWS, true, true>(g, sh, &odd_lds, early);
    __syncthreads();
    // the rows that have no source are read back, four to a load
    const bool odd = odd_lds != 0;
    const bool count_nodes = a.need_constraints && odd;
    int2 *rows_lds = (int2 *)(sh.src + ((a.J + 1) & ~1));
    uint16_t *list_lds = (uint16_t *)(rows_lds + a.J);
    for (int at = t; at < a.J; at += kGaThreads) {
        const int from = odd ? -1 : sh.src[at];
        if (from >= 0) rows_lds[at] = make_int2(from, kInherited);
        else list_lds[atomicAdd(&listed, 1)] = (uint16_t)at;
    }
    __syncthreads();
    const int rows = __builtin_amdgcn_readfirstlane(listed);
    const RowLane at_row = row_lane(lane & 15, a.N);
    const int32_t *__restrict__ pop = a.population + (size_t)c * a.J * a.N;
    bool any_neg = false;
    for (int q0 = 4 * wave; q0 < rows; q0 += 4 * (kGaThreads / kWave)) {
        const int q = q0 + (lane >> 4);
        const int at = list_lds[q < rows ? q : rows - 1];
        const Entries v = *(const Entries *)(pop + (size_t)at * a.N + at_row.base);
        const Entries was = *(const Entries *)(a.current_alloc + (size_t)at * a.N + at_row.base);
        const int2 row = reduce_rows(at_row, v, was, q < rows, count_nodes, node_lds, any_neg);
        if (q < rows && (lane & 15) == 0) rows_lds[at] = row;
    }
    if (any_neg && lane == 0) atomicOr(a.status, PX_ST_NEG_ALLOC);
    __syncthreads();
    Real acc = 0, wsum = 0;
    finish_pairs<KIND, true, true>(a, c, 0, a.J, k1, rows_lds, ahead, acc, wsum);
    if (t < kCandThreads) {
        red_acc[t] = acc;
        red_w[t] = wsum;
    }
    const long long v = count_nodes && t < a.N ? node_violations(node_lds[t], a.node_capacity[t]) : 0;
    __syncthreads();
    if (wave != 0) return;
    static_assert(kArrayNodes <= kWave, "the first wavefront holds every node's violations");
    const Real total = tree_sum(red_acc), weight = tree_sum(red_w);
    const long long V = wave_sum(v);
    if (t == 0) store_fitness(a, c, total, weight, V);
}

}  // namespace px

// ---- host side -----------------------------------------------------------------

namespace px {

// The job-level part of the arguments: dimensions, inputs that describe the jobs, workspace sections.
static FitnessArgs job_level_args(const pollux_dims *d, const double *job_params, const int32_t *m_grid, void *workspace)
{
    const WorkspaceLayout L = workspace_layout(*d);
    char *ws = (char *)workspace;
    FitnessArgs a = {};
    a.P = d->P; a.J = d->J; a.N = d->N; a.Gm = d->Gm; a.Gs = d->Gs; a.flags = d->flags;
    a.m_grid = m_grid; a.job_params = job_params;
    a.status = (int32_t *)(ws + L.status);
    a.rs = (double *)(ws + L.rs);
    a.rsf = (float *)(ws + L.rsf);
    a.rk = (double *)(ws + L.rk);
    a.tg = (double2 *)(ws + L.tg);
    a.lntg = (double *)(ws + L.lntg);
    a.pu = (double *)(ws + L.pu);
    a.qh5 = (double *)(ws + L.qh5);
    a.ql5 = (double *)(ws + L.ql5);
    a.lt = (double *)(ws + L.lt);
    a.ca = (double2 *)(ws + L.ca);
    a.srange = (int32_t *)(ws + L.srange);
    a.k1 = (int32_t *)(ws + L.k1);
    a.gs_pad = ((d->Gs + 31) / 32) * 32;
    return a;
}

// Rows (placement class, K) one wavefront of prepare_kernel takes: of the tables table_rows.  Memoised, whose rows end in an election,
// two, from 256 jobs on four.  Calls of 40 candidates, 64 x 16, us with two, four and eight rows: 140 jobs 16.5, 17.8, 18.7; 200 jobs
// 19.9, 19.9, 20.3; 300 jobs 34.5, 33.4, 33.4; 900 jobs 81.5, 74.5, 74.5; with 128 batch sizes 140 jobs 22.1, 25.6, 27.9; 500 jobs 63.4,
// 61.2, 64.2; 900 jobs 107.7, 100.8, 103.3 (an election for both groups of 64 batch sizes since: 500 jobs 57.1, 900 jobs 95.2).
// The sampling argmax has no such terms: one row, or two where the jobs are many (200 jobs 30.8 and 29.5 us a call).
template <int MODE>
static void launch_prepare_rows(const FitnessArgs &a, hipStream_t stream)
{
    auto blocks = [&](int rows) {
        return dim3(prep_blocks(a.J, prep_tasks(MODE, rows), a.clear_counters ? (long long)a.P * a.N : 0));
    };
    if constexpr (MODE == kPrepSampled || MODE == kPrepSampledMemo) {
        if (a.J < 128) hipLaunchKernelGGL((prepare_kernel<1, MODE>), blocks(1), dim3(256), 0, stream, a);
        else hipLaunchKernelGGL((prepare_kernel<2, MODE>), blocks(2), dim3(256), 0, stream, a);
    } else {
        const int rows = MODE == kPrepMemo ? (a.J < 256 ? 2 : 4) : table_rows(a.J, a.Gm);
        if (rows == 2) hipLaunchKernelGGL((prepare_kernel<2, MODE>), blocks(2), dim3(256), 0, stream, a);
        else if (rows == 4) hipLaunchKernelGGL((prepare_kernel<4, MODE>), blocks(4), dim3(256), 0, stream, a);
        else if constexpr (MODE != kPrepMemo) hipLaunchKernelGGL((prepare_kernel<8, MODE>), blocks(8), dim3(256), 0, stream, a);
    }
}

// The population pass of memoised mode, P_eff workgroups.  Up to 256 candidates leave most of a compute unit idle with four
// wavefronts each; from 64 jobs on (a load of rows per wavefront) they get sixteen.  Calls that keep their tables, us, 256
// candidates with sixteen and 257 with four: 64 jobs on 138 nodes 8.3, 10.3; 200 on 64 8.6, 11.1; 200 on 256 15.9, 26.5; 1000 on 64
// 21.9, 34.4; 1000 on 256 52, 105.  19 candidates, 63 jobs with four and 64 with sixteen: on 64 nodes 5.6, 5.6, on 138 9.6, 8.0.
template <int KIND>
static void launch_memo_candidates(const FitnessArgs &a, int P_eff, bool child, bool pairs_kept, hipStream_t stream)
{
    const dim3 grid((unsigned)P_eff);
    const bool short_rows = a.N <= kWave, few = P_eff <= 256 && a.J >= kWave;
#define PX_LAUNCH_MEMO(CHILD, PAIRS, WAVES)                                                                                                \
    do {                                                                                                                                   \
        if (short_rows) hipLaunchKernelGGL((memo_candidates_kernel<KIND, true, CHILD, PAIRS, WAVES>), grid, dim3(WAVES * kWave), 0, stream, a); \
        else hipLaunchKernelGGL((memo_candidates_kernel<KIND, false, CHILD, PAIRS, WAVES>), grid, dim3(WAVES * kWave), 0, stream, a);      \
    } while (0)
    if (child) PX_LAUNCH_MEMO(true, true, 4);
    else if (pairs_kept && few) PX_LAUNCH_MEMO(false, true, 16);
    else if (pairs_kept) PX_LAUNCH_MEMO(false, true, 4);
    else if (few) PX_LAUNCH_MEMO(false, false, 16);
    else PX_LAUNCH_MEMO(false, false, 4);
#undef PX_LAUNCH_MEMO
}

static int launch_queries(const pollux_dims *d, const double *job_params, const int32_t *m_grid, const QueryArgs &q, hipStream_t stream)
{
    FitnessArgs a = {};
    a.J = d->J; a.Gm = d->Gm; a.Gs = d->Gs;
    a.m_grid = m_grid; a.job_params = job_params;
    const int per_job = q.mode == 0 ? q.max_nodes + 1 : 1, rows = query_rows(d->J, per_job);
    if (rows > 1) {
        const long long waves = (long long)d->J * ((per_job + rows - 1) / rows);
        hipLaunchKernelGGL(queries_rows_kernel, dim3((unsigned)((waves + kWavesPerBlock - 1) / kWavesPerBlock)), dim3(256), 0, stream, a, q, rows);
        return hipGetLastError() == hipSuccess ? PX_OK : PX_E_HIP;
    }
    const long long queries = (long long)d->J * per_job;
    const dim3 grid((unsigned)((queries + kWavesPerBlock - 1) / kWavesPerBlock));
    hipLaunchKernelGGL(queries_kernel, grid, dim3(256), 0, stream, a, q);
    return hipGetLastError() == hipSuccess ? PX_OK : PX_E_HIP;
}

int launch_goodput_per_gpu(const pollux_dims *d, const double *job_params, const int32_t *m_grid, int gpus_per_node,
                           int max_nodes, double *per_gpu, hipStream_t stream)
{
    QueryArgs q = {};
    q.mode = 0; q.gpus_per_node = gpus_per_node; q.max_nodes = max_nodes; q.per_gpu = per_gpu;
    return launch_queries(d, job_params, m_grid, q, stream);
}

int launch_autoscale(int J, int max_nodes, const double *per_gpu, const int32_t *nodes_now, double U, double L,
                     int32_t *nodes_new, hipStream_t stream)
{
    hipLaunchKernelGGL(autoscale_kernel, dim3((unsigned)((J + 255) / 256)), dim3(256), 0, stream, J, max_nodes, per_gpu,
                       nodes_now, U, L, nodes_new);
    return hipGetLastError() == hipSuccess ? PX_OK : PX_E_HIP;
}

int launch_sim_tick(const pollux_dims *d, const double *job_params, const int32_t *m_grid, const int32_t *K,
                    const int32_t *nodes, const int32_t *changed, const double *target, double dt, double restart_delay,
                    double *progress, double *goodput, int32_t *finished, hipStream_t stream)
{
    QueryArgs q = {};
    q.mode = 1; q.K = K; q.nodes = nodes; q.changed = changed; q.target = target; q.dt = dt;
    q.restart_delay = restart_delay; q.progress = progress; q.goodput = goodput; q.finished = finished;
    return launch_queries(d, job_params, m_grid, q, stream);
}

__global__ void copy_status_kernel(const int32_t *__restrict__ from, int32_t *__restrict__ to)
{
    const bool negative = threadIdx.x > 0 && from[threadIdx.x] != 0;
    const int bits = __ballot(negative) != 0ull ? PX_ST_NEG_ALLOC : 0;
    if (threadIdx.x == 0) *to = from[0] | bits;
}

int launch_copy_status(const void *workspace, int32_t *status_out, hipStream_t stream)
{
    pollux_dims d = {1, 1, 1, 1, 1, 0, 0};
    const int32_t *word = (const int32_t *)((const char *)workspace + workspace_layout(d).status);
    hipLaunchKernelGGL(copy_status_kernel, dim3(1), dim3(kStatusWords), 0, stream, word, status_out);
    return hipGetLastError() == hipSuccess ? PX_OK : PX_E_HIP;
}

// The arguments of a fitness call: all candidates, or (first_rank > 0) those of rank first_rank and beyond in the order the search
// step left in the workspace, i.e. the slots it has just rewritten; the others keep the results they have.
static FitnessArgs call_args(const pollux_dims *d, const int32_t *population, const double *job_params, const int32_t *m_grid,
                             const int32_t *fair_share, const int32_t *current_alloc, const int32_t *node_capacity, double p,
                             double delta, void *workspace, double *fitness, int32_t *best_m, int32_t *best_s,
                             double *best_goodput, double *speedup, int32_t *violations, int first_rank)
{
    const WorkspaceLayout L = workspace_layout(*d);
    char *ws = (char *)workspace;
    FitnessArgs a = job_level_args(d, job_params, m_grid, workspace);
    a.population = population; a.fair_share = fair_share; a.current_alloc = current_alloc;
    a.node_capacity = node_capacity;
    a.p = p; a.delta = delta;
    a.denom = (double *)(ws + L.denom);
    a.factor = (double *)(ws + L.factor);
    a.jobstat = (int32_t *)(ws + L.jobstat);
    a.G = (double *)(ws + L.G);
    a.meta = (int32_t *)(ws + L.meta);
    a.memo = (MemoEntry *)(ws + L.memo);
    a.curmask = (unsigned long long *)(ws + L.curmask);
    a.zeros = (int32_t *)(ws + L.zeros);
    a.colpack = (unsigned long long *)(ws + L.colpack);
    a.need_constraints = (violations != nullptr || !(d->flags & PX_FLAG_NO_CONSTRAINT_CHECK)) ? 1 : 0;
    if (first_rank > 0) {
        a.sel = (const int32_t *)(ws + L.order) + first_rank;
        a.n_sel = d->P - first_rank;
    }
    a.fitness = fitness; a.best_goodput = best_goodput; a.speedup = speedup;
    a.best_m = best_m; a.best_s = best_s; a.violations = violations;
    return a;
}

// The sampling argmax of a pair depends on (job, K, one node or several) only, as the grid's does, and each of its list
// entries takes a last pass of Eq. 10 (no table holds it): from as many candidates on as a job has rows to take the argmax
// of (64, and one per GPU of the largest node), the call takes them once per row whether PX_FLAG_MEMOISE asks for it or
// not (200 jobs, 1000 candidates: 165 us a call with an argmax per pair, 30 so).  P is the same in all calls that
// share a workspace, so a generation finds the rows its fitness call has left.
static bool memoised(const pollux_dims &d)
{
    const bool sampled_rows = (d.flags & PX_FLAG_SAMPLE_M) != 0 && d.P >= 2 * kTableK && d.N >= 4 && d.N <= kMemoNodes;
    return (d.flags & PX_FLAG_MEMOISE) != 0 || sampled_rows;
}

bool generation_in_one(const pollux_dims &d, const pollux_ga_params &ga)
{
    return (ga.flags & PX_GA_INHERIT_ROWS) && (ga.flags & PX_GA_IN_PLACE) && !ga.job_gpu_cap && (int)ga.elite_k < d.P && memoised(d) &&
           !small_call(d) && d.N >= 4 && d.N <= kArrayNodes && d.J <= kFinishJobs;
}

int launch_generation(const pollux_dims *d, int32_t *population, const double *job_params, const int32_t *m_grid,
                      const int32_t *fair_share, const int32_t *current_alloc, const int32_t *node_capacity, double p,
                      double delta, const pollux_ga_params *ga, void *workspace, double *fitness, int32_t *best_m, int32_t *best_s,
                      double *best_goodput, double *speedup, int32_t *violations, hipStream_t stream)
{
    const FitnessArgs a = call_args(d, population, job_params, m_grid, fair_share, current_alloc, node_capacity, p, delta, workspace,
                                    fitness, best_m, best_s, best_goodput, speedup, violations, (int)ga->elite_k);
    const GaArgs g = ga_args(d, population, fitness, node_capacity, ga, workspace, population);
    launch_rank(g, stream);
    const size_t lds = ga_shared_bytes(d->J, d->N);
    const bool whole = (d->N & 3) == 0 && ((uintptr_t)population & 15) == 0;
    const int kind = (d->flags & PX_FLAG_SAMPLE_M) ? kMemoSampled : (d->precision == 1 ? kMemoF32 : kMemoGrid);
    const void *kernels[3][2] = {{(const void *)child_kernel<kMemoGrid, kRows64>, (const void *)child_kernel<kMemoGrid, kRows64Whole>},
                                 {(const void *)child_kernel<kMemoF32, kRows64>, (const void *)child_kernel<kMemoF32, kRows64Whole>},
                                 {(const void *)child_kernel<kMemoSampled, kRows64>, (const void *)child_kernel<kMemoSampled, kRows64Whole>}};
    static_assert(kMemoGrid == 0 && kMemoF32 == 1 && kMemoSampled == 2, "the rows above");
    static size_t allowed[3][2][kGaDevices];
    const int rc = allow_dynamic_lds(kernels[kind][whole], lds, allowed[kind][whole]);
    if (rc != PX_OK) return rc;
    void *args[] = {(void *)&g, (void *)&a};
    if (hipLaunchKernel(kernels[kind][whole], dim3((unsigned)(d->P - (int)ga->elite_k)), dim3(kGaThreads), args, lds, stream) != hipSuccess)
        return PX_E_HIP;
    return hipGetLastError() == hipSuccess ? PX_OK : PX_E_HIP;
}

int launch_fitness(const pollux_dims *d, const int32_t *population, const double *job_params, const int32_t *m_grid,
                   const int32_t *fair_share, const int32_t *current_alloc, const int32_t *node_capacity, double p,
                   double delta, void *workspace, double *fitness, int32_t *best_m, int32_t *best_s,
                   double *best_goodput, double *speedup, int32_t *violations, hipEvent_t sweep_start,
                   hipEvent_t sweep_stop, int first_rank, bool inherit_rows, hipStream_t stream)
{
    const WorkspaceLayout L = workspace_layout(*d);
    char *ws = (char *)workspace;
    FitnessArgs a = call_args(d, population, job_params, m_grid, fair_share, current_alloc, node_capacity, p, delta, workspace, fitness,
                              best_m, best_s, best_goodput, speedup, violations, first_rank);
    const int P_eff = first_rank > 0 ? d->P - first_rank : d->P;
    if (P_eff <= 0) return PX_OK;

    // unrolled s-chunk: the smallest of 8, 16, 24, 32 that covers Gs (32 with several chunks beyond that).  (21 counts in a chunk
    // of 24, and table rows staged in LDS on grids that are no whole groups of 64 too: 1021 candidates of 331 jobs with 50
    // batch sizes 140 us a call, 159 without either.)
    const int ch = d->Gs <= 8 ? 8 : (d->Gs <= 16 ? 16 : (d->Gs <= 24 ? 24 : 32));
    const bool inherit = inherit_rows && first_rank > 0;
    const bool row1 = d->N >= 4 && d->N <= 4 * kWave;
    const bool aligned = row1 && (d->N & 3) == 0 && (((uintptr_t)population | (uintptr_t)current_alloc) & 15) == 0;
    const bool whole = d->Gm % kWave == 0;
    const bool near = a.gs_pad <= kNearRecips;      // the kernels keep reciprocals and thresholds of all counts in LDS
    // four rows per load of a wavefront (cand_per_wave <= 16 holds); its sweeps pack a batch size's index into 15 bits
    const bool row4 = row1 && d->N <= kWave && d->Gm <= 0x7FFF && near && !(d->flags & PX_FLAG_SAMPLE_M);
    const bool sampled = (d->flags & PX_FLAG_SAMPLE_M) != 0;       // fp64 only (checked by the caller)
    const PairSplit split = balanced_split(split_pairs(P_eff, d->J, d->Gm, d->Gs, d->precision == 1, row4, aligned && whole, inherit, row1, sampled),
                                           P_eff, d->J, d->Gm, d->Gs, d->precision == 1, row4, inherit, row1, sampled);
    a.cand_per_wave = split.per_wave;
    a.stage_rows = d->Gm <= kStageGm && near && split.per_wave >= stage_candidates(a.sel != nullptr) ? 1 : 0;
    a.cand_groups = pair_groups(P_eff, split.per_wave);
    const unsigned pair_blocks = (unsigned)(8 * ((d->J + 7) / 8) * a.cand_groups);

    const bool f32 = d->precision == 1;
    if (small_call(*d)) {
        if (sweep_start) (void)hipEventRecord(sweep_start, stream);
        const bool kept = (d->flags & PX_FLAG_KEEP_JOB_TABLES) != 0, halves = d->Gm <= kSmallHalf;
        const dim3 grid((unsigned)P_eff), block((unsigned)small_threads(*d, kept));
        if (kept && halves) hipLaunchKernelGGL((small_kernel<true, true>), grid, block, 0, stream, a);
        else if (halves) hipLaunchKernelGGL((small_kernel<false, true>), grid, block, 0, stream, a);
        else if (kept) hipLaunchKernelGGL((small_kernel<true, false>), grid, block, 0, stream, a);
        else hipLaunchKernelGGL((small_kernel<false, false>), grid, block, 0, stream, a);
        if (sweep_stop) (void)hipEventRecord(sweep_stop, stream);
        return hipGetLastError() == hipSuccess ? PX_OK : PX_E_HIP;
    }
    const bool memo = memoised(*d);
    // The per-node counters start every call at zero.  A call that uses them leaves them at zero again
    // (candidates_kernel clears what it reads), so a call that keeps the job tables, whose caller guarantees an
    // untouched workspace and unchanged dimensions, does not clear them once more.
    // memoised pass over rows of 4 to 256 entries: one workgroup per candidate, counters in LDS, fitness included
    const bool candidate_pass = memo && d->N >= 4 && d->N <= kMemoNodes;
    if (inherit) {
        // the children of the step that has just run: unchanged rows take over their source's results
        a.src_row = (const int32_t *)(ws + L.src_row);
        a.odd = (const int32_t *)(ws + L.odd);
    }
    if (inherit && !candidate_pass) {
        // the other rows are listed per job and go through the population pass below like any pair
        a.dirty_count = (int32_t *)(ws + L.dirty_count);
        a.dirty = (int32_t *)(ws + L.dirty);
        hipLaunchKernelGGL(inherit_kernel, dim3((unsigned)P_eff), dim3(256), 0, stream, a);
    }
    // done by prepare_kernel, i.e. not by a call that keeps the job tables; the candidate pass keeps its counters on chip
    a.clear_counters = candidate_pass ? 0 : 1;
    if (!(d->flags & PX_FLAG_KEEP_JOB_TABLES)) {
        // everything that depends on the jobs only (not on the population)
        a.or_job_status = 1;
        if (sampled && memo) launch_prepare_rows<kPrepSampledMemo>(a, stream);
        else if (sampled) launch_prepare_rows<kPrepSampled>(a, stream);
        else if (f32 && d->Gs <= kSmallGs) launch_prepare_rows<kPrepTablesF32>(a, stream);
        else if (f32) launch_prepare_rows<kPrepTables>(a, stream);
        else if (memo) launch_prepare_rows<kPrepMemo>(a, stream);
        else launch_prepare_rows<kPrepPlain>(a, stream);
        if (f32) {
            const dim3 job_grid((unsigned)((d->J + kWavesPerBlock - 1) / kWavesPerBlock));
            // (up to kSmallGs counts found with everything else: 200 jobs a call of 74.6 us with a launch for them, 69.5 without)
            if (d->Gs > kSmallGs) hipLaunchKernelGGL(jobs_kernel_f32, job_grid, dim3(256), 0, stream, a);
            if (memo) {
                const dim3 memo_grid((unsigned)(((long long)d->J * 2 * kTableK + kWavesPerBlock - 1) / kWavesPerBlock));
                if (ch == 8) hipLaunchKernelGGL((memo_kernel_f32<8>), memo_grid, dim3(256), 0, stream, a);
                else hipLaunchKernelGGL((memo_kernel_f32<16>), memo_grid, dim3(256), 0, stream, a);
            }
        }
    }
    if (sweep_start) (void)hipEventRecord(sweep_start, stream);
#define PX_LAUNCH_PAIRS(CH, F32, MEMO, ROW1, WHOLE, ROW4, RAG)                                                               \
    do {                                                                                                                     \
        if (a.dirty) hipLaunchKernelGGL((pairs_kernel<CH, F32, MEMO, ROW1, WHOLE, ROW4, RAG, 2>), dim3(pair_blocks), dim3(256), 0, stream, a); \
        else if (a.sel) hipLaunchKernelGGL((pairs_kernel<CH, F32, MEMO, ROW1, WHOLE, ROW4, RAG, 1>), dim3(pair_blocks), dim3(256), 0, stream, a); \
        else hipLaunchKernelGGL((pairs_kernel<CH, F32, MEMO, ROW1, WHOLE, ROW4, RAG, 0>), dim3(pair_blocks), dim3(256), 0, stream, a); \
    } while (0)
    // the instance for the row length (four rows per load, one row per load, any) and the grid (whole groups of 64 batch sizes or not).
    // Ragged rows of at most 64 nodes with fewer than four candidates a wavefront go entry by entry, a lane each (64 x 500 x 17 with
    // 500 batch sizes 47.0 us against 51.2 in 16-byte loads), but for the children of a generation (76 against 44).
    constexpr int kSwept = kFourRowsSwept, kLoaded = kFourRowsLoaded, kOne = kRowAtATime;
    const bool entries = !row1 || (row4 && !aligned && split.entry_by_entry && !a.sel);
#define PX_LAUNCH_PAIRS_GRID(CH, F32, FOUR)                                                          \
    do {                                                                                             \
        if (memo) PX_LAUNCH_PAIRS(16, F32, true, false, false, kOne, false);                         \
        else if (entries) PX_LAUNCH_PAIRS(CH, F32, false, false, false, kOne, false);                \
        else if (split.four && aligned && whole) PX_LAUNCH_PAIRS(CH, F32, false, true, true, FOUR, false);  \
        else if (split.four) PX_LAUNCH_PAIRS(CH, F32, false, true, false, FOUR, true);               \
        else if (aligned && whole) PX_LAUNCH_PAIRS(CH, F32, false, true, true, kOne, false);         \
        else if (aligned) PX_LAUNCH_PAIRS(CH, F32, false, true, false, kOne, false);                 \
        else if (whole) PX_LAUNCH_PAIRS(CH, F32, false, true, true, kOne, true);                     \
        else PX_LAUNCH_PAIRS(CH, F32, false, true, false, kOne, true);                               \
    } while (0)
    if (candidate_pass) {
        const bool pairs_kept = (d->flags & PX_FLAG_PAIR_RESULTS) != 0 || !(d->flags & PX_FLAG_MEMOISE);
        if (sampled) launch_memo_candidates<kMemoSampled>(a, P_eff, inherit, pairs_kept, stream);
        else if (f32) launch_memo_candidates<kMemoF32>(a, P_eff, inherit, pairs_kept, stream);
        else launch_memo_candidates<kMemoGrid>(a, P_eff, inherit, pairs_kept, stream);
        if (sweep_stop) (void)hipEventRecord(sweep_stop, stream);
        return hipGetLastError() == hipSuccess ? PX_OK : PX_E_HIP;
    } else if (sampled) {
        if (memo) PX_LAUNCH_PAIRS(0, false, true, false, false, kOne, false);
        else PX_LAUNCH_PAIRS(0, false, false, false, false, kOne, false);
    } else if (f32 && row4 && aligned && whole && !split.four && !memo) {
        if (ch == 8) PX_LAUNCH_PAIRS(8, true, false, true, true, kLoaded, false);
        else PX_LAUNCH_PAIRS(16, true, false, true, true, kLoaded, false);
    } else if (f32) {
        if (ch == 8) PX_LAUNCH_PAIRS_GRID(8, true, kSwept);
        else PX_LAUNCH_PAIRS_GRID(16, true, kSwept);
    } else if (ch == 8) {
        PX_LAUNCH_PAIRS_GRID(8, false, kSwept);
    } else if (ch == 16) {
        PX_LAUNCH_PAIRS_GRID(16, false, kSwept);
    } else if (ch == 24) {
        PX_LAUNCH_PAIRS_GRID(24, false, kLoaded);
    } else {
        PX_LAUNCH_PAIRS_GRID(32, false, kLoaded);
    }
#undef PX_LAUNCH_PAIRS_GRID
#undef PX_LAUNCH_PAIRS
    if (sweep_stop) (void)hipEventRecord(sweep_stop, stream);
    const dim3 candidates((unsigned)P_eff), threads(kCandThreads);
    if (d->J <= kCandThreads) {
        if (f32) hipLaunchKernelGGL((candidates_kernel<float, 1>), candidates, threads, 0, stream, a);
        else hipLaunchKernelGGL((candidates_kernel<double, 1>), candidates, threads, 0, stream, a);
    } else {
        if (f32) hipLaunchKernelGGL((candidates_kernel<float, 4>), candidates, threads, 0, stream, a);
        else hipLaunchKernelGGL((candidates_kernel<double, 4>), candidates, threads, 0, stream, a);
    }
    return hipGetLastError() == hipSuccess ? PX_OK : PX_E_HIP;
}

}  // namespace px
