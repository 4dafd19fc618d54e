// Batched fitting of theta_sys on gfx950 (Pollux, arXiv 2008.12260, Sec. 4.1 "Online
// model fitting" and "Prior-driven exploration"): for every job, the seven throughput
// parameters (Eq. 12) that minimise the root mean squared logarithmic error between
// Eq. 11 and the job's recorded (K, nodes, m, s, T_iter) tuples, with every alpha and
// beta >= 0 and 1 <= gamma <= 10, and with the parameters the exploration priors hold
// at zero.
//
// One workgroup per job, one wavefront per starting point.  The lanes of a wavefront share the
// job's records; of the seven unknowns lane i < 7 holds the i-th (value, scale, bounds, gradient, its row of the
// matrix to factorise), and what all lanes need of them travels through scalar registers.  The error is a sum of squares of
//     r_o = ln T_iter(theta; K_o, nodes_o, m_o, s_o) - ln T_o,
// so the minimiser is a damped Gauss-Newton (Levenberg-Marquardt) iteration on the box:
// per iteration the lanes form r_o and its seven partial derivatives, the wave reduces
// SUM r^2, J^T r (7 sums) and J^T J (28 sums) in a fixed binary tree (sum_terms),
// solves the damped 7 x 7 system on the variables that are free (not held by a prior,
// not at a bound with the gradient pointing outwards) by Cholesky factorisation, clips
// the step to the box and accepts it if SUM r^2 went down.  The unknowns are scaled by
// the starting point (they differ by four orders of magnitude).
//
// Eq. 10 is evaluated with the larger term factored out, as in the fitness kernels:
// with D = ln T_sync - ln T_grad and e = exp(-gamma |D|),
//     ln last = max(ln T_grad, ln T_sync) + log1p(e) / gamma,
//     w_s = T_sync^gamma / (T_grad^gamma + T_sync^gamma) = 1/(1+e) or e/(1+e),
//     d last / d T_grad = w_g last / T_grad,   d last / d T_sync = w_s last / T_sync,
//     d ln last / d gamma = (w_g ln T_grad + w_s ln T_sync) / gamma - ln(T_grad^gamma + T_sync^gamma) / gamma^2.

#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include "../../include/pollux.h"
#include "pollux_device.h"
#include "pollux_host.h"
#include "pollux_launch.h"
#include "pollux_math.h"

namespace px {

constexpr int kTheta = 7;                 // unknowns, in the order of the first seven PX_* rows
constexpr int kPacked = 28;               // lower triangle of a symmetric 7 x 7 matrix, row-major: (i, k <= i) at i(i+1)/2 + k
constexpr double kTgradFloor = 1e-12;     // keeps ln T_grad finite should alpha_grad = beta_grad = 0 ever be tried

struct FitArgs {
    int J, max_obs, max_iter, n_starts;
    const int32_t *count, *K, *nodes, *m, *s;
    const double *T, *init;
    double *theta, *rmsle;
    int32_t *iterations;
};

// The 36 sums over a wavefront, through LDS.  Sixteen at a time: every lane puts its terms into a row of its own, then lane
// 16 q + k adds term k of the sixteen lanes of quarter q, and the quarters are added across lanes.  A butterfly per sum was
// 648 vector instructions (six steps of two moves and an addition, 36 times) of an iteration's 1600; this is 120, in the same
// binary tree ((0+1)+(2+3)) + ..., so every sum has the same bits.  Rows of 17 doubles keep writes and reads off each other's
// banks.  The sums stay in LDS, where the solver reads them, and the unknowns are spread over lanes, so that four wavefronts fit
// a SIMD, not two, and the 3000 chains of 1000 jobs with three starts run side by side: 2.44 ms a call before, 1.15 so.  What is
// left is a chain of 3.5 us per iteration (100 jobs, 200 iterations: 0.70 ms), half of it the seven pivots of the solver.
constexpr int kSums = 1 + 7 + 28;                       // SUM r^2, J^T r, J^T J
constexpr int kSumRow = 17;
constexpr int kSumTable = 64 * kSumRow;                 // doubles of one wavefront's table of terms
constexpr int kWaveDoubles = kSumTable + 2 * kSums;     // and two sets of sums: of the iterate and of the trial

// What the lanes of a wavefront write becomes visible to all of them: the LDS serves a wavefront's accesses in order, so only
// the compiler has to keep them so.
__device__ __forceinline__ void wave_fence()
{
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// Lane 16 q + k: the sum of term FIRST + k over the lanes of quarter q (sixteen terms, or up to the last).
template <int FIRST>
__device__ __forceinline__ double sum_quarter(double *table, const double (&term)[kSums])
{
    constexpr int kCount = kSums - FIRST < 16 ? kSums - FIRST : 16;
    const int lane = lane_id();
    wave_fence();
#pragma unroll
    for (int k = 0; k < kCount; ++k) table[lane * kSumRow + k] = term[FIRST + k];
    wave_fence();
    const int k = lane & 15;
    const double *column = table + (lane & 48) * kSumRow + (k < kCount ? k : 0);
    double v[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) v[i] = column[i * kSumRow];
#pragma unroll
    for (int width = 1; width < 16; width *= 2) {
#pragma unroll
        for (int i = 0; i < 16; i += 2 * width) v[i] += v[i + width];
    }
    return v[0];
}

// All sums, to out[0 .. kSums-1].
__device__ __forceinline__ void sum_terms(double *table, const double (&term)[kSums], double *out)
{
    static_assert(kSums > 32 && kSums <= 48, "three passes of sixteen");
    double s0 = sum_quarter<0>(table, term), s1 = sum_quarter<16>(table, term), s2 = sum_quarter<32>(table, term);
    // the quarters, all three together so that their exchanges overlap
    s0 += exchange<4>(s0); s1 += exchange<4>(s1); s2 += exchange<4>(s2);
    s0 += exchange<5>(s0); s1 += exchange<5>(s1); s2 += exchange<5>(s2);
    const int lane = lane_id();
    if (lane < 16) {
        out[lane] = s0;
        out[16 + lane] = s1;
        if (lane < kSums - 32) out[32 + lane] = s2;
    }
    wave_fence();
}

// The value lane `src` holds, in every lane.
__device__ __forceinline__ double wave_read(double v, int src)
{
    return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), src), __builtin_amdgcn_readlane(__double2loint(v), src));
}

__device__ __forceinline__ double uniform_f64(double v)
{
    return __hiloint2double(__builtin_amdgcn_readfirstlane(__double2hiint(v)),
                            __builtin_amdgcn_readfirstlane(__double2loint(v)));
}

// One recorded tuple in the form the iteration uses it.
struct Record {
    int K, nodes;
    double md, sd, lnT;
};

__device__ __forceinline__ Record load_record(const FitArgs &f, size_t at)
{
    Record r;
    r.K = f.K[at]; r.nodes = f.nodes[at];
    r.md = (double)f.m[at]; r.sd = (double)f.s[at];
    r.lnT = px_log(f.T[at]);
    return r;
}

// The sums of one job at theta = z * scale (lane i < 7 holds the i-th of each), in `out` (LDS): SUM r^2, then J^T r, then J^T J as a packed lower triangle.
// mine: the l-th record of the job, read once and kept in lane l's registers over all iterations.  HELD: the job has no more than
// these 64; otherwise those beyond are read from memory in every evaluation.
template <bool HELD>
__device__ __forceinline__ void normal_equations(const FitArgs &f, int j, int n, double my_z, double my_scale, const Record &mine,
                                                 double *table, double *out)
{
    const int lane = lane_id();
    const double my_th = my_z * my_scale;
    double th[kTheta], scale[kTheta];
#pragma unroll
    for (int i = 0; i < kTheta; ++i) {
        th[i] = wave_read(my_th, i);
        scale[i] = wave_read(my_scale, i);
    }
    const double gamma = th[PX_GAMMA], inv_gamma = 1.0 / gamma;

    // the residual of one record and its derivatives with respect to z
    auto evaluate = [&](const Record &rec, double &r, double (&d)[kTheta]) {
        const int K = rec.K, nodes = rec.nodes;
        const double md = rec.md, sd = rec.sd;
        const double lnT = rec.lnT;
        double tg = th[PX_ALPHA_G] + th[PX_BETA_G] * md;                                  // Eq. 8
        tg = tg > kTgradFloor ? tg : kTgradFloor;
        const bool local = K > 1 && nodes == 1, node = K > 1 && nodes != 1;
        const double km2 = (double)(K - 2);
        double ts = 0.0;                                                                  // Eq. 9
        if (local) ts = th[PX_ALPHA_SL] + th[PX_BETA_SL] * km2;
        if (node) ts = th[PX_ALPHA_SN] + th[PX_BETA_SN] * km2;
        double last = tg, dl_dtg = 1.0, dl_dts = gamma == 1.0 ? 1.0 : 0.0, dlnl_dg = 0.0;
        if (ts > 0.0) {                                                                   // Eq. 10
            const double lntg = px_log(tg), lnts = px_log(ts);
            const double d = lnts - lntg;
            const double e = px_exp(-gamma * fabs(d));
            const double l1p = px_log1p_unit(e);
            const double big = d >= 0.0 ? ts : tg, lnbig = d >= 0.0 ? lnts : lntg;
            last = big * px_exp(l1p * inv_gamma);
            const double w_small = px_div(e, 1.0 + e), w_big = px_div(1.0, 1.0 + e);
            const double w_s = d >= 0.0 ? w_big : w_small, w_g = d >= 0.0 ? w_small : w_big;
            dl_dtg = w_g * px_div(last, tg);
            dl_dts = w_s * px_div(last, ts);
            const double lnsum = gamma * lnbig + l1p;                                     // ln(T_grad^g + T_sync^g)
            dlnl_dg = (w_g * lntg + w_s * lnts) * inv_gamma - lnsum * inv_gamma * inv_gamma;
        }
        const double pred = sd * tg + last;                                               // Eq. 11
        r = px_log(pred) - lnT;
        const double inv_pred = px_div(1.0, pred);
        d[PX_ALPHA_G] = (sd + dl_dtg) * inv_pred;
        d[PX_BETA_G] = d[PX_ALPHA_G] * md;
        const double dts = dl_dts * inv_pred;
        d[PX_ALPHA_SL] = local ? dts : 0.0;
        d[PX_BETA_SL] = local ? dts * km2 : 0.0;
        d[PX_ALPHA_SN] = node ? dts : 0.0;
        d[PX_BETA_SN] = node ? dts * km2 : 0.0;
        d[PX_GAMMA] = last * dlnl_dg * inv_pred;
#pragma unroll
        for (int i = 0; i < kTheta; ++i) d[i] *= scale[i];
    };
    double term[kSums];
    // the record's terms: r^2; d_i r; d_i d_k, k <= i, row by row
    auto add = [&](double r, const double (&d)[kTheta]) {
        term[0] = px_fma(r, r, term[0]);
#pragma unroll
        for (int i = 0; i < kTheta; ++i) {
            term[1 + i] = px_fma(d[i], r, term[1 + i]);
#pragma unroll
            for (int k = 0; k <= i; ++k) term[1 + kTheta + i * (i + 1) / 2 + k] = px_fma(d[i], d[k], term[1 + kTheta + i * (i + 1) / 2 + k]);
        }
    };
#pragma unroll
    for (int t = 0; t < kSums; ++t) term[t] = 0.0;
    const size_t base = (size_t)j * f.max_obs;
    for (int o0 = 0; o0 < (HELD ? 1 : n); o0 += kWave) {
        const int o = o0 + lane;
        Record rec = mine;
        if (!HELD && o0 > 0) rec = load_record(f, base + (size_t)(o < n ? o : n - 1));
        double r, d[kTheta];
        evaluate(rec, r, d);
        if (o >= n) {
            r = 0.0;
#pragma unroll
            for (int i = 0; i < kTheta; ++i) d[i] = 0.0;
        }
        add(r, d);
    }
    sum_terms(table, term, out);
}

// Solves (A + lambda diag(A)) x = -g on the free variables (bit i of `held` set: x_i = 0) by Cholesky factorisation.
// Lane i < 7 holds row i and returns x_i; per column the pivot, its reciprocal (one division; the entries below it and both
// substitutions multiply by it) and the column's entries are known to all lanes.  Every entry takes its subtractions in
// ascending order of the column, as in the textbook's row-by-row form.  Returns false if a pivot is not positive.
__device__ __forceinline__ bool damped_step(const double *sums, double lambda, unsigned held, double &x)
{
    const int lane = lane_id();
    const int row = lane < kTheta ? lane : kTheta - 1;                  // (the lanes beyond repeat the last row)
    const double *g = sums + 1, *a = sums + 1 + kTheta;
    const bool mine_held = (held >> row) & 1u;
    const double dii = a[row * (row + 3) / 2];
    const double diagonal = mine_held ? 1.0 : dii + lambda * (dii > 1e-300 ? dii : 1e-300);
    double w[kTheta];
#pragma unroll
    for (int k = 0; k < kTheta; ++k) {
        const double entry = a[row * (row + 1) / 2 + k];                // (right of the diagonal: some other entry, never used)
        w[k] = row == k ? diagonal : ((mine_held || ((held >> k) & 1u)) ? 0.0 : entry);
    }
    double b = mine_held ? 0.0 : -g[row];
    double l[kPacked], inv[kTheta], y[kTheta];
#pragma unroll
    for (int k = 0; k < kTheta; ++k) {
        const double pivot = wave_read(w[k], k);
        if (!(pivot > 0.0)) return false;
        inv[k] = 1.0 / sqrt(pivot);
        const double column = w[k] * inv[k];
        y[k] = wave_read(b, k) * inv[k];
        b = px_fma(-column, y[k], b);
#pragma unroll
        for (int i = k + 1; i < kTheta; ++i) {
            l[i * (i + 1) / 2 + k] = wave_read(column, i);
            w[i] = px_fma(-column, l[i * (i + 1) / 2 + k], w[i]);
        }
    }
#pragma unroll
    for (int i = kTheta - 1; i >= 0; --i) {
        double s = y[i];
#pragma unroll
        for (int t = i + 1; t < kTheta; ++t) s = px_fma(-l[t * (t + 1) / 2 + i], y[t], s);
        y[i] = s * inv[i];
        x = lane == i ? y[i] : x;
    }
    return true;
}

constexpr int kMaxStarts = 5;

// Dynamic LDS: kWaveDoubles doubles per wavefront.  HELD: no job has more than 64 records.
template <bool HELD>
__global__ void __launch_bounds__(64 * kMaxStarts) __attribute__((amdgpu_waves_per_eu(3, 8))) fit_theta_kernel(FitArgs f)
{
    extern __shared__ __align__(16) double fit_lds[];
    __shared__ double end_sse[kMaxStarts];
    __shared__ double end_z[kMaxStarts][kTheta];
    __shared__ int end_it[kMaxStarts];
    const int j = blockIdx.x;
    const int lane = lane_id();
    const int k = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));      // this wavefront's starting point
    const int n = f.count[j] < f.max_obs ? f.count[j] : f.max_obs;
    if (n <= 0) {
        if (k == 0 && lane < kTheta) f.theta[(size_t)lane * f.J + j] = lane == PX_GAMMA ? 1.0 : 0.0;
        if (k == 0 && lane == 0) {
            f.rmsle[j] = 0.0;
            if (f.iterations) f.iterations[j] = 0;
        }
        return;
    }
    const size_t base = (size_t)j * f.max_obs;

    // what the job has explored, and the record with the shortest time per pass (first one on ties)
    int max_k = 0, max_nodes = 0;
    double best = __builtin_inf();
    int best_o = 0x7FFFFFFF;
    for (int o = lane; o < n; o += kWave) {
        const int K = f.K[base + o], nd = f.nodes[base + o];
        max_k = K > max_k ? K : max_k;
        max_nodes = nd > max_nodes ? nd : max_nodes;
        const double per_pass = f.T[base + o] / (double)(f.s[base + o] + 1);
        if (per_pass < best) { best = per_pass; best_o = o; }
    }
    max_k = (int)wave_max((unsigned)max_k);
    max_nodes = (int)wave_max((unsigned)max_nodes);
    {
        // positive doubles order like their bit patterns
        const unsigned hi = (unsigned)__double2hiint(best), lo = (unsigned)__double2loint(best);
        const unsigned hmin = wave_min(hi);
        const unsigned lmin = wave_min(hi == hmin ? lo : 0xFFFFFFFFu);
        best_o = wave_min((hi == hmin && lo == lmin) ? best_o : 0x7FFFFFFF);
        best = __hiloint2double((int)hmin, (int)lmin);
    }
    const double t_min = uniform_f64(best);
    // each lane keeps one record for the whole fit; usually there are no more
    Record mine = {1, 1, 1.0, 0.0, 0.0};
    if (lane < n) mine = load_record(f, base + lane);
    // (a job whose times are all infinite, NaN or negative has no such record: what is fitted to it is unspecified, what is read is its own)
    const double m_at = (double)f.m[base + (size_t)record_or_first(__builtin_amdgcn_readfirstlane(best_o), n)];

    // priors (Sec. 4.1, "Prior-driven exploration"): parameters without evidence are held at zero
    unsigned prior = 0u;
    if (max_k <= 1) prior |= (1u << PX_ALPHA_SL) | (1u << PX_BETA_SL) | (1u << PX_ALPHA_SN) | (1u << PX_BETA_SN);
    if (max_nodes <= 1) prior |= (1u << PX_ALPHA_SN) | (1u << PX_BETA_SN);
    if (max_k <= 2) prior |= (1u << PX_BETA_SL) | (1u << PX_BETA_SN);
    prior = (unsigned)__builtin_amdgcn_readfirstlane((int)prior);
    // lane i < 7: what the iteration keeps of unknown i (the lanes beyond hold nothing that is read)
    const bool is_sync = lane >= PX_ALPHA_SL && lane <= PX_BETA_SN, is_gamma = lane == PX_GAMMA;
    const bool my_prior = lane < kTheta && ((prior >> lane) & 1u);
    // the default starting value of this lane's sync parameter
    const double sync_default = (lane == PX_ALPHA_SL || lane == PX_ALPHA_SN) ? t_min / 10.0 : t_min / 100.0;
    double start = is_gamma ? 2.0 : (is_sync ? sync_default : (lane == PX_ALPHA_G ? t_min * 0.5 : t_min / (2.0 * m_at)));
    if (f.init && lane < kTheta) start = f.init[(size_t)lane * f.J + j];
    if (my_prior) start = 0.0;
    const double scale = (!is_gamma && start > 0.0) ? start : 1.0;
    const double lo = is_gamma ? 1.0 : 0.0, hi = is_gamma ? 10.0 : __builtin_inf();
    constexpr unsigned kAll = (1u << kTheta) - 1u;

    // The error has several local minima (and a flat spot at T_sync = 0 when gamma > 1), so the iteration is
    // run from a few starting points, one per wavefront, and the best end point is kept (the first one on
    // ties).  Start 0 is the start itself.  Starts 1 and 2 first minimise with gamma held at 1, where
    // Eq. 11 is linear in the alphas and betas, then release gamma from 2 and from 5 with the sync
    // parameters raised to at least a tenth of their starting values.  Starts 3 and 4 scale the sync
    // parameters by 3 and 0.3 and begin at gamma = 1.2 and 5.
    {
        const bool two_phase = k == 1 || k == 2;
        const double sync_factor = (k == 3) ? 3.0 : (k == 4 ? 0.3 : 1.0);
        const double gamma0 = (k == 0) ? wave_read(start, PX_GAMMA) : (k == 1 ? 2.0 : (k == 3 ? 1.2 : 5.0));
        double z;
        {
            double v = start;
            if (is_sync) v *= sync_factor;
            if (is_gamma) v = two_phase ? 1.0 : gamma0;
            v /= scale;
            z = v < lo ? lo : (v > hi ? hi : v);
        }

        double *table = fit_lds + k * kWaveDoubles, *cur = table + kSumTable, *trial = cur + kSums;
        double cur_sse = 0.0;
        int it = 0;
        // Up to four descents, written as one loop so that the iteration is in the code once (inlined four times it was 110 KB,
        // more than the instruction cache, and the wavefronts of a compute unit are all somewhere else in it): with gamma
        // held at 1 (two-phase starts), the descent proper, and one more for either sync pair that has ended at zero.
#pragma unroll 1
        for (int phase = two_phase ? 0 : 1; phase < 4; ++phase) {
            const double z_before = z, sse_before = cur_sse;
            if (phase >= 2) {
                // A sync pair that has ended at zero may only be stuck there: with T_sync = 0 and gamma > 1 the error
                // does not feel the pair at all (the flat spot).  It is put back to its default starting value once, the
                // others staying where they are, and the iteration is continued; the better end point is kept.
                const int ia = phase == 2 ? PX_ALPHA_SL : PX_ALPHA_SN, ib = ia + 1;
                const unsigned zero = (unsigned)__ballot(z == 0.0);
                const bool stuck = !((prior >> ia) & 1u) && ((zero >> ia) & 1u) && (((prior | zero) >> ib) & 1u);
                if (!(stuck && it < f.max_iter && cur_sse > 0.0)) continue;
                if (lane == ia) z = sync_default / scale;
            }
            // The damped Gauss-Newton iteration from z, until it converges or the budget of steps is spent; the
            // variables in `hold` stay where they are.  Leaves the end point in z and its error in cur_sse.
            const unsigned hold = phase == 0 ? prior | (1u << PX_GAMMA) : prior;
            double lambda = 1e-3, moved = 0.0, zn = z;
            bool first = true;
            for (;;) {
                normal_equations<HELD>(f, j, n, zn, scale, mine, table, trial);
                const double trial_sse = uniform_f64(trial[0]);
                if (first || trial_sse < cur_sse) {
                    const double gain = (cur_sse - trial_sse) / cur_sse;
                    z = zn;
                    double *sums = cur;
                    cur = trial;
                    trial = sums;
                    cur_sse = trial_sse;
                    if (!first) {
                        lambda = lambda * 0.2 > 1e-15 ? lambda * 0.2 : 1e-15;
                        if (gain < 1e-13 && moved < 1e-9) break;
                    }
                    first = false;
                } else {
                    lambda *= 5.0;
                    if (lambda > 1e15 || moved < 1e-15) break;
                }
                // the next trial point
                bool found = false;
                while (!found && it < f.max_iter && cur_sse > 0.0) {
                    ++it;
                    const double g = cur[1 + (lane < kTheta ? lane : 0)];
                    unsigned held = hold | ((unsigned)__ballot((z <= lo && g > 0.0) || (z >= hi && g < 0.0)) & kAll);
                    // a free variable that sits on a bound and would be pushed across it joins the held set
                    double step = 0.0;
                    bool solved = false;
#pragma unroll 1
                    for (int pass = 0; pass < kTheta + 1; ++pass) {
                        solved = damped_step(cur, lambda, held, step);
                        if (!solved) break;
                        const unsigned more = (unsigned)__ballot((z <= lo && step < 0.0) || (z >= hi && step > 0.0)) & kAll & ~held;
                        if (!more) break;
                        held |= more;
                    }
                    if (!solved) {
                        lambda *= 10.0;
                        if (lambda > 1e15) break;
                        continue;
                    }
                    const double v = ((held >> (lane & 31)) & 1u) ? z : z + step;
                    zn = v < lo ? lo : (v > hi ? hi : v);
                    // the largest relative change of an unknown (lanes 0 .. 7 among themselves)
                    const double rel = lane < kTheta ? fabs(zn - z) / (fabs(z) + 1e-12) : 0.0;
                    double most = rel > 0.0 ? rel : 0.0, other = exchange<0>(most);
                    most = other > most ? other : most;
                    other = exchange<1>(most);
                    most = other > most ? other : most;
                    other = exchange<2>(most);
                    most = other > most ? other : most;
                    moved = wave_read(most, 0);
                    if (moved == 0.0) break;
                    found = true;
                }
                if (!found) break;
            }
            if (phase == 0) {
                if (is_gamma) z = gamma0;
                const double least = 0.1 * sync_default / scale;
                if (is_sync && !my_prior && z < least) z = least;
            } else if (phase >= 2 && !(cur_sse < sse_before)) {
                z = z_before;
                cur_sse = sse_before;
            }
        }
        if (lane == 0) {
            end_sse[k] = cur_sse;
            end_it[k] = it;
        }
        if (lane < kTheta) end_z[k][lane] = z;
    }
    __syncthreads();
    if (k != 0) return;

    int best_k = 0, total_it = 0;
    for (int c = 0; c < f.n_starts; ++c) {
        total_it += end_it[c];
        if (end_sse[c] < end_sse[best_k]) best_k = c;
    }
    const double best_sse = end_sse[best_k];
    if (lane < kTheta) f.theta[(size_t)lane * f.J + j] = end_z[best_k][lane] * scale;
    if (lane == 0) {
        f.rmsle[j] = sqrt(best_sse / (double)n);
        if (f.iterations) f.iterations[j] = total_it;
    }
}

int launch_fit_theta(int J, int max_obs, int max_iter, int n_starts, const int32_t *count, const int32_t *K, const int32_t *nodes,
                     const int32_t *m, const int32_t *s, const double *T, const double *init, double *theta,
                     double *rmsle, int32_t *iterations, hipStream_t stream)
{
    FitArgs f;
    f.J = J; f.max_obs = max_obs; f.max_iter = max_iter; f.n_starts = n_starts;
    f.count = count; f.K = K; f.nodes = nodes; f.m = m; f.s = s; f.T = T; f.init = init;
    f.theta = theta; f.rmsle = rmsle; f.iterations = iterations;
    const size_t lds = sizeof(double) * kWaveDoubles * (size_t)n_starts;
    const dim3 grid((unsigned)J), block(64 * (unsigned)n_starts);
    // The instance without the loop over further records needs 128 registers, not 162, so four wavefronts fit a SIMD: 1000 jobs of
    // up to 48 records in 48 slots 1062 us, in 65 slots 1148 with the other (1213 while that read every record in every
    // evaluation; 1000 jobs of up to 128 records 1345).
    if (max_obs <= kWave) hipLaunchKernelGGL(fit_theta_kernel<true>, grid, block, lds, stream, f);
    else hipLaunchKernelGGL(fit_theta_kernel<false>, grid, block, lds, stream, f);
    return hipGetLastError() == hipSuccess ? PX_OK : PX_E_HIP;
}

}  // namespace px
