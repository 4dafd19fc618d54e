// Batched fitting of theta_sys on gfx950 (Pollux, arXiv 2008.12260, Sec. 4.1 "Online
// model fitting" and "Prior-driven exploration"): for every job, the seven throughput
// parameters (Eq. 12) that minimise the root mean squared logarithmic error between
// Eq. 11 and the job's recorded (K, nodes, m, s, T_iter) tuples, with every alpha and
// beta >= 0 and 1 <= gamma <= 10, and with the parameters the exploration priors hold
// at zero.
//
// One workgroup per job, one wavefront per starting point.  The lanes of a wavefront share the
// job's records; of the seven unknowns lanes 2 i and 2 i + 1 hold the i-th (value, scale, bounds, gradient, its row of
// the matrix to factorise), and what all lanes need of them travels through scalar registers.  The error is a sum of squares of
//     r_o = ln T_iter(theta; K_o, nodes_o, m_o, s_o) - ln T_o,
// so the minimiser is a damped Gauss-Newton (Levenberg-Marquardt) iteration on the box:
// per iteration the lanes form r_o and its seven partial derivatives, the wave reduces
// SUM r^2, J^T r (7 sums) and J^T J (24 sums) in a fixed binary tree (sum_terms),
// solves the damped 7 x 7 system on the variables that are free (not held by a prior,
// not at a bound with the gradient pointing outwards) by Cholesky factorisation, clips
// the step to the box and accepts it if SUM r^2 went down.  The unknowns are scaled by
// the starting point (they differ by four orders of magnitude).
//
// Bound by the vector ALU's issue, wavefront by wavefront: an instruction, scalar ones included, takes four cycles whether it
// waits for the one before it or not, so what counts is how many there are.  An iteration is 840 (1240 with the sums through
// LDS, the library's roots and divisions and the polynomials' constants formed where they are used), 540 where the trial point
// is refused, as half of them are: its error is summed first, and only a point that is taken gets derivatives and the other
// sums.  1000 jobs of up to 48 records with three starts, ms: 1.1 to 1.18 with the first of these forms, 0.77 to 0.82 with all sums
// for every point, 0.69 to 0.71 now; 80 jobs with one start 0.39 and 0.36 (0.98 to 1.03 times where nearly every point is taken).
// Beyond 256 jobs SIMDs hold two chains and three, and the slowest job is the one whose neighbours are slow (two chains of 200
// iterations on one SIMD take 1.45 times as long as one alone).  Every result has the same bits: on the flat stretches of this error
// other roundings end at other parameters.
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

#include <type_traits>

#include "../../include/pollux.h"
#include "pollux_device.h"
#include "pollux_host.h"
#include "pollux_launch.h"
#include "pollux_math.h"

namespace px {

constexpr int kTheta = 7;                 // unknowns, in the order of the first seven PX_* rows
constexpr double kTgradFloor = 1e-12;     // keeps ln T_grad finite should alpha_grad = beta_grad = 0 ever be tried

struct FitArgs {
    int J, max_obs, max_iter, n_starts;
    const int32_t *count, *K, *nodes, *m, *s;
    const double *T, *init;
    double *theta, *rmsle;
    int32_t *iterations;
};

// The sums over a wavefront: SUM r^2, J^T r, J^T J.  A record is a local or a distributed one, so its derivative with respect to
// one of the two sync pairs is zero and the four sums that mix the pairs are too: 32 sums remain, one per pair of lanes.
// Sum t ends in lanes 2 t and 2 t + 1:
//   0 .. 6  J^T r      7  SUM r^2      8 ..  the entries (i, k <= i) of J^T J, kOrder
constexpr int kSums = 32;
struct SumOrder {
    int row[kSums], column[kSums];       // of J^T J (8 ..)
    int at[kTheta][kTheta];              // the sum of entry (i, k <= i), -1: zero
};
constexpr SumOrder make_order()
{
    SumOrder o = {};
    int t = 8;
    for (int i = 0; i < kTheta; ++i) {
        for (int k = 0; k <= i; ++k) {
            const bool mixed = (i == PX_ALPHA_SN || i == PX_BETA_SN) && (k == PX_ALPHA_SL || k == PX_BETA_SL);
            o.at[i][k] = mixed ? -1 : t;
            if (!mixed) {
                o.row[t] = i;
                o.column[t++] = k;
            }
        }
    }
    return o;
}
constexpr SumOrder kOrder = make_order();

// Unknown i belongs to lanes 2 i and 2 i + 1, and has both their bits in the sets of unknowns below.
constexpr unsigned unknown(int i) { return 3u << (2 * i); }
constexpr unsigned kAll = (1u << (2 * kTheta)) - 1u;
constexpr int kRowDoubles = 8;                          // a row of the system in LDS: its entries, and the right-hand side
constexpr int kWaveDoubles = (kTheta + 1) * kRowDoubles;  // of one wavefront (the last row: what belongs to none)

// What the lanes of a wavefront write becomes visible to all of them: the LDS serves a wavefront's accesses in order, so only
// the compiler has to keep them so.
__device__ __forceinline__ void wave_fence()
{
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// Lane l holds record bit_reversed(l), so the tree ((0+1)+(2+3)) + ... over the records begins with lanes 32 apart, which
// gfx950 exchanges between two registers by one instruction, as it does rows of 16 lanes; and at every level a lane hands
// half of its sums to its partner, so 32 values become one in 16 + 8 + 4 + 2 + 1 + 1 additions.  (Through a table in LDS, as it was
// before, the stores alone took 15 cycles each, an eighth of an iteration.)
__device__ __forceinline__ int bit_reversed(int lane) { return (int)(__builtin_bitreverse32((unsigned)lane) >> 26); }

// Lanes of the lower half: x of the lane and of the one 32 above; of the upper half: y of the lane and of the one 32 below.
__device__ __forceinline__ double add_halves(double x, double y)
{
    const auto lo = __builtin_amdgcn_permlane32_swap((unsigned)__double2loint(x), (unsigned)__double2loint(y), false, false);
    const auto hi = __builtin_amdgcn_permlane32_swap((unsigned)__double2hiint(x), (unsigned)__double2hiint(y), false, false);
    return __hiloint2double((int)hi[0], (int)lo[0]) + __hiloint2double((int)hi[1], (int)lo[1]);
}

// The same for rows of 16 lanes: rows 0 and 2 x, rows 1 and 3 y.
__device__ __forceinline__ double add_rows(double x, double y)
{
    const auto lo = __builtin_amdgcn_permlane16_swap((unsigned)__double2loint(x), (unsigned)__double2loint(y), false, false);
    const auto hi = __builtin_amdgcn_permlane16_swap((unsigned)__double2hiint(x), (unsigned)__double2hiint(y), false, false);
    return __hiloint2double((int)hi[0], (int)lo[0]) + __hiloint2double((int)hi[1], (int)lo[1]);
}

// The same for lanes FAR = 8 or 4 apart: the lanes without that bit x, the others y.  The banks of four lanes that want the
// shifted y take it over the shifted x.
template <int FAR>
__device__ __forceinline__ int fetch(int x, int y)
{
    if constexpr (FAR == 8) {                            // row_ror:8
        const int v = __builtin_amdgcn_mov_dpp(x, 0x128, 0xF, 0xF, true);
        return __builtin_amdgcn_update_dpp(v, y, 0x128, 0xF, 0xC, false);
    } else {                                             // row_shl:4 (from the lane four above), row_shr:4
        const int v = __builtin_amdgcn_mov_dpp(x, 0x104, 0xF, 0xF, true);
        return __builtin_amdgcn_update_dpp(v, y, 0x114, 0xF, 0xA, false);
    }
}

template <int FAR>
__device__ __forceinline__ double add_near(double x, double y)
{
    const double mine = (lane_id() & FAR) != 0 ? y : x;
    return mine + __hiloint2double(fetch<FAR>(__double2hiint(x), __double2hiint(y)), fetch<FAR>(__double2loint(x), __double2loint(y)));
}

// All sums: sum t in lanes 2 t and 2 t + 1.
__device__ __forceinline__ double sum_terms(const double (&term)[kSums])
{
    double v[16];
#pragma unroll
    for (int t = 0; t < 16; ++t) v[t] = add_halves(term[t], term[t + 16]);
#pragma unroll
    for (int t = 0; t < 8; ++t) v[t] = add_rows(v[t], v[t + 8]);
#pragma unroll
    for (int t = 0; t < 4; ++t) v[t] = add_near<8>(v[t], v[t + 4]);
#pragma unroll
    for (int t = 0; t < 2; ++t) v[t] = add_near<4>(v[t], v[t + 2]);
    const bool second = (lane_id() & 2) != 0;
    const double mine = second ? v[1] : v[0], other = second ? v[0] : v[1];
    const double sum = mine + exchange<1>(other);
    return sum + exchange<0>(sum);
}

// The sum of one term alone, in every lane, in the same tree: what sum_terms leaves in its lanes, bit by bit.
__device__ __forceinline__ double sum_term(double term)
{
    double v = add_halves(term, term);
    v = add_rows(v, v);
    v += rotate16<8>(v);                     // (from here on lanes eight apart hold the same: four further on is as good as lane ^ 4)
    v += rotate16<4>(v);
    v += exchange<1>(v);
    return v + exchange<0>(v);
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

// What all lanes need of a trial point theta = z * scale (lanes 2 i and 2 i + 1 hold z_i).
struct Theta {
    double th[kTheta], inv_gamma;
};

__device__ __forceinline__ Theta make_theta(double my_z, double my_scale)
{
    Theta p;
    const double my_th = my_z * my_scale;
#pragma unroll
    for (int i = 0; i < kTheta; ++i) p.th[i] = wave_read(my_th, 2 * i);
    p.inv_gamma = px_div(1.0, p.th[PX_GAMMA]);
    return p;
}

// One record at a trial point: the prediction and what its derivatives are made of (lntg .. l1p only where ts > 0).
struct Prediction {
    double tg, ts, lntg, lnts, d, e, l1p, last, pred;
};

__device__ __forceinline__ Prediction predict(const Theta &p, const Record &rec, const Coefs &c)
{
    Prediction q = {};
    q.tg = p.th[PX_ALPHA_G] + p.th[PX_BETA_G] * rec.md;                               // Eq. 8
    q.tg = q.tg > kTgradFloor ? q.tg : kTgradFloor;
    const bool local = rec.K > 1 && rec.nodes == 1, node = rec.K > 1 && rec.nodes != 1;
    const double km2 = (double)(rec.K - 2);
    q.ts = 0.0;                                                                       // Eq. 9
    if (local) q.ts = p.th[PX_ALPHA_SL] + p.th[PX_BETA_SL] * km2;
    if (node) q.ts = p.th[PX_ALPHA_SN] + p.th[PX_BETA_SN] * km2;
    q.last = q.tg;
    if (q.ts > 0.0) {                                                                 // Eq. 10
        q.lntg = px_log(c, q.tg);
        q.lnts = px_log(c, q.ts);
        q.d = q.lnts - q.lntg;
        q.e = px_exp(c, -p.th[PX_GAMMA] * fabs(q.d));
        q.l1p = px_log1p_unit(c, q.e);
        q.last = (q.d >= 0.0 ? q.ts : q.tg) * px_exp(c, q.l1p * p.inv_gamma);
    }
    q.pred = rec.sd * q.tg + q.last;                                                  // Eq. 11
    return q;
}

// The residual (some: the lane holds a record; selected, not branched around).
__device__ __forceinline__ double residual(const Prediction &q, const Record &rec, bool some, const Coefs &c)
{
    double r = px_log(c, q.pred) - rec.lnT;
    asm("" : "+v"(r));
    return some ? r : 0.0;
}

// Its derivatives with respect to z.  In a lane without a record every one of them has the factor 1 / pred, which is made zero.
__device__ __forceinline__ void derivatives(const Theta &p, const Prediction &q, const Record &rec, bool some,
                                            const double (&scale)[kTheta], double (&d)[kTheta])
{
    const double gamma = p.th[PX_GAMMA], inv_gamma = p.inv_gamma;
    const bool local = rec.K > 1 && rec.nodes == 1, node = rec.K > 1 && rec.nodes != 1;
    const double km2 = (double)(rec.K - 2);
    double dl_dtg = 1.0, dl_dts = gamma == 1.0 ? 1.0 : 0.0, dlnl_dg = 0.0;
    if (q.ts > 0.0) {
        const double w_small = px_div(q.e, 1.0 + q.e), w_big = px_div(1.0, 1.0 + q.e);
        const double w_s = q.d >= 0.0 ? w_big : w_small, w_g = q.d >= 0.0 ? w_small : w_big;
        dl_dtg = w_g * px_div(q.last, q.tg);
        dl_dts = w_s * px_div(q.last, q.ts);
        const double lnsum = gamma * (q.d >= 0.0 ? q.lnts : q.lntg) + q.l1p;          // ln(T_grad^g + T_sync^g)
        dlnl_dg = (w_g * q.lntg + w_s * q.lnts) * inv_gamma - lnsum * inv_gamma * inv_gamma;
    }
    double inv_pred = px_div(1.0, q.pred);
    asm("" : "+v"(inv_pred));
    inv_pred = some ? inv_pred : 0.0;
    d[PX_ALPHA_G] = (rec.sd + dl_dtg) * inv_pred;
    d[PX_BETA_G] = d[PX_ALPHA_G] * rec.md;
    const double dts = dl_dts * inv_pred;
    d[PX_ALPHA_SL] = local ? dts : 0.0;
    d[PX_BETA_SL] = local ? dts * km2 : 0.0;
    d[PX_ALPHA_SN] = node ? dts : 0.0;
    d[PX_BETA_SN] = node ? dts * km2 : 0.0;
    d[PX_GAMMA] = q.last * dlnl_dg * inv_pred;
#pragma unroll
    for (int i = 0; i < kTheta; ++i) d[i] *= scale[i];
}

// The sums of one job at a trial point: sum t in lanes 2 t and 2 t + 1 (kOrder).  HELD: the job has no more than 64 records, each
// lane's (bit_reversed) is in its registers with its prediction and residual; otherwise the records beyond `mine` are read from
// memory in every evaluation.
template <bool HELD>
__device__ __forceinline__ double normal_equations(const FitArgs &f, int j, int n, const Theta &p, const double (&scale)[kTheta],
                                                   const Record &mine, const Prediction &at, double r_at, const Coefs &c)
{
    const int lane = lane_id();
    double term[kSums];
    // (a job whose records are all held has one a lane: its products as they are)
    auto accumulate = [](double a, double b, double to) { return HELD ? a * b : px_fma(a, b, to); };
    // the record's terms, in the order of kOrder
    auto add = [&](double r, const double (&d)[kTheta]) {
        term[7] = accumulate(r, r, term[7]);
#pragma unroll
        for (int i = 0; i < kTheta; ++i) {
            term[i] = accumulate(d[i], r, term[i]);
#pragma unroll
            for (int k = 0; k <= i; ++k) {
                if (kOrder.at[i][k] >= 0) term[kOrder.at[i][k]] = accumulate(d[i], d[k], term[kOrder.at[i][k]]);
            }
        }
    };
#pragma unroll
    for (int t = 0; t < kSums; ++t) term[t] = 0.0;
    double d[kTheta];
    if constexpr (HELD) {
        derivatives(p, at, mine, bit_reversed(lane) < n, scale, d);
        add(r_at, d);
    } else {
        const size_t base = (size_t)j * f.max_obs;
        for (int o0 = 0; o0 < n; o0 += kWave) {
            const int o = o0 + bit_reversed(lane);
            Record rec = mine;
            if (o0 > 0) rec = load_record(f, base + (size_t)(o < n ? o : n - 1));
            const Prediction q = predict(p, rec, c);
            derivatives(p, q, rec, o < n, scale, d);
            add(residual(q, rec, o < n, c), d);
        }
    }
    return sum_terms(term);
}

// One over the root of a pivot, from one chain of thirteen instructions (seed 2^-23, two steps of second order, a correction each),
// rounded as the library's root and division round it (30 and 12 instructions) for pivots well inside the exponent range.
__device__ __forceinline__ double inverse_root(double pivot)
{
    const double seed = __builtin_amdgcn_rsq(pivot);
    double root = pivot * seed, half = 0.5 * seed;                  // sqrt(pivot), 1 / (2 sqrt(pivot))
    double r = px_fma(-half, root, 0.5);
    root = px_fma(root, r, root);
    half = px_fma(half, r, half);
    r = px_fma(-half, root, 0.5);
    root = px_fma(root, r, root);
    half = px_fma(half, r, half);
    root = px_fma(px_fma(-root, root, pivot), half, root);
    const double near = half + half;
    return px_fma(px_fma(-root, near, 1.0), near, near);
}

// What lane 2 N of the lane's row of 16 holds, that is what belongs to unknown N.
template <int N>
__device__ __forceinline__ double of_unknown(double v)
{
    return __builtin_amdgcn_update_dpp(v, v, 0x150 + 2 * N, 0xF, 0xF, true);       // row_newbcast:2 N
}

// a - (x of unknown N) * y.  The multiply-add takes its operand across lanes itself; two instructions that are not vector
// writes of x have to lie in front of it.
#define PX_OF_UNKNOWN(N) " row_newbcast:" #N " row_mask:0xf bank_mask:0xf\n\t"
#define PX_LESS(A, X, N, Y) "v_fmac_f64_dpp " A ", -" X ", " Y PX_OF_UNKNOWN(N)

// Column K of the factorisation: what it takes from the entries to its right and from the right-hand side, the column itself
// and the right-hand side's share of it, and the next pivot.  Unknown i's lanes hold row i.
template <int K>
__device__ __forceinline__ void eliminate(double (&w)[kTheta], double &b, double inv, double &column, double &share, double &pivot)
{
#define PX_BEGIN "v_mul_f64 %0, %[k], %[i]\n\tv_mul_f64 %1, %[b], %[i]\n\ts_nop 0\n\t"
#define PX_NEXT(N) "v_mov_b64_dpp %2, %3" PX_OF_UNKNOWN(N)
#define PX_OUT "=&v"(column), "=&v"(share), "=&v"(pivot), "+v"(w[K + 1])
#define PX_IN [k] "v"(w[K]), [i] "v"(inv)
    if constexpr (K == 0)
        asm(PX_BEGIN PX_LESS("%3", "%0", 2, "%0") PX_LESS("%4", "%0", 4, "%0") PX_LESS("%5", "%0", 6, "%0") PX_LESS("%6", "%0", 8, "%0")
            PX_LESS("%7", "%0", 10, "%0") PX_LESS("%8", "%0", 12, "%0") PX_LESS("%[b]", "%1", 0, "%0") PX_NEXT(2)
            : PX_OUT, "+v"(w[2]), "+v"(w[3]), "+v"(w[4]), "+v"(w[5]), "+v"(w[6]), [b] "+v"(b) : PX_IN);
    else if constexpr (K == 1)
        asm(PX_BEGIN PX_LESS("%3", "%0", 4, "%0") PX_LESS("%4", "%0", 6, "%0") PX_LESS("%5", "%0", 8, "%0") PX_LESS("%6", "%0", 10, "%0")
            PX_LESS("%7", "%0", 12, "%0") PX_LESS("%[b]", "%1", 2, "%0") PX_NEXT(4)
            : PX_OUT, "+v"(w[3]), "+v"(w[4]), "+v"(w[5]), "+v"(w[6]), [b] "+v"(b) : PX_IN);
    else if constexpr (K == 2)
        asm(PX_BEGIN PX_LESS("%3", "%0", 6, "%0") PX_LESS("%4", "%0", 8, "%0") PX_LESS("%5", "%0", 10, "%0") PX_LESS("%6", "%0", 12, "%0")
            PX_LESS("%[b]", "%1", 4, "%0") PX_NEXT(6)
            : PX_OUT, "+v"(w[4]), "+v"(w[5]), "+v"(w[6]), [b] "+v"(b) : PX_IN);
    else if constexpr (K == 3)
        asm(PX_BEGIN PX_LESS("%3", "%0", 8, "%0") PX_LESS("%4", "%0", 10, "%0") PX_LESS("%5", "%0", 12, "%0") PX_LESS("%[b]", "%1", 6, "%0")
            PX_NEXT(8)
            : PX_OUT, "+v"(w[5]), "+v"(w[6]), [b] "+v"(b) : PX_IN);
    else if constexpr (K == 4)
        asm(PX_BEGIN PX_LESS("%3", "%0", 10, "%0") PX_LESS("%4", "%0", 12, "%0") PX_LESS("%[b]", "%1", 8, "%0") PX_NEXT(10)
            : PX_OUT, "+v"(w[6]), [b] "+v"(b) : PX_IN);
    else if constexpr (K == 5)
        asm(PX_BEGIN PX_LESS("%3", "%0", 12, "%0") PX_LESS("%[b]", "%1", 10, "%0") "s_nop 0\n\t" PX_NEXT(12)
            : PX_OUT, [b] "+v"(b) : PX_IN);
    else
        asm("v_mul_f64 %0, %1, %2" : "=v"(share) : "v"(b), "v"(inv));
#undef PX_BEGIN
#undef PX_NEXT
#undef PX_OUT
#undef PX_IN
}

// Back substitution: x_K is the right-hand side's share less the column's entries times x_{K+1} .., by the pivot's root.
// One block: the shares and columns it reads across lanes are written before it, by whatever instruction the compiler has put
// last (a copy, a reload), so it begins with the two wait states such a read needs; within it only x changes.
__device__ __forceinline__ void substitute(double (&x)[kTheta], const double (&column)[kTheta], const double (&share)[kTheta],
                                           const double (&inv)[kTheta])
{
#define PX_FIRST(K, N) "v_mov_b64_dpp %[x" #K "], %[s" #K "]" PX_OF_UNKNOWN(N)
#define PX_TAKE(K, T, N) PX_LESS("%[x" #K "]", "%[c" #K "]", N, "%[x" #T "]")
#define PX_LAST(K) "v_mul_f64 %[x" #K "], %[x" #K "], %[i" #K "]\n\t"
    asm("s_nop 1\n\t"
        PX_FIRST(6, 12) PX_LAST(6)
        PX_FIRST(5, 10) PX_TAKE(5, 6, 12) PX_LAST(5)
        PX_FIRST(4, 8) PX_TAKE(4, 5, 10) PX_TAKE(4, 6, 12) PX_LAST(4)
        PX_FIRST(3, 6) PX_TAKE(3, 4, 8) PX_TAKE(3, 5, 10) PX_TAKE(3, 6, 12) PX_LAST(3)
        PX_FIRST(2, 4) PX_TAKE(2, 3, 6) PX_TAKE(2, 4, 8) PX_TAKE(2, 5, 10) PX_TAKE(2, 6, 12) PX_LAST(2)
        PX_FIRST(1, 2) PX_TAKE(1, 2, 4) PX_TAKE(1, 3, 6) PX_TAKE(1, 4, 8) PX_TAKE(1, 5, 10) PX_TAKE(1, 6, 12) PX_LAST(1)
        PX_FIRST(0, 0) PX_TAKE(0, 1, 2) PX_TAKE(0, 2, 4) PX_TAKE(0, 3, 6) PX_TAKE(0, 4, 8) PX_TAKE(0, 5, 10) PX_TAKE(0, 6, 12) PX_LAST(0)
        : [x0] "=&v"(x[0]), [x1] "=&v"(x[1]), [x2] "=&v"(x[2]), [x3] "=&v"(x[3]), [x4] "=&v"(x[4]), [x5] "=&v"(x[5]), [x6] "=&v"(x[6])
        : [s0] "v"(share[0]), [s1] "v"(share[1]), [s2] "v"(share[2]), [s3] "v"(share[3]), [s4] "v"(share[4]), [s5] "v"(share[5]),
          [s6] "v"(share[6]), [c0] "v"(column[0]), [c1] "v"(column[1]), [c2] "v"(column[2]), [c3] "v"(column[3]), [c4] "v"(column[4]),
          [c5] "v"(column[5]), [i0] "v"(inv[0]), [i1] "v"(inv[1]), [i2] "v"(inv[2]), [i3] "v"(inv[3]), [i4] "v"(inv[4]),
          [i5] "v"(inv[5]), [i6] "v"(inv[6]));
#undef PX_FIRST
#undef PX_TAKE
#undef PX_LAST
}

// Solves the 7 x 7 system in LDS by Cholesky factorisation: unknown i's lanes hold row i (all four rows of 16 lanes do the
// same), everything that is about all rows comes across lanes as an operand of the multiply-add.  Every entry takes its
// subtractions in ascending order of the column.  PLAIN: roots and divisions of the library.
// Returns false if a pivot is not positive, or, not PLAIN, not well inside the exponent range.
template <bool PLAIN>
__device__ __forceinline__ bool solve(const double *system, double (&x)[kTheta])
{
    const int mine = (lane_id() & 15) >> 1, row = mine < kTheta ? mine : kTheta - 1;
    double w[kTheta], b, inv[kTheta], column[kTheta], share[kTheta];
    {
        const double2 *from = (const double2 *)(system + row * kRowDoubles);
        const double2 v0 = from[0], v1 = from[1], v2 = from[2], v3 = from[3];
        w[0] = v0.x; w[1] = v0.y; w[2] = v1.x; w[3] = v1.y; w[4] = v2.x; w[5] = v2.y; w[6] = v3.x;
        b = v3.y;
    }
    double pivot = of_unknown<0>(w[0]);
    bool good = true;
    unsigned off = 0u;                   // of the pivots' high words from that of 2^-900, the largest (negative, zero and NaN far off)
    auto column_of = [&](auto K) {
        constexpr int k = decltype(K)::value;
        if constexpr (PLAIN) {
            good = good && pivot > 0.0;
            inv[k] = 1.0 / sqrt(pivot);
        } else {
            const unsigned d = (unsigned)__double2hiint(pivot) - ((1023u - 900u) << 20);
            off = d > off ? d : off;
            inv[k] = inverse_root(pivot);
        }
        eliminate<k>(w, b, inv[k], column[k], share[k], pivot);
    };
    column_of(std::integral_constant<int, 0>());
    column_of(std::integral_constant<int, 1>());
    column_of(std::integral_constant<int, 2>());
    column_of(std::integral_constant<int, 3>());
    column_of(std::integral_constant<int, 4>());
    column_of(std::integral_constant<int, 5>());
    column_of(std::integral_constant<int, 6>());
    if (!PLAIN) good = off <= (1800u << 20);
    if (__builtin_amdgcn_readfirstlane((int)good) == 0) return false;
    substitute(x, column, share, inv);
    return true;
}
#undef PX_LESS
#undef PX_OF_UNKNOWN

// What a lane does with its sum when a system is set up: the unknowns the sum belongs to, and where it goes.
struct SumLane {
    unsigned unknowns;
    int place;                           // in the system in LDS
    unsigned long long row;              // of a diagonal entry: the lanes of all sums its unknown belongs to
    bool gradient, diagonal;
};

constexpr unsigned long long lanes_of_unknown(int i)
{
    unsigned long long lanes = 3ull << (2 * i);
    for (int t = 8; t < kSums; ++t) {
        if (kOrder.row[t] == i || kOrder.column[t] == i) lanes |= 3ull << (2 * t);
    }
    return lanes;
}

__device__ __forceinline__ SumLane sum_lane()
{
    const int t = lane_id() >> 1;
    SumLane me = {t < kTheta ? 3u << (2 * t) : 0u, t * kRowDoubles + kTheta, 0ull, t < kTheta, false};     // (SUM r^2: behind the last row)
#pragma unroll
    for (int k = 8; k < kSums; ++k) {
        if (t == k) {
            me.unknowns = unknown(kOrder.row[k]) | unknown(kOrder.column[k]);
            me.place = kOrder.row[k] * kRowDoubles + kOrder.column[k];
            me.diagonal = kOrder.row[k] == kOrder.column[k];
            if (me.diagonal) me.row = lanes_of_unknown(kOrder.row[k]);
        }
    }
    return me;
}

// Solves (A + lambda diag(A)) x = -g on the free variables (x = 0 for those in `held`); `sum`: what normal_equations returned.
// The lanes of unknown i return x_i.  A variable that no record feels (its row, column and gradient are zero: the sync
// parameters of a job that has never run on several GPUs of one node, or any pair on the flat spot T_sync = 0) gets a pivot of
// one; its x is zero whatever the pivot, and lambda 1e-300 would be out of inverse_root's range.  A zero on the diagonal alone
// does not say so: the squares of derivatives below 1e-162 are zero and their products with the others and with r are not (a pair
// started at 1e-18 of T_grad, gamma = 10).
// Returns false if a pivot is not positive.
__device__ __forceinline__ bool damped_step(double *system, const SumLane &me, double sum, double lambda, unsigned held, double &step)
{
    const double damped = sum + lambda * (sum > 1e-300 ? sum : 1e-300);
    double entry = me.gradient ? -sum : (me.diagonal ? damped : sum);
    const unsigned long long felt = __builtin_amdgcn_ballot_w64(sum != 0.0);
    if ((held & me.unknowns) != 0u || (me.diagonal && (felt & me.row) == 0ull)) entry = me.diagonal ? 1.0 : 0.0;
    wave_fence();
    system[me.place] = entry;
    wave_fence();
    double x[kTheta];
    if (!solve<false>(system, x)) {
        wave_fence();                    // (reads the system again, rather than have the other keep it)
        if (!solve<true>(system, x)) return false;
    }
    const int lane = lane_id();
#pragma unroll
    for (int i = 0; i < kTheta; ++i) step = (lane >> 1) == i ? x[i] : step;
    return true;
}

constexpr int kMaxStarts = 5;

// Dynamic LDS: kWaveDoubles doubles per wavefront.  HELD: no job has more than 64 records.
// Three wavefronts a SIMD (168 registers): held to 128 it spills, 0.52 ms where it takes 0.39, 0.88 where it takes 0.81.
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
    if (bit_reversed(lane) < n) mine = load_record(f, base + bit_reversed(lane));
    // (a job whose times are all infinite, NaN or negative has no such record: what is fitted to it is unspecified, what is read is its own)
    const double m_at = (double)f.m[base + (size_t)record_or_first(__builtin_amdgcn_readfirstlane(best_o), n)];

    // priors (Sec. 4.1, "Prior-driven exploration"): parameters without evidence are held at zero
    unsigned prior = 0u;
    if (max_k <= 1) prior |= unknown(PX_ALPHA_SL) | unknown(PX_BETA_SL) | unknown(PX_ALPHA_SN) | unknown(PX_BETA_SN);
    if (max_nodes <= 1) prior |= unknown(PX_ALPHA_SN) | unknown(PX_BETA_SN);
    if (max_k <= 2) prior |= unknown(PX_BETA_SL) | unknown(PX_BETA_SN);
    prior = (unsigned)__builtin_amdgcn_readfirstlane((int)prior);
    // lanes 2 i and 2 i + 1, i < 7: what the iteration keeps of unknown i (the lanes beyond hold nothing that is read)
    const int which = lane >> 1;
    const bool is_sync = which >= PX_ALPHA_SL && which <= PX_BETA_SN, is_gamma = which == PX_GAMMA;
    const bool my_prior = which < kTheta && ((prior >> lane) & 1u);
    // the default starting value of this lane's sync parameter
    const double sync_default = (which == PX_ALPHA_SL || which == PX_ALPHA_SN) ? t_min / 10.0 : t_min / 100.0;
    double start = is_gamma ? 2.0 : (is_sync ? sync_default : (which == PX_ALPHA_G ? t_min * 0.5 : t_min / (2.0 * m_at)));
    if (f.init && which < kTheta) start = f.init[(size_t)which * f.J + j];
    if (my_prior) start = 0.0;
    const double scale = (!is_gamma && start > 0.0) ? start : 1.0;
    const double lo = is_gamma ? 1.0 : 0.0, hi = is_gamma ? 10.0 : __builtin_inf();

    // The error has several local minima (and a flat spot at T_sync = 0 when gamma > 1), so the iteration is
    // run from a few starting points, one per wavefront, and the best end point is kept (the first one on
    // ties).  Start 0 is the start itself.  Starts 1 and 2 first minimise with gamma held at 1, where
    // Eq. 11 is linear in the alphas and betas, then release gamma from 2 and from 5 with the sync
    // parameters raised to at least a tenth of their starting values.  Starts 3 and 4 scale the sync
    // parameters by 3 and 0.3 and begin at gamma = 1.2 and 5.
    {
        const bool two_phase = k == 1 || k == 2;
        const double sync_factor = (k == 3) ? 3.0 : (k == 4 ? 0.3 : 1.0);
        const double gamma0 = (k == 0) ? wave_read(start, 2 * PX_GAMMA) : (k == 1 ? 2.0 : (k == 3 ? 1.2 : 5.0));
        double z;
        {
            double v = start;
            if (is_sync) v *= sync_factor;
            if (is_gamma) v = two_phase ? 1.0 : gamma0;
            v /= scale;
            z = v < lo ? lo : (v > hi ? hi : v);
        }

        double *system = fit_lds + k * kWaveDoubles;
        if (lane < kWaveDoubles) system[lane] = 0.0;           // (the entries that are always zero)
        const SumLane me = sum_lane();
        double scales[kTheta];
#pragma unroll
        for (int i = 0; i < kTheta; ++i) {
            scales[i] = wave_read(scale, 2 * i);
            asm volatile("" : "+v"(scales[i]));             // (the scalar registers are taken by the constants)
        }
        const Coefs math = held_coefs();
        double cur = 0.0;                    // the lane's sum at the iterate
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
                const bool stuck = !(prior & unknown(ia)) && (zero & unknown(ia)) && ((prior | zero) & unknown(ib));
                if (!(stuck && it < f.max_iter && cur_sse > 0.0)) continue;
                if (which == ia) z = sync_default / scale;
            }
            // The damped Gauss-Newton iteration from z, until it converges or the budget of steps is spent; the
            // variables in `hold` stay where they are.  Leaves the end point in z and its error in cur_sse.
            const unsigned hold = phase == 0 ? prior | unknown(PX_GAMMA) : prior;
            double lambda = 1e-3, zn = z;
            bool first = true;
            unsigned moved = 0u, moved_little = 0u;   // unknowns the last step has changed by 1e-9 of themselves or more, 1e-15 or more
            for (;;) {
                // Half of the trial points are refused.  Their error alone decides that, so derivatives and the other sums wait for
                // it; a point that is taken costs 35 instructions more for it.  (Guessing from the fate of the points before which
                // of the two to begin with was slower: 0.76 ms where this takes 0.71.  Beyond 64 records a second pass over them
                // would cost what it saves.)
                const Theta point = make_theta(zn, scale);
                Prediction at = {};
                double r = 0.0, trial = 0.0, trial_sse;
                if constexpr (HELD) {
                    at = predict(point, mine, math);
                    r = residual(at, mine, bit_reversed(lane) < n, math);
                    trial_sse = uniform_f64(sum_term(r * r));
                } else {
                    trial = normal_equations<HELD>(f, j, n, point, scales, mine, at, r, math);
                    trial_sse = wave_read(trial, 2 * 7);
                }
                if (first || trial_sse < cur_sse) {
                    const double before = cur_sse;
                    z = zn;
                    if constexpr (HELD) trial = normal_equations<HELD>(f, j, n, point, scales, mine, at, r, math);
                    cur = trial;
                    cur_sse = trial_sse;
                    if (!first) {
                        lambda = lambda * 0.2 > 1e-15 ? lambda * 0.2 : 1e-15;
                        if (moved == 0u && (before - trial_sse) / before < 1e-13) break;
                    }
                    first = false;
                } else {
                    lambda *= 5.0;
                    if (lambda > 1e15 || moved_little == 0u) break;
                }
                // the next trial point
                bool found = false;
                while (!found && it < f.max_iter && cur_sse > 0.0) {
                    ++it;
                    const double g = cur;                               // (of the lane's unknown)
                    unsigned held = hold | ((unsigned)__ballot((z <= lo && g > 0.0) || (z >= hi && g < 0.0)) & kAll);
                    // a free variable that sits on a bound and would be pushed across it joins the held set
                    double step = 0.0;
                    bool solved = false;
#pragma unroll 1
                    for (int pass = 0; pass < kTheta + 1; ++pass) {
                        solved = damped_step(system, me, cur, lambda, held, step);
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
                    const double change = fabs(zn - z), size = fabs(z) + 1e-12;
                    moved = (unsigned)__ballot(change >= 1e-9 * size) & kAll;
                    moved_little = (unsigned)__ballot(change >= 1e-15 * size) & kAll;
                    if (((unsigned)__ballot(change > 0.0) & kAll) == 0u) break;
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
        if (which < kTheta) end_z[k][which] = z;
    }
    __syncthreads();
    if (k != 0) return;

    // the arguments again, rather than keep them in scalar registers through the fit
    typedef const FitArgs __attribute__((address_space(4))) *KernelArgs;
    KernelArgs again = (KernelArgs)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(again));
    const FitArgs e = *(const FitArgs *)again;
    int best_k = 0, total_it = 0;
    for (int c = 0; c < e.n_starts; ++c) {
        total_it += end_it[c];
        if (end_sse[c] < end_sse[best_k]) best_k = c;
    }
    const double best_sse = end_sse[best_k];
    if (which < kTheta) e.theta[(size_t)which * e.J + j] = end_z[best_k][which] * scale;
    if (lane == 0) {
        e.rmsle[j] = sqrt(best_sse / (double)n);
        if (e.iterations) e.iterations[j] = total_it;
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
    // The instance without the loop over further records multiplies where the other accumulates (1000 jobs of up to 48 records in
    // 48 slots 829 us, in 65 slots 902 with the other).
    if (max_obs <= kWave) hipLaunchKernelGGL(fit_theta_kernel<true>, grid, block, lds, stream, f);
    else hipLaunchKernelGGL(fit_theta_kernel<false>, grid, block, lds, stream, f);
    return hipGetLastError() == hipSuccess ? PX_OK : PX_E_HIP;
}

}  // namespace px
