// One generation of the population search on gfx950 (Pollux, arXiv 2008.12260,
// Sec. 4.3: candidate allocation matrices are perturbed and combined, then
// modified to satisfy node capacity and interference avoidance, Sec. 4.2).
// The operators are the ones documented at pollux_ga_step in pollux.h; all
// arithmetic is integer.
//
// Kernels
//   rank_kernel                 order[] = candidates by (fitness desc, index asc)
//   generation_kernel           one workgroup per child: elite copy, or row-wise
//                               crossover + mutation, then both repairs, with the
//                               per-node bookkeeping in LDS (form_child, pollux_step.h)

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <mutex>

#include "../../include/pollux.h"
#include "pollux_device.h"
#include "pollux_host.h"
#include "pollux_step.h"

namespace px {

// ---- rank ----------------------------------------------------------------------
// rank(c) = number of candidates that come before c; ranks are distinct, so
// order[rank(c)] = c is a permutation.
__global__ void __launch_bounds__(256) rank_kernel(GaArgs a)
{
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int c = blockIdx.x * 4 + wave;           // one wavefront per candidate, lanes over the others
    if (a.dirty_count && blockIdx.x == 0) {
        for (int j = threadIdx.x; j < a.J; j += blockDim.x) a.dirty_count[j] = 0;
    }
    if (c >= a.P) return;
    const int lane = lane_id();
    double f = a.fitness[c];
    if (!(f == f)) f = -__builtin_inf();
    // every lane counts among the candidates o = lane, lane + 64, ...; eight loads are requested together
    // (past the end the last candidate is read again and not counted)
    constexpr int kBatch = 8;
    int mine = 0;
    for (int o0 = 0; o0 < a.P; o0 += kBatch * kWave) {
        double g[kBatch];
#pragma unroll
        for (int u = 0; u < kBatch; ++u) {
            const int o = o0 + u * kWave + lane;
            g[u] = a.fitness[o < a.P ? o : a.P - 1];
        }
#pragma unroll
        for (int u = 0; u < kBatch; ++u) {
            const int o = o0 + u * kWave + lane;
            const double gu = (g[u] == g[u]) ? g[u] : -__builtin_inf();
            const bool first = (gu > f) | ((gu == f) & (o < c));
            mine += (int)((o < a.P) & first);
        }
    }
    const int before = wave_sum(mine);
    if (lane == 0) a.order[before] = c;
}

template <int ROWS, bool INHERIT>
__global__ void __launch_bounds__(kGaThreads) __attribute__((amdgpu_num_sgpr(96))) generation_kernel(GaArgs a)
{
    extern __shared__ __align__(16) unsigned char ga_lds[];
    const GaShared sh = carve_shared(ga_lds, a.J, a.N, a.max_entries);
    form_child<ROWS, INHERIT, false>(a, sh, nullptr, [](int, int) {});
}

bool ga_shapes_fit(int J, int N) { return ga_shared_bytes(J, N) <= kGaMaxShared; }

int allow_dynamic_lds(const void *kernel, size_t lds, size_t (&allowed)[kGaDevices])
{
    if (lds <= 48 * 1024) return PX_OK;
    static std::mutex lock;
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kGaDevices) return PX_E_HIP;
    std::lock_guard<std::mutex> hold(lock);
    if (allowed[dev] < lds) {
        if (hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds) != hipSuccess) return PX_E_HIP;
        allowed[dev] = lds;
    }
    return PX_OK;
}

void launch_rank(const GaArgs &a, hipStream_t stream)
{
    hipLaunchKernelGGL(rank_kernel, dim3((unsigned)((a.P + 3) / 4)), dim3(256), 0, stream, a);
}

// ---- applying the outcome of a search --------------------------------------------------
// The matrix PolluxSched applies at the end of a scheduling interval is the candidate of highest fitness
// (Sec. 4.3), i.e. the first in the order of rank_kernel: fitness descending, index ascending, NaN last.
__global__ void __launch_bounds__(256) best_kernel(int P, const double *__restrict__ fitness, int32_t *__restrict__ best)
{
    __shared__ double red_f[256];
    __shared__ int red_c[256];
    const int t = threadIdx.x;
    double f = -__builtin_inf();
    int c = 0x7FFFFFFF;
    for (int o = t; o < P; o += 256) {
        double g = fitness[o];
        if (!(g == g)) g = -__builtin_inf();
        if (c == 0x7FFFFFFF || g > f) { f = g; c = o; }        // ascending o: an equal value keeps the lower index
    }
    red_f[t] = f;
    red_c[t] = c;
    __syncthreads();
    for (int half = 128; half > 0; half >>= 1) {
        if (t < half) {
            const double g = red_f[t + half];
            const int o = red_c[t + half];
            if (o != 0x7FFFFFFF && (red_c[t] == 0x7FFFFFFF || g > red_f[t] || (g == red_f[t] && o < red_c[t]))) {
                red_f[t] = g;
                red_c[t] = o;
            }
        }
        __syncthreads();
    }
    if (t == 0) *best = red_c[0];
}

// One wavefront per job: the job's row of the best candidate becomes its current row; K, nodes and the
// re-allocation flag (row differs from the previous current row, which held at least one GPU) are reported.
__global__ void __launch_bounds__(256) apply_kernel(int J, int N, const int32_t *__restrict__ population,
                                                    const int32_t *__restrict__ best, int32_t *__restrict__ current,
                                                    int32_t *__restrict__ K_out, int32_t *__restrict__ nodes_out,
                                                    int32_t *__restrict__ changed_out)
{
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int j = blockIdx.x * 4 + wave;
    if (j >= J) return;
    const int lane = lane_id();
    const int32_t *__restrict__ row = population + ((size_t)*best * J + j) * N;
    int32_t *__restrict__ cur = current + (size_t)j * N;
    long long k = 0, held = 0;
    int nodes = 0;
    bool differs = false;
    for (int n0 = 0; n0 < N; n0 += kWave) {
        const int n = n0 + lane;
        const int32_t v = n < N ? row[n] : 0, was = n < N ? cur[n] : 0;
        k += v;
        held += was;
        nodes += __popcll(__ballot(v > 0));
        differs |= __ballot(v != was) != 0;
        if (n < N) cur[n] = v;
    }
    k = wave_sum(k);
    held = wave_sum(held);
    if (lane == 0) {
        K_out[j] = (int32_t)k;
        nodes_out[j] = nodes;
        changed_out[j] = (differs && held > 0) ? 1 : 0;
    }
}

int launch_apply_best(const pollux_dims *d, const int32_t *population, const double *fitness, int32_t *current_alloc,
                      int32_t *best, int32_t *K, int32_t *nodes, int32_t *changed, hipStream_t stream)
{
    hipLaunchKernelGGL(best_kernel, dim3(1), dim3(256), 0, stream, d->P, fitness, best);
    hipLaunchKernelGGL(apply_kernel, dim3((unsigned)((d->J + 3) / 4)), dim3(256), 0, stream, d->J, d->N, population, best,
                       current_alloc, K, nodes, changed);
    return hipGetLastError() == hipSuccess ? PX_OK : PX_E_HIP;
}

int launch_ga_step(const pollux_dims *d, const int32_t *parents, const double *fitness, const int32_t *node_capacity,
                   const pollux_ga_params *ga, void *workspace, int32_t *children, bool inherit_rows, hipStream_t stream)
{
    const WorkspaceLayout L = workspace_layout(*d);
    GaArgs a = ga_args(d, parents, fitness, node_capacity, ga, workspace, children);
    if (inherit_rows && a.in_place) {
        a.src_row = (int32_t *)((char *)workspace + L.src_row);
        a.odd = (int32_t *)((char *)workspace + L.odd);
        a.dirty_count = (int32_t *)((char *)workspace + L.dirty_count);
    }

    launch_rank(a, stream);
    const size_t lds = ga_shared_bytes(d->J, d->N);
    const unsigned children_formed = a.in_place ? (unsigned)d->P - ga->elite_k : (unsigned)d->P;
    const bool four = d->N >= 4 && d->N <= kWave && !a.job_gpu_cap;
    // Rows of 65 to 256 nodes: four requested at a time up to 1 GiB of children, where a wavefront otherwise waits for one row after
    // the other (128 x 1000 x 256: 161 -> 137 us, 326 x 201 x 88: 49 -> 44, 1024 x 1000 x 256: 489 -> 473); beyond, the copy of whole
    // 16-byte groups runs at the memory's rate without it (2048 x 1000 x 256: 881 us against 889).  Other rows would go entry by entry
    // there, so they come this way at any size (2048 x 1000 x 250: 1247 -> 911 us, 2048 x 900 x 254: 1151 -> 850).
    const bool groups16 = (d->N & 3) == 0 && (((uintptr_t)a.parents | (uintptr_t)a.children) & 15) == 0;
    const bool ahead = !four && d->N >= 4 && d->N <= 4 * kWave && !a.job_gpu_cap &&
                       (!groups16 || 4ull * children_formed * (unsigned long long)d->J * d->N <= (1ull << 30));
    const bool inherit = a.src_row != nullptr;
    const bool whole = four && groups16;
    constexpr int kInstances = 8;
    const void *kernels[kInstances] = {(const void *)generation_kernel<kRowsAny, false>, (const void *)generation_kernel<kRowsAhead, false>,
                                       (const void *)generation_kernel<kRows64, false>, (const void *)generation_kernel<kRows64Whole, false>,
                                       (const void *)generation_kernel<kRowsAny, true>, (const void *)generation_kernel<kRowsAhead, true>,
                                       (const void *)generation_kernel<kRows64, true>, (const void *)generation_kernel<kRows64Whole, true>};
    const int instance = (whole ? kRows64Whole : (four ? kRows64 : (ahead ? kRowsAhead : kRowsAny))) + (inherit ? 4 : 0);
    static size_t allowed[kInstances][kGaDevices];
    const int rc = allow_dynamic_lds(kernels[instance], lds, allowed[instance]);
    if (rc != PX_OK) return rc;
    if (children_formed > 0) {
        void *args[] = {&a};
        if (hipLaunchKernel(kernels[instance], dim3(children_formed), dim3(kGaThreads), args, lds, stream) != hipSuccess) return PX_E_HIP;
    }
    return hipGetLastError() == hipSuccess ? PX_OK : PX_E_HIP;
}

}  // namespace px
