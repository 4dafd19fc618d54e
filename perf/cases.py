"""The calls this library is timed by: what a scheduler built on it asks of it, from the smallest cluster to the largest.

A case is a dict of plain values.  `prepare` draws its inputs on the GPU from a seed alone, `run` is one pass through the
package's public entry points, `work` says what the pass cannot do without, `tolerance` how far another correct
implementation's outputs may be off, and `exact` gives the outputs in plain 64-bit torch arithmetic.

Job parameters, batch-size grids and allocation matrices follow the distributions of the repository's own workloads
(8 jobs on 4x4 GPUs, 30 on 16x4, 200 on 64x8, 1000 on 256x8); sizes between them are generic.
"""
import math

import numpy as np
import torch

import paper_2008_12260_amd as px

TABLED_K = 64          # a memoised call sweeps every job once per GPU count up to this and placement class


def listed():
    """The listed cases; each stands for the use its comment names."""
    return [
        # an operator trying the scheduler on one rack: 4 nodes, 8 jobs; the call is all launches and latency
        dict(name="tiny_call", kind="fitness", P=16, J=8, N=4, cap=4, Gm=32, Gs=8, p=-1.0, outputs="all"),
        # one scheduling interval on the paper's testbed (16 nodes x 4 GPUs, 30 jobs): 20 generations of the search from
        # the allocation in force, the best matrix applied, the jobs advanced
        dict(name="testbed_interval", kind="interval", P=256, J=30, N=16, cap=4, Gm=64, Gs=16, p=-1.0, generations=20),
        # one evaluation of a population on a mid-size simulated cluster, the dense (m, s) grid for every pair
        dict(name="sim_call", kind="fitness", P=1000, J=200, N=64, cap=8, Gm=64, Gs=16, p=-1.0, outputs="argmax"),
        # the same cluster in single precision, another fairness knob, every output
        dict(name="sim_call_fp32", kind="fitness", P=1000, J=200, N=64, cap=8, Gm=64, Gs=16, p=0.5, outputs="all", precision=1),
        # one scheduling interval on that cluster
        dict(name="sim_interval", kind="interval", P=1000, J=200, N=64, cap=8, Gm=64, Gs=16, p=-1.0, generations=20),
        # that cluster with the paper's sampling of total batch sizes in place of the dense grid
        dict(name="sim_sampled", kind="fitness", P=1000, J=200, N=64, cap=8, Gm=64, Gs=16, p=1.0, outputs="argmax", sampled=True),
        # a cluster whose sizes are nobody's round numbers (rows that are no whole 16-byte groups), the geometric mean
        dict(name="odd_call", kind="fitness", P=1021, J=331, N=130, cap=4, Gm=50, Gs=21, p=0.0, outputs="all"),
        # the benchmark configuration: 4096 candidates of 1000 jobs on 256 nodes x 8 GPUs
        dict(name="cluster_call", kind="fitness", P=4096, J=1000, N=256, cap=8, Gm=128, Gs=32, p=-1.0, outputs="argmax"),
        # a search's evaluation on a large cluster of 250 nodes, sweeps memoised: bound by reading the matrices
        dict(name="cluster_memo", kind="fitness", P=2048, J=900, N=250, cap=8, Gm=128, Gs=32, p=-1.0, outputs="argmax", memo=True),
        # one step of the search on 256 nodes into a second buffer: crossover, mutation, both repairs
        dict(name="cluster_step", kind="step", P=2048, J=1000, N=256, cap=8),
        # the agents' part before a search: the throughput parameters of 1000 jobs fitted to their recorded iterations
        dict(name="fit_jobs", kind="theta", J=1000, max_obs=48, cap=8, n_starts=3),
        # the auto-scaling decision for 200 jobs that may hold up to 16 nodes of 8 GPUs
        dict(name="autoscale", kind="autoscale", J=200, max_nodes=16, cap=8, Gm=64, Gs=16),
    ]


def draw(rng):
    """One more case of the ranges the listed ones stand for."""
    def log_int(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    kind = rng.choice(["fitness", "fitness", "memo", "sampled", "fp32", "interval", "interval", "step", "theta", "autoscale"])
    cap = rng.choice([4, 8])
    if kind == "theta":
        return dict(kind="theta", J=log_int(8, 1000), max_obs=rng.randint(12, 64), cap=cap, n_starts=rng.choice([1, 3, 3]))
    if kind == "autoscale":
        return dict(kind="autoscale", J=log_int(8, 1000), max_nodes=rng.randint(2, 24), cap=cap, Gm=rng.choice([32, 50, 64, 128]),
                    Gs=rng.choice([8, 12, 16, 32]))
    if kind == "interval":
        N = log_int(4, 96)
        return dict(kind="interval", P=log_int(32, 1000), J=min(log_int(8, 250), N * cap), N=N, cap=cap, Gm=rng.choice([32, 50, 64]),
                    Gs=rng.choice([8, 12, 16]), p=rng.choice([-1.0, -1.0, 0.5]), generations=20)
    N = log_int(4, 256)
    P, J = log_int(16, 4096), min(log_int(8, 1000), N * cap)
    if kind == "step":
        return dict(kind="step", P=min(P, 2048), J=J, N=N, cap=cap)
    Gm, Gs = rng.choice([32, 50, 64, 100, 128]), rng.choice([8, 12, 16, 21, 32])
    case = dict(kind="fitness", P=P, J=J, N=N, cap=cap, Gm=Gm, Gs=Gs, p=rng.choice([-1.0, -1.0, 0.0, 0.5, 1.0]),
                outputs=rng.choice(["all", "argmax"]))
    if kind == "memo":
        case["memo"] = True
    elif kind == "sampled":
        case["sampled"] = True
        case["P"] = min(P, 1024)
    elif kind == "fp32":
        case["precision"] = 1
    return case


# ---- inputs --------------------------------------------------------------------------------------------------------

def _jobs(case, rng):
    """Job parameters [14, J] (rows of the library's job_params), the per-GPU memory bound and the grid [J, Gm]."""
    J, Gm = case["J"], case.get("Gm", 16)

    def uniform(lo, hi):
        return rng.uniform(lo, hi, J)

    def log_uniform(lo, hi):
        return np.exp(rng.uniform(math.log(lo), math.log(hi), J))

    M0 = rng.choice(np.array([32.0, 64.0, 128.0, 256.0]), J)
    m_max = rng.integers(64, 513, J).astype(np.float64)
    age = log_uniform(120.0, 8 * 3600.0)
    # a fifth of the jobs may not run a batch larger than one GPU holds
    M_max = np.where(rng.uniform(size=J) < 0.2, np.maximum(2.0 * M0, m_max), 32.0 * M0)
    params = np.stack([
        uniform(0.01, 0.2), log_uniform(1e-5, 1e-3), uniform(0.005, 0.05), uniform(0.001, 0.01), uniform(0.02, 0.2),
        uniform(0.005, 0.05), uniform(1.0, 5.0), log_uniform(1e2, 1e6), M0, M_max, np.ones(J), age,
        np.floor(rng.uniform(size=J) * age / 210.0), m_max])
    t = np.arange(Gm) / max(1, Gm - 1)
    lo, hi = (M0, M_max) if case.get("sampled") else (np.full(J, 8.0), m_max)
    grid = np.clip(np.floor(lo[:, None] * (hi / lo)[:, None] ** t + 0.5), lo[:, None], hi[:, None]).astype(np.int32)
    return params, grid


def _fair(J, N, cap):
    """(GPUs, nodes) of the packed fair share."""
    gpus = max(1, N * cap // J)
    return gpus, -(-gpus // cap)


def _matrices(count, J, N, cap, seed):
    """Allocation matrices [count, J, N]: the first is the packed fair share; the others visit the jobs in random order, draw
    GPU counts around the fair share and pack (70 %) or spread them, within the nodes' capacities and with at most one
    multi-node job per node.  One in ten has pending jobs, one in twenty breaks a constraint on purpose."""
    g = torch.Generator("cuda").manual_seed(seed)
    dev, i32 = "cuda", torch.int32
    fair, _ = _fair(J, N, cap)
    order = torch.rand((count, J), generator=g, device=dev).argsort(1)
    want = (fair * torch.exp(0.7 * torch.randn((J, count), generator=g, device=dev))).round().clamp(1, 4 * cap).to(i32)
    packed = torch.rand((J, count), generator=g, device=dev) < 0.7
    start = torch.randint(0, N, (J, count), generator=g, device=dev)
    which = torch.arange(count, device=dev)
    pending = (which % 10 == 3) & (torch.rand((J, count), generator=g, device=dev) < 0.02)
    # candidate 0: the jobs in order, the fair share each, packed from the first node
    order[0] = torch.arange(J, device=dev)
    want[:, 0], packed[:, 0], start[:, 0] = fair, True, 0
    out = torch.empty((count, J, N), dtype=i32, device=dev)
    flat = out.view(-1)
    free = torch.full((count, N), cap, dtype=i32, device=dev)
    held = torch.zeros((count, N), dtype=torch.bool, device=dev)
    nodes = torch.arange(N, device=dev)
    left = torch.full((count,), N * cap, dtype=i32, device=dev)
    for t in range(J):
        k = torch.minimum(want[t], left - (J - 1 - t)).clamp_(min=0)
        k = torch.where(pending[t], 0, k)[:, None]
        at = (nodes + start[t][:, None]) % N
        f, h = free.gather(1, at), held.gather(1, at)
        whole = f >= k
        one = (whole.cumsum(1, dtype=i32) == 1) & whole & packed[t][:, None]
        room = torch.where(h, 0, f)
        room = torch.where(packed[t][:, None], room, room.clamp(max=1))
        before = room.cumsum(1, dtype=i32) - room
        spread = torch.minimum((k - before).clamp(min=0), room)
        take = torch.where(one.any(1, keepdim=True), one * k, spread)
        # nothing placed under the sharing rule: one GPU on the first node that has one
        none = (take.sum(1, keepdim=True) == 0) & (k > 0)
        has = f > 0
        take = torch.where(none, ((has.cumsum(1, dtype=i32) == 1) & has).to(i32), take).to(i32)
        several = (take > 0).sum(1, keepdim=True) >= 2
        held.scatter_(1, at, h | (several & (take > 0)))
        free.scatter_(1, at, f - take)
        left = left - take.sum(1, dtype=i32)
        flat[(which * J + order[:, t])[:, None] * N + at] = take
    broken = which[which % 20 == 7]
    if broken.numel():
        n = broken.numel()
        j, where = (torch.randint(0, hi, (n,), generator=g, device=dev) for hi in (J, N))
        out[broken, j, where] += cap
        j, where = torch.randint(0, J, (n,), generator=g, device=dev), torch.randint(0, N, (n,), generator=g, device=dev)
        out[broken, j, where] += 1
        out[broken, j, (where + 1) % N] += 1
    return out


def _cluster(case, seed, count):
    """What a fitness call is given: job arrays, fair shares, the current allocation, capacities and `count` matrices."""
    J, N, cap = case["J"], case["N"], case["cap"]
    params, grid = _jobs(case, np.random.default_rng(seed))
    matrices = _matrices(count + 1, J, N, cap, seed)
    current = matrices[count].clone()
    fair = np.tile(np.array(_fair(J, N, cap), dtype=np.int32), (J, 1))
    return dict(params=params, grid=grid, fair=fair, current=current, capacity=np.full(N, cap, dtype=np.int32),
                population=matrices[:count])


def _records(case, seed):
    """Recorded (K, nodes, m, s, T) tuples per job, from a measurement process of its own with 3 % noise."""
    rng = np.random.default_rng(seed)
    J, n, cap = case["J"], case["max_obs"], case["cap"]
    count = rng.integers(min(6, n), n + 1, J).astype(np.int32)
    level = rng.choice(4, (J, 1), p=[0.1, 0.1, 0.3, 0.5])          # one GPU, two, one node, several nodes explored so far
    k_max = np.array([1, 2, cap, 4 * cap])[level]
    K = 1 + np.floor(rng.uniform(size=(J, n)) * k_max).astype(np.int64)
    packed = -(-K // cap)
    nodes = np.where(rng.uniform(size=(J, n)) < 0.7, packed, np.maximum(packed, np.minimum(K, rng.integers(1, 5, (J, n)))))
    nodes = np.where((level == 0) | (level == 2), 1, np.where(level == 1, np.where(K == 2, rng.integers(1, 3, (J, n)), 1), nodes))
    m = np.floor(8.0 * (rng.integers(64, 513, (J, 1)) / 8.0) ** rng.uniform(size=(J, n)) + 0.5)
    s = rng.integers(0, 4, (J, n))
    compute = rng.uniform(0.01, 0.2, (J, 1)) + np.exp(rng.uniform(math.log(1e-5), math.log(1e-3), (J, 1))) * m
    latency = np.where(nodes == 1, rng.uniform(0.005, 0.05, (J, 1)), rng.uniform(0.02, 0.2, (J, 1)))
    comm = np.where(K == 1, 0.0, latency * (1.0 + 0.15 * np.log2(K)))
    T = (s * compute + np.maximum(compute, comm) + 0.3 * np.minimum(compute, comm)) * np.exp(0.03 * rng.standard_normal((J, n)))
    device = lambda a, kind: torch.as_tensor(np.ascontiguousarray(a, dtype=kind)).cuda()
    return [device(a, np.int32) for a in (count, K, nodes, m, s)] + [device(T, np.float64)]


def _call(case, c, flags):
    return px.FitnessCall(case["P"], case["J"], case["N"], case["Gm"], case["Gs"], c["params"], c["grid"], c["fair"], c["current"],
                          c["capacity"], p=case["p"], delta=30.0, flags=flags, precision=case.get("precision", 0), device="cuda:0")


def prepare(case, seed):
    """What a program holds before the call, on the GPU."""
    kind = case["kind"]
    if kind == "fitness":
        c = _cluster(case, seed, case["P"])
        flags = (px.PX_FLAG_MEMOISE if case.get("memo") else 0) | (px.PX_FLAG_SAMPLE_M if case.get("sampled") else 0)
        return dict(kind=kind, call=_call(case, c, flags), population=c["population"], outputs=case["outputs"])
    if kind == "interval":
        c = _cluster(case, seed, 1)
        J = case["J"]
        empty = lambda n, t=torch.int32: torch.empty(n, dtype=t, device="cuda")
        return dict(kind=kind, call=_call(case, c, px.PX_FLAG_MEMOISE | px.PX_FLAG_PAIR_RESULTS), alloc=c["current"], seed=seed,
                    generations=case["generations"], population=empty((case["P"], J, case["N"])), best=empty(1), K=empty(J),
                    nodes=empty(J), changed=empty(J), target=torch.full((J,), 1e7, dtype=torch.float64, device="cuda"),
                    goodput=empty(J, torch.float64), finished=empty(J))
    if kind == "step":
        matrices = _matrices(case["P"], case["J"], case["N"], case["cap"], seed)
        dims = px.Dims(case["P"], case["J"], case["N"], 1, 1, 0, 0)
        g = torch.Generator("cuda").manual_seed(seed + 1)
        return dict(kind=kind, dims=dims, parents=matrices, children=torch.empty_like(matrices),
                    fitness=torch.rand(case["P"], dtype=torch.float64, device="cuda", generator=g),
                    capacity=torch.full((case["N"],), case["cap"], dtype=torch.int32, device="cuda"),
                    ga=px.GaParams(seed, 7, max(1, case["P"] // 2), (1 << 32) // case["J"], 0, None),
                    workspace=torch.empty(px.workspace_size(dims), dtype=torch.uint8, device="cuda"))
    if kind == "theta":
        J = case["J"]
        return dict(kind=kind, records=_records(case, seed), n_starts=case["n_starts"],
                    theta=torch.empty((7, J), dtype=torch.float64, device="cuda"),
                    rmsle=torch.empty(J, dtype=torch.float64, device="cuda"))
    rng = np.random.default_rng(seed)
    params, grid = _jobs(case, rng)
    J, n = case["J"], case["max_nodes"]
    dims = px.Dims(1, J, 1, case["Gm"], case["Gs"], 0, 0)
    return dict(kind=kind, dims=dims, params=torch.as_tensor(params).cuda(), grid=torch.as_tensor(grid).cuda(), cap=case["cap"],
                max_nodes=n, now=torch.as_tensor(rng.integers(1, n + 1, J).astype(np.int32)).cuda(),
                workspace=torch.empty(px.workspace_size(dims), dtype=torch.uint8, device="cuda"),
                per_gpu=torch.empty((J, n + 1), dtype=torch.float64, device="cuda"),
                new=torch.empty(J, dtype=torch.int32, device="cuda"))


# ---- one pass ------------------------------------------------------------------------------------------------------

def run(state):
    """One pass, as a program makes it; returns its outputs."""
    kind = state["kind"]
    if kind == "fitness":
        call = state["call"]
        call.run(state["population"], outputs=state["outputs"])
        out = [call.fitness, call.violations, call.best_m, call.best_s]
        return out + [call.best_goodput, call.speedup] if state["outputs"] == "all" else out
    if kind == "interval":
        # the allocation in force is uploaded, the search starts from copies of it; see the package's closed loop
        s, call = state, state["call"]
        P, J = call.dims.P, call.dims.J
        call.current_alloc.copy_(s["alloc"])
        pop = s["population"]
        pop.copy_(call.current_alloc.unsqueeze(0).expand_as(pop))
        call.run(pop, outputs="fitness")
        for g in range(s["generations"]):
            call.generation(pop, s["seed"], g, max(1, P // 2), max(1, (1 << 32) // J), outputs="fitness", inherit_rows=True)
        px.pollux_apply_best(call.dims, pop, call.fitness, call.current_alloc, s["best"], s["K"], s["nodes"], s["changed"])
        progress = torch.zeros(J, dtype=torch.float64, device=pop.device)
        d = call.dims
        px.pollux_sim_tick(px.Dims(P, J, d.N, d.Gm, d.Gs, 0, 0), call.job_params, call.m_grid, s["K"], s["nodes"], s["changed"],
                           s["target"], 60.0, 30.0, call.workspace, progress, s["goodput"], s["finished"])
        return [pop, call.fitness, call.violations, call.current_alloc, s["best"], s["K"], s["nodes"], s["changed"], progress,
                s["goodput"], s["finished"]]
    if kind == "step":
        px.pollux_ga_step(state["dims"], state["parents"], state["fitness"], state["capacity"], state["ga"], state["workspace"],
                          state["children"])
        return [state["children"]]
    if kind == "theta":
        px.pollux_fit_theta(*state["records"], state["theta"], state["rmsle"], n_starts=state["n_starts"])
        return [state["theta"], state["rmsle"]]
    px.pollux_goodput_per_gpu(state["dims"], state["params"], state["grid"], state["cap"], state["max_nodes"], state["workspace"],
                              state["per_gpu"])
    px.pollux_autoscale(state["per_gpu"], state["now"], 2.0 / 3.0, 0.5, state["new"])
    return [state["per_gpu"], state["new"]]


# ---- what a pass needs, and how exact it is ------------------------------------------------------------------------

def work(case):
    """Bytes: every input read and every output written once.  Operations: seven per grid point the call is asked to evaluate
    (Eq. 4), for a memoised call per point of the sweeps it shares."""
    kind, J = case["kind"], case["J"]
    if kind == "step":
        return dict(bytes=8.0 * case["P"] * J * case["N"], flops=0.0)
    if kind == "theta":
        # per start about thirty evaluations of residual, gradient and normal equations over half the record slots
        return dict(bytes=24.0 * J * case["max_obs"] + 64.0 * J, flops=30.0 * 200.0 * case["n_starts"] * J * case["max_obs"] / 2)
    points = case["Gm"] * (1 if case.get("sampled") else case["Gs"])
    job_bytes = J * (14 * 8.0 + 4.0 * case["Gm"])
    if kind == "autoscale":
        queries = J * (case["max_nodes"] + 1)
        return dict(bytes=job_bytes + 8.0 * queries + 8.0 * J, flops=7.0 * queries * points)
    P, N = case["P"], case["N"]
    sweeps = J * (TABLED_K + case["cap"])
    if kind == "interval":
        children = P - max(1, P // 2)
        # the population is laid out once; every generation reads the children's parents and writes the children
        return dict(bytes=job_bytes + 4.0 * P * J * N + case["generations"] * 8.0 * children * J * N, flops=7.0 * sweeps * points)
    outputs = P * (12.0 + J * (24.0 if case["outputs"] == "all" else 8.0))
    return dict(bytes=job_bytes + 4.0 * (P + 1) * J * N + outputs, flops=7.0 * (sweeps if case.get("memo") else P * J) * points)


def tolerance(case):
    """Largest difference from another correct implementation at the same precision."""
    kind = case["kind"]
    if kind == "step":
        return "exact"                  # integers throughout, the draws are defined bit by bit
    if kind == "theta":
        # the end point of an iteration on an error with flat directions and several minima: with the records of a job in
        # reverse order the errors reached agree to 1e-5, but the parameters differ by up to 0.15 (0.02 as a rule)
        return dict(rel=0.03, max=0.99)
    if case.get("precision"):
        return dict(rel=4e-6, max=4e-5, differ=1e-3)
    # 64-bit: the elected point is priced with one expression, sums over jobs may run in another order; elections between
    # points that agree to the last places may go either way
    return dict(rel=4e-15, max=4e-14, differ=1e-6)


# ---- the same results in plain 64-bit arithmetic -------------------------------------------------------------------

def _goodput(params, grid, job, K, one_node, Gs, sampled):
    """Largest GOODPUT (Eq. 4, 13) of each (job, K, placement) and the batch size and accumulation count that attain it."""
    q = params[:, job]
    a_g, b_g, a_l, b_l, a_n, b_n, gamma, phi, M0, M_max = (q[i][:, None] for i in range(10))
    k = K.double()[:, None]
    if sampled:
        M, mem = grid[job].double(), q[13].floor()[:, None]
        s = torch.ceil(M / (k * mem)) - 1.0
        m = torch.ceil(M / (k * (s + 1.0)))
        fits = s <= Gs - 1
    else:
        m = grid[job].double().repeat_interleave(Gs, 1)
        s = torch.arange(Gs, device=m.device, dtype=torch.float64).repeat(grid.shape[1])[None, :]
        fits = torch.ones_like(m, dtype=torch.bool)
    t_grad = a_g + b_g * m
    t_sync = torch.where(one_node[:, None], a_l + b_l * (k - 2.0), a_n + b_n * (k - 2.0))
    last = torch.where(k > 1, (t_grad ** gamma + torch.where(k > 1, t_sync, 1.0) ** gamma) ** (1.0 / gamma), t_grad)
    M = k * m * (s + 1.0)
    good = M / (s * t_grad + last) * ((phi + M0) / (phi + M))
    good = torch.where(fits & (M >= M0) & (M <= M_max), good, 0.0)
    top = good.max(1, keepdim=True).values
    where = torch.arange(good.shape[1], device=good.device)
    first = torch.where(good == top, where, good.shape[1]).min(1, keepdim=True).values
    found = top[:, 0] > 0
    pick = lambda v: torch.where(found, v.expand_as(good).gather(1, first)[:, 0], -1.0).to(torch.int32)
    return top[:, 0], pick(m), pick(s)


def _goodput_rows(params, grid, job, K, one_node, Gs, sampled):
    """_goodput over many rows, a few million grid points at a time."""
    step = max(1, (1 << 23) // (grid.shape[1] * (1 if sampled else Gs)))
    parts = [_goodput(params, grid, job[i:i + step], K[i:i + step], one_node[i:i + step], Gs, sampled)
             for i in range(0, job.numel(), step)]
    return [torch.cat(v) for v in zip(*parts)]


def exact(case, seed):
    """The outputs of `run` in 64 bits; None where none exist (an iteration's end point, a search's path)."""
    kind = case["kind"]
    if kind in ("step", "theta", "interval"):
        return None
    if kind == "autoscale":
        rng = np.random.default_rng(seed)
        params, grid = (torch.as_tensor(a).cuda() for a in _jobs(case, rng))
        J, n = case["J"], case["max_nodes"]
        job = torch.arange(J, device="cuda").repeat_interleave(n + 1)
        nodes = torch.arange(n + 1, device="cuda").repeat(J)
        K = torch.where(nodes == 0, 1, nodes * case["cap"])
        best, _, _ = _goodput_rows(params, grid, job, K, nodes <= 1, case["Gs"], False)
        return [(best / K).view(J, n + 1), None]
    c = _cluster(case, seed, case["P"])
    params, grid = torch.as_tensor(c["params"]).cuda(), torch.as_tensor(c["grid"]).cuda()
    current, capacity = c["current"], torch.as_tensor(c["capacity"]).cuda()
    P, J, sampled = case["P"], case["J"], bool(case.get("sampled"))
    K, nodes, changed, violations = [], [], [], []
    for part in c["population"].split(max(1, (1 << 26) // (J * case["N"]))):
        on = part > 0
        K.append(part.sum(2))
        nodes.append(on.sum(2))
        changed.append((part != current).any(2))
        shared = (on & (nodes[-1] >= 2)[:, :, None]).sum(1) - 1
        violations.append(shared.clamp(min=0).sum(1) + (part.sum(1) - capacity).clamp(min=0).sum(1))
    K, nodes, changed, violations = (torch.cat(v) for v in (K, nodes, changed, violations))
    # one evaluation per distinct (job, GPU count, placement); job j's fair share beside them
    span = int(K.max()) + 1
    job = torch.arange(J, device="cuda")
    key, at = torch.unique((job[None, :] * 2 + (nodes == 1)) * span + K, return_inverse=True)
    gpus, fair_nodes = int(c["fair"][0, 0]), int(c["fair"][0, 1])
    fair = _goodput_rows(params, grid, job, torch.full_like(job, gpus), torch.full_like(job, int(fair_nodes == 1)) > 0, case["Gs"], sampled)[0]
    rows_K = key % span
    good, m, s = _goodput_rows(params, grid, key // (2 * span), rows_K.clamp(min=1), (key // span) % 2 == 1, case["Gs"], sampled)
    good, m, s = torch.where(rows_K > 0, good, 0.0), torch.where(rows_K > 0, m, -1), torch.where(rows_K > 0, s, -1)
    good, m, s = good[at], m[at], s[at]
    age, restarts = params[11], params[12]
    factor = torch.where(current.sum(1) > 0, (age - restarts * 30.0) / (age + 30.0), 1.0)
    speedup = torch.where(fair > 0, good / fair, 0.0) * torch.where(changed, factor, 1.0)
    p, w = case["p"], params[10]
    mean = (w * (speedup.log() if p == 0.0 else speedup ** p)).sum(1) / w.sum()
    fitness = mean.exp() if p == 0.0 else mean ** (1.0 / p)
    fitness = torch.where(violations > 0, -violations.double(), fitness)
    out = [fitness, violations.to(torch.int32), m, s]
    return out + [good, speedup] if case["outputs"] == "all" else out
