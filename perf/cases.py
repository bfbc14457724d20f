"""What a user of the library has it do: the estimate, drop decision and survivor queues of a batch of queue
snapshots (pard_estimate_drop + pard_compact, or both in one call), its sequentially consistent and ranked variants,
and the State Planner's periodic step (queue lengths + downstream latency with the sampled batch-wait quantile).

A case says the shape of the snapshots and of the pipeline; requests are drawn on the GPU from the seed alone.  All
values are whole microseconds, so every output has one valid answer and is compared bit for bit.
"""
import math

import numpy as np
import torch

from paper_2602_08747_amd import binding, workloads

SLO_US = (150_000, 250_000, 400_000)          # the SLOs of the sweep and of the mixed configuration
LAMBDA = (1, 10)                              # the batch-wait quantile the paper uses
INT32_MAX = 2**31 - 1


def _case(name, kind, snapshots, requests, stages, dag, arrive, order="lbf", ragged=False, bursty=False, relaxed=False, samples=0):
    """kind      which entry points: two_calls, one_call, consistent, ranked, planner
    snapshots, requests   how many snapshots, and the requests of each (the most of any, when ragged)
    dag       chain / layered: one pipeline shared by all snapshots; own: every snapshot its own layered pipeline
    arrive    in_order: one SLO per snapshot, requests by arrival, so by deadline; mixed: three SLOs in one queue, by
              arrival; shuffled: three SLOs, no order
    order     lbf / hbf: low or high budget first
    bursty    bursts of ten times the rate and skewed stages
    relaxed   fast stages and half of the deadlines still ahead, so that a part of every queue survives (else overload)"""
    return dict(name=name, kind=kind, snapshots=snapshots, requests=requests, stages=stages, dag=dag, arrive=arrive, order=order,
                ragged=ragged, bursty=bursty, relaxed=relaxed, samples=samples)


def listed():
    return [
        # the broker of one worker pool looks at its queue: a thousand requests, a three-module chain (latency of a call)
        _case("one-1k", "two_calls", 1, 1024, 3, "chain", "shuffled", relaxed=True),
        # many worker queues of a few dozen requests each, taken together
        _case("tiny-queues", "two_calls", 100_000, 64, 5, "chain", "mixed", ragged=True, relaxed=True),
        # ordinary queues of some hundred requests, every pipeline with its own DAG
        _case("small-queues", "two_calls", 16_000, 1000, 6, "own", "in_order", ragged=True, relaxed=True),
        # the benchmark's default sweep: 4096 pipelines x 8192 queued requests under overload
        _case("sweep", "two_calls", 4096, 8192, 6, "own", "in_order"),
        # the same kind of sweep with SLO classes mixed and arriving in no order, uneven sizes, through the one call
        _case("sweep-shuffled", "one_call", 3001, 8001, 6, "own", "shuffled", ragged=True, relaxed=True),
        # one queue snapshot of a million requests in arrival order, a five-module chain
        _case("one-1m", "two_calls", 1, 1 << 20, 5, "chain", "in_order"),
        # four million requests of three SLO classes on an eight-stage DAG
        _case("one-4m-mixed", "two_calls", 1, 4_194_301, 8, "layered", "mixed"),
        # sixteen million requests, bursty and skewed, high budget first (the load-shedding order), twelve stages
        _case("one-16m-bursty", "two_calls", 1, 1 << 24, 12, "layered", "in_order", order="hbf", bursty=True),
        # as many collected from several brokers, so in no order
        _case("one-16m-shuffled", "two_calls", 1, 1 << 24, 12, "layered", "shuffled", order="hbf", bursty=True, relaxed=True),
        # sequentially consistent dropping over the sweep
        _case("consistent", "consistent", 4096, 8192, 6, "own", "in_order"),
        # later queues joined where the budget puts a request, over the sweep
        _case("ranked", "ranked", 4096, 8192, 6, "own", "in_order"),
        # the State Planner's step over the sweep with the paper's 10,000 samples
        _case("planner", "planner", 4096, 8192, 6, "own", "in_order", samples=10_000),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["two_calls", "two_calls", "two_calls", "one_call", "consistent", "ranked", "planner"])
    shape = "many" if kind == "planner" else rng.choice(["many", "many", "many", "one", "some"])
    if shape == "many":                        # up to what one workgroup holds each
        requests = _log(rng, 16, 8192)
        snapshots = _log(rng, 64, max(64, min(131_072, (1 << 25) // requests)))
    elif shape == "one":
        requests = _log(rng, 1000, 1 << (20 if kind == "ranked" else 24))
        snapshots = 1
    else:                                      # several large ones
        requests = _log(rng, 8193, 200_000)
        snapshots = _log(rng, 2, (1 << (20 if kind == "ranked" else 23)) // requests)
    if kind == "planner":
        snapshots = min(snapshots, 4096)
    stages = rng.choice([3, 4, 5, 6, 6, 8, 12])
    dag = rng.choice(["own", "own", "layered", "chain"])
    if snapshots > 4096 and dag == "own":
        stages = min(stages, 6)                # the tables of a hundred thousand pipelines of their own
    if kind == "planner":
        stages = min(stages, 6)
    c = _case("", kind, snapshots, requests, stages, dag, rng.choice(["in_order", "mixed", "shuffled"]), order=rng.choice(["lbf", "lbf", "hbf"]),
              ragged=snapshots > 1 and rng.random() < 0.6, bursty=rng.random() < 0.3, relaxed=rng.random() < 0.6,
              samples=rng.randint(2000, 10_000) if kind == "planner" else 0)
    del c["name"]
    return c


# ---- inputs ----------------------------------------------------------------------------------------------------

def _pipeline(case, seed):
    """The plan's arrays, and which of a few DAGs every snapshot has (as the exact values need them too)."""
    rng = np.random.default_rng([20260208, seed])
    K, S, own = case["snapshots"], case["stages"], case["dag"] == "own"
    if case["dag"] == "chain":
        dags = [workloads.csr_from_edges(S, workloads.chain_edges(S))]
    else:
        dags = [workloads.random_layered_dag(rng, S, 1 if S < 4 else 2, 8 if S <= 6 else 24)[:2] for _ in range(64 if own else 1)]
    D = K if own else 1
    pick = rng.integers(0, len(dags), D)
    lat = workloads.monotone_tables(rng, D * S)
    if case["relaxed"]:
        lat = np.maximum(1, lat // 200).astype(np.int32)
    mode = workloads.MODE_HBF if case["order"] == "hbf" else workloads.MODE_LBF
    plan = dict(K=K, S=S, dag_shared=0 if own else 1, dag_row_ptr=np.concatenate([dags[i][0] for i in pick]),
                dag_col=np.concatenate([dags[i][1] for i in pick]), batch=rng.choice([4, 8, 16, 32], D * S).astype(np.int32),
                workers=rng.integers(1, 17, D * S).astype(np.int32), lat_us=np.ascontiguousarray(lat.reshape(-1)),
                order_mode=np.full(D * S, mode, np.int32))
    return plan, dags, pick


def _requests(case, seed, dev="cuda"):
    g = torch.Generator(device=dev)
    g.manual_seed(1_000_003 * (seed + 1))
    K, P, S = case["snapshots"], case["requests"], case["stages"]

    def rand(*shape):
        return torch.rand(*shape, generator=g, device=dev)

    sizes = torch.full((K,), P, dtype=torch.int64, device=dev)
    if case["ragged"]:                          # from a tenth of the largest up to it, in an order of the seed's
        sizes = torch.linspace(max(1, P // 10), P, K, device=dev).to(torch.int64)
        sizes[-1] = P
        sizes = sizes[torch.argsort(rand(K))]
    snap_ptr = torch.zeros(K + 1, dtype=torch.int64, device=dev)
    torch.cumsum(sizes, 0, out=snap_ptr[1:])
    n = int(snap_ptr[-1].item())
    owner = torch.repeat_interleave(torch.arange(K, device=dev), sizes, output_size=n)
    # arrivals: exponential gaps, 5 us on average in one big queue that is bursty, 20 us in others, 20-200 us in many
    mean = (20.0 + 180.0 * rand(K))[owner] if K > 1 else torch.full((n,), 5.0 if case["bursty"] else 20.0, device=dev)
    if case["bursty"]:
        mean = torch.where((rand(n // 500 + 1) < 0.3)[torch.arange(n, device=dev) // 500], mean * 0.1, mean)
    arrival = torch.cumsum(-torch.log1p(-rand(n).double()) * mean, 0)
    arrival = (arrival - arrival[snap_ptr[:-1]][owner]).to(torch.int64)
    last = arrival[snap_ptr[1:] - 1]
    slo = torch.tensor(SLO_US, device=dev)[torch.randint(0, 3, (K if case["arrive"] == "in_order" else n,), generator=g, device=dev)]
    deadline = arrival + (slo[owner] if case["arrive"] == "in_order" else slo)
    if case["bursty"]:                          # Zipf(1.5) over the stages
        w = torch.arange(1, S + 1, device=dev, dtype=torch.float64) ** -1.5
        stage = torch.searchsorted(torch.cumsum(w / w.sum(), 0), rand(n).double()).clamp(max=S - 1)
    else:
        stage = torch.randint(0, S, (n,), generator=g, device=dev)
    if case["arrive"] == "shuffled":
        perm = torch.argsort(owner * (1 << 32) + torch.randint(0, 1 << 32, (n,), generator=g, device=dev))
        arrival, deadline = arrival[perm], deadline[perm]
    now = last // (2 if case["relaxed"] else 1)
    as32 = lambda t: t.to(torch.int32).contiguous()  # noqa: E731
    return dict(n=n, arrival=as32(arrival), deadline=as32(deadline), stage=as32(stage), snap_ptr=as32(snap_ptr), now=as32(now))


def _draws(case, seed, dev="cuda"):
    """The arrivals the planner has collected and the random words its samples are drawn with."""
    g = torch.Generator(device=dev)
    g.manual_seed(7_000_003 * (seed + 1))
    M = case["samples"]
    arrivals = torch.cumsum(-torch.log1p(-torch.rand(M, generator=g, device=dev).double()) * 20.0, 0)
    picks = torch.randint(0, 1 << 32, (M * case["stages"],), generator=g, device=dev)
    return arrivals.to(torch.int32), picks


def prepare(case, seed):
    plan, _, _ = _pipeline(case, seed)
    s = _requests(case, seed)
    s["kind"] = case["kind"]
    s["plan"] = binding.pard_plan_create(**plan)
    s["max_snap"] = case["requests"]
    segs, dev = plan["K"] * plan["S"], s["stage"].device
    new = lambda count, dtype=torch.int32: torch.zeros(count, dtype=dtype, device=dev)  # noqa: E731
    if case["kind"] == "planner":
        samples, picks = _draws(case, seed)
        s.update(samples=samples, picks=torch.where(picks >= 1 << 31, picks - (1 << 32), picks).to(torch.int32), qlen=new(segs), sub=new(segs, torch.int64))
        return s
    s.update(est=new(s["n"]), drop=new(s["n"], torch.uint8), order=new(s["n"]), seg_ptr=new(segs + 1), surv_idx=new(s["n"]), surv_ptr=new(segs + 1))
    s["workspace"] = new(binding.pard_workspace_bytes(s["plan"], s["n"], s["max_snap"]) // 4 + 64)
    return s


def run(s):
    plan, n, most = s["plan"], s["n"], s["max_snap"]
    if s["kind"] == "planner":
        binding.pard_queue_lengths(plan, n, s["stage"], s["snap_ptr"], s["qlen"])
        binding.pard_sub_latency(plan, s["qlen"], binding.SUB_FULL, *LAMBDA, s["samples"].numel(), s["samples"], s["picks"], s["sub"])
        return s["qlen"], s["sub"]
    inputs = [s[k] for k in ("arrival", "deadline", "stage", "snap_ptr", "now")]
    outputs = [s[k] for k in ("est", "drop", "order", "seg_ptr")]
    if s["kind"] == "one_call":
        binding.pard_estimate_drop_compact(plan, n, most, *inputs, *outputs, s["surv_idx"], s["surv_ptr"], s["workspace"])
    else:
        if s["kind"] == "consistent":
            binding.pard_estimate_drop_consistent(plan, n, most, *inputs, None, *outputs, s["workspace"])
        elif s["kind"] == "ranked":
            binding.pard_estimate_drop_ranked(plan, n, most, *inputs, *outputs, s["workspace"])
        else:
            binding.pard_estimate_drop(plan, n, most, *inputs, *outputs, s["workspace"])
        binding.pard_compact(plan, n, most, s["order"], s["seg_ptr"], s["drop"], s["surv_idx"], s["surv_ptr"], s["workspace"])
    return outputs + [s["surv_idx"], s["surv_ptr"]]


def work(case):
    """Inputs once, outputs once: deadline and stage in (8 B), estimate, decision and queue order out (9 B), and the
    survivors (4 B for those that stay: taken as a third of the requests).  Operations: a compare per bit of the
    queue position for the order, and about twenty for the estimate."""
    n = case["snapshots"] * case["requests"] * (0.55 if case["ragged"] else 1.0)
    segs = case["snapshots"] * case["stages"]
    if case["kind"] == "planner":                # stages in, lengths and latencies out; a wait and an add per sample and stage
        return {"bytes": 4 * n + 12 * segs + 4 * case["samples"] * (case["stages"] + 1), "flops": 4.0 * segs * case["samples"]}
    return {"bytes": 17 * n + 4 * n / 3 + 8 * segs, "flops": n * (20 + math.log2(max(2, case["requests"])))}


def tolerance(case):
    return "exact"


# ---- the same in 64 bits, in plain torch ------------------------------------------------------------------------

def _longest(dags, pick, S, K, cost):
    """down[..., k] = the largest sum of `cost` over the stages after k on any path (stages are numbered along the paths).
    `cost` is [rows, S]; `pick` names the DAG of each row."""
    adj = torch.zeros(len(dags), S, S, dtype=torch.bool)
    for d, (ptr, col) in enumerate(dags):
        for a in range(S):
            adj[d, a, torch.as_tensor(col[ptr[a]:ptr[a + 1]], dtype=torch.int64)] = True
    adj = adj.to(cost.device)
    down = torch.zeros_like(cost)
    for k in range(S - 1, -1, -1):
        for j in range(k + 1, S):
            down[:, k] = torch.where(adj[pick, k, j], torch.maximum(down[:, k], cost[:, j] + down[:, j]), down[:, k])
    return down


def exact(case, seed):
    plan, dags, pick = _pipeline(case, seed)
    r = _requests(case, seed)
    K, S, n, dev = plan["K"], plan["S"], r["n"], r["stage"].device
    up = lambda a: torch.as_tensor(a, dtype=torch.int64, device=dev)  # noqa: E731
    B, W, lat = up(plan["batch"]), up(plan["workers"]), up(plan["lat_us"]).view(-1, workloads.LAT_ENTRIES)
    pick = up(pick).expand(K) if len(pick) == 1 else up(pick)
    shared = plan["dag_shared"] == 1

    def cost(queue, ahead):                      # wait and execution with `ahead` requests before one's own
        rec = queue % S if shared else queue
        return (ahead + B[rec] - 1) // B[rec] * lat[rec, B[rec] - 1] // W[rec] + lat[rec, torch.minimum(ahead + 1, B[rec]) - 1]

    stage, deadline, now = r["stage"].long(), r["deadline"].long(), r["now"].long()
    owner = torch.repeat_interleave(torch.arange(K, device=dev), torch.diff(r["snap_ptr"].long()), output_size=n)
    queue = owner * S + stage
    qlen = torch.bincount(queue, minlength=K * S)
    if case["kind"] == "planner":
        return qlen, _planner_exact(case, seed, dags, pick, qlen, cost(torch.arange(K * S, device=dev), qlen), B, lat, shared)
    seg_ptr = torch.cat([torch.zeros(1, dtype=torch.int64, device=dev), torch.cumsum(qlen, 0)])
    key = -deadline if case["order"] == "hbf" else deadline
    place = queue * (1 << 33) + key + (1 << 32)
    place_sorted, order = torch.sort(place, stable=True)
    every = torch.arange(K * S, device=dev)
    if case["kind"] == "ranked":                 # in a later queue, those its order serves first
        down = torch.empty(n, dtype=torch.int64, device=dev)
        for lo in range(0, n, 1 << 22):
            at = slice(lo, lo + (1 << 22))
            later = owner[at, None] * S + torch.arange(S, device=dev)
            ahead = torch.searchsorted(place_sorted, later * (1 << 33) + key[at, None] + (1 << 32), right=True) - seg_ptr[later]
            down[at] = _longest(dags, pick[owner[at]], S, K, cost(later, ahead)).gather(1, stage[at, None])[:, 0]
    else:
        down = _longest(dags, pick, S, K, cost(every, qlen).view(K, S)).view(-1)[queue]
    position = torch.empty(n, dtype=torch.int64, device=dev)
    position[order] = torch.arange(n, device=dev) - seg_ptr[queue[order]]
    if case["kind"] == "consistent":             # positions count the kept requests only, so a queue is walked in order
        if int(qlen.max().item()) > 50_000:
            return None
        kept = torch.zeros(K * S, dtype=torch.int64, device=dev)
        for i in range(int(qlen.max().item())):
            some = torch.nonzero(qlen > i)[:, 0]
            who = order[seg_ptr[some] + i]
            position[who] = kept[some]
            kept[some] += now[owner[who]] + cost(some, kept[some]) + down[who] <= deadline[who]
    total = cost(queue, position) + down
    drop = torch.clamp(now[owner] + total, max=INT32_MAX) > deadline
    stay = order[~drop[order]]
    surv_idx = torch.zeros(n, dtype=torch.int64, device=dev)
    surv_idx[:stay.numel()] = stay
    surv_ptr = torch.cat([seg_ptr[:1], torch.cumsum(torch.bincount(queue[~drop], minlength=K * S), 0)])
    return [torch.clamp(total, max=INT32_MAX), drop.to(torch.uint8), order, seg_ptr, surv_idx, surv_ptr]


def _planner_exact(case, seed, dags, pick, qlen, cost, B, lat, shared):
    """Per (snapshot, stage), the largest over the later paths of the summed costs plus the quantile of the summed waits."""
    S, M, dev = case["stages"], case["samples"], qlen.device
    samples, picks = _draws(case, seed, dev)
    drawn = samples.long()[picks % M].view(M, S)
    K = qlen.numel() // S
    rec = torch.arange(K * S, device=dev) % S if shared else torch.arange(K * S, device=dev)
    dur = lat[rec, torch.minimum(qlen + 1, B[rec]) - 1].view(K, S)
    cost = cost.view(K, S)
    rank = -(-LAMBDA[0] * M // LAMBDA[1])
    sub = torch.zeros(K, S, dtype=torch.int64, device=dev)
    for d, (ptr, col) in enumerate(dags):
        paths = {k: [] for k in range(S)}        # the stages after k, one list per path
        for k in range(S - 1, -1, -1):
            for j in col[ptr[k]:ptr[k + 1]]:
                paths[k] += [[int(j)] + p for p in (paths[int(j)] or [[]])]
        for rows in torch.nonzero(pick == d)[:, 0].split(256):
            wait = (dur[rows, None] - drawn % dur[rows, None]) % dur[rows, None]
            for k in range(S):
                for p in paths[k]:
                    w = torch.kthvalue(wait[:, :, p].sum(2), rank, dim=1).values
                    sub[rows, k] = torch.maximum(sub[rows, k], cost[rows][:, p].sum(1) + w)
    return sub.view(-1)
