"""Workloads of the planner's public calls: what a training loop asks of it at each step.

Four kinds of case, each one call of paper_2608_03676_amd:
  step    plan_step         ids -> loads, flow hint and schedule, outputs allocated by the call
  loads   plan_loads        the expert-load histogram and the marginals
  sink    sinkhorn_batched  the flow hint, cost shared by all problems (dense: one per problem)
  sched   round_schedule    replica matching and token split
The shapes are those of the benchmark's five configurations and of its hot-rank
family (fewer problems where the ids would not fit the card three times), with
odd sizes beside them.  The single calls write into outputs and a workspace
that the caller keeps from step to step, as a training loop does.

Routing is synthetic: experts follow a Zipf law over a seeded permutation, no
expert above a share of 1 / top_k (a token's choices are distinct), or a
seeded hot rank takes a fixed share of the choices.
"""
import dataclasses
import math

import numpy as np
import torch

import paper_2608_03676_amd as taot

NODE = 8  # ranks per node


def listed():
    return [
        # one layer over two nodes: the smallest step, all launches and latency
        dict(name="step_r16", kind="step", B=1, R=16, E=128, tokens=256, top_k=8, K=2, frac=0.5, tiers=2, cost=3.0,
             eps=3.0, iters=200),
        # the hot-rank regime at EP32: one step of a 48-layer model
        dict(name="step_r32", kind="step", B=48, R=32, E=128, tokens=8192, top_k=8, K=2, frac=0.7, tiers=2, cost=3.0,
             eps=3.0, iters=200),
        # 58 layers, 64 ranks, 16384 tokens a rank: counts past 16 bits are possible
        dict(name="loads_r64", kind="loads", B=58, R=64, E=256, tokens=16384, top_k=8, zipf=1.2),
        # 61 layers x 2 micro-batches, 256 ranks: the large histogram
        dict(name="loads_r256", kind="loads", B=122, R=256, E=384, tokens=8192, top_k=8, zipf=1.3),
        # ragged batch: a token count that no vector width divides, a few layers over few ranks
        dict(name="loads_odd", kind="loads", B=7, R=24, E=160, tokens=12289, top_k=6, zipf=1.1),
        dict(name="sink_r64", kind="sink", B=58, R=64, E=256, tokens=16384, top_k=8, zipf=1.2, tiers=2, cost=4.0,
             eps=0.08, iters=500),
        # 61 layers x 32 micro-batches: the benchmark's metric
        dict(name="sink_r256", kind="sink", B=1952, R=256, E=384, tokens=8192, top_k=8, zipf=1.3, tiers=3, cost=8.0,
             eps=0.08, iters=1000),
        dict(name="sink_r1024", kind="sink", B=64, R=1024, E=4096, tokens=8192, top_k=8, zipf=1.5, tiers=3, cost=16.0,
             eps=0.08, iters=2000),
        # a measured cost matrix per problem, all R x R entries
        dict(name="sink_dense_r1024", kind="sink", B=64, R=1024, E=4096, tokens=8192, top_k=8, zipf=1.5, tiers=3,
             cost=16.0, eps=0.08, iters=500, dense=True),
        dict(name="sched_r64", kind="sched", B=58, R=64, E=256, tokens=16384, top_k=8, K=2, zipf=1.2, tiers=2,
             cost=4.0, eps=0.08),
        dict(name="sched_r256", kind="sched", B=1952, R=256, E=384, tokens=8192, top_k=8, K=2, zipf=1.3, tiers=3,
             cost=8.0, eps=0.08),
        dict(name="sched_r1024", kind="sched", B=64, R=1024, E=4096, tokens=8192, top_k=8, K=2, zipf=1.5, tiers=3,
             cost=16.0, eps=0.08),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(max(lo, hi))))))


def draw(rng):
    kind = rng.choice(["step", "loads", "loads", "loads", "sink", "sink", "dense", "sched", "sched", "sched"])
    c = dict(kind=kind, tokens=_log_int(rng, 256, 16384), top_k=rng.choice([1, 2, 4, 6, 8]))
    if kind == "step":
        c.update(R=_log_int(rng, 4, 64), K=rng.choice([1, 2, 4]), frac=rng.choice([0.3, 0.5, 0.7, 0.9]), tiers=2,
                 cost=3.0, eps=3.0, iters=200)
        c.update(E=c["R"] * rng.choice([2, 4, 8]), B=_log_int(rng, 1, 64))
        return c
    c["zipf"] = round(rng.uniform(0.8, 1.5), 2)
    if kind == "loads":
        c["R"] = _log_int(rng, 4, 1024)
        c["E"] = min(4096, max(8, int(c["R"] * rng.choice([1, 1.5, 2, 4])) + rng.choice([0, 0, 0, 1, 2])))
        c["B"] = _log_int(rng, 1, min(256, (1 << 30) // (c["R"] * c["tokens"] * c["top_k"])))
        return c
    c.update(R=_log_int(rng, 16, 1024), tiers=rng.choice([2, 3]), cost=rng.choice([4.0, 8.0, 16.0]))
    c["E"] = int(c["R"] * rng.choice([1, 1.5, 2, 4]))
    c["eps"] = round(c["cost"] * rng.choice([0.005, 0.01, 0.02, 0.05]), 3)
    c["B"] = _log_int(rng, 1, min(1024, (1 << 25) // c["R"] ** 2))
    if kind == "sched":
        c["K"] = rng.choice([1, 2, 2, 4]) if c["R"] <= 512 else rng.choice([1, 2])
    else:
        c.update(kind="sink", iters=_log_int(rng, 100, 400 if kind == "dense" else 2000), dense=kind == "dense")
    return c


# ---- inputs -----------------------------------------------------------------

def _home(c):
    e = np.arange(c["E"])
    return e // (c["E"] // c["R"]) if c["E"] % c["R"] == 0 else e % c["R"]


def _costs(c):
    """Topology cost: 0 on the diagonal, 1 inside a node, then one tier (or two: a rack of 4 or 8 nodes) up to `cost`."""
    r = np.arange(c["R"])
    far = np.full((c["R"], c["R"]), c["cost"], np.float32)
    if c["tiers"] == 3:
        rack = r // (NODE * (8 if c["R"] > 256 else 4))
        far[rack[:, None] == rack[None, :]] = 3.0 if c["cost"] < 16 else 4.0
    far[(r // NODE)[:, None] == (r // NODE)[None, :]] = 1.0
    np.fill_diagonal(far, 0.0)
    return far


def _gen(seed):
    return torch.Generator(device="cuda").manual_seed(seed)


def _shares(c, g):
    """[B][E] fp64 routing shares."""
    B, E, R = c["B"], c["E"], c["R"]
    if "frac" in c:
        hot = torch.randint(R, (B, 1), generator=g, device="cuda")
        mine = (torch.from_numpy(_home(c)).cuda()[None, :] == hot).double()
        return (1 - c["frac"]) / E + c["frac"] * mine / mine.sum(1, keepdim=True)
    order = torch.rand((B, E), generator=g, device="cuda", dtype=torch.float64).argsort(1)
    p = torch.arange(1, E + 1, device="cuda", dtype=torch.float64) ** -c["zipf"]
    p = (p / p.sum()).expand(B, E).gather(1, order)
    most = max(1.0 / c["top_k"], 2.0 / E)
    for _ in range(12):  # shares above the most an expert can have go to the others
        over = (p - most).clamp(min=0)
        room = torch.where(over > 0, torch.zeros_like(p), p)
        p = torch.minimum(p, torch.full_like(p, most)) + room * over.sum(1, keepdim=True) / room.sum(1, keepdim=True)
    return p / p.sum(1, keepdim=True)


def _ids(c, g):
    """[B][R][N] int32 routing ids."""
    B, R, E, N = c["B"], c["R"], c["E"], c["tokens"] * c["top_k"]
    cdf = _shares(c, g).cumsum(1).float()
    ids = torch.empty((B, R, N), dtype=torch.int32, device="cuda")
    for b in range(B):
        x = torch.rand((R, N), generator=g, device="cuda")
        ids[b] = torch.searchsorted(cdf[b].contiguous(), x, right=True, out_int32=True).clamp_(max=E - 1)
    return ids


def _counts(c, g):
    """[B][R][E] int32 token counts of rows of N ids each, as routing of these shares gives them."""
    N = c["tokens"] * c["top_k"]
    p = _shares(c, g)
    n = torch.randn((c["B"], c["R"], c["E"]), generator=g, device="cuda")
    n = n.mul_((N * p * (1 - p)).sqrt().float()[:, None, :]).add_((N * p).float()[:, None, :]).round_()
    n = n.clamp_(min=0).int()
    top = p.argmax(1)  # the largest expert takes what rounding left over
    rest = N - n.sum(2, dtype=torch.int64)
    at = top[:, None, None].expand(c["B"], c["R"], 1)
    n.scatter_(2, at, (n.gather(2, at) + rest[:, :, None]).clamp(min=0).int())
    return n


def _loads(c, x):
    """load_r, excess, spare, mean (int64) of expert loads x [B][E]."""
    home = torch.from_numpy(_home(c)).cuda()
    load = torch.zeros((c["B"], c["R"]), dtype=torch.int64, device="cuda").index_add_(1, home, x)
    mean = load.sum(1, keepdim=True) // c["R"]
    return load, (load - mean).clamp(min=0), (mean - load).clamp(min=0), mean


def _spill(c, x, mean):
    """[B][E] spill of each expert: its share of the excess, experts of a rank in ascending (load, id) order."""
    home = torch.from_numpy(_home(c)).cuda()
    e = torch.arange(c["E"], device="cuda")
    key, order = ((home << 48) + (x << 13) + e).sort(1)
    xs = x.gather(1, order)
    run = xs.cumsum(1)
    first = torch.searchsorted(key, (home[order] << 48).contiguous())  # start of the rank's experts
    P = run - torch.where(first > 0, run.gather(1, (first - 1).clamp(min=0)), torch.zeros_like(run))
    s = (P - mean).clamp(min=0) - (P - xs - mean).clamp(min=0)
    return torch.zeros_like(x).scatter_(1, order, s)


def _plan(a, b, C, eps, iters):
    """The entropic plan of the supports of a and b after `iters` iterations in 64 bits:
    T, f, g as the flow hint defines them, without the column cap (which is 1 to rounding)."""
    a, b, C = a.double(), b.double(), C.double()
    gamma = (b.sum(1) / a.sum(1).clamp(min=1e-12)).clamp(max=1.0)
    s = a * gamma[:, None]
    M = (-C / eps).exp()
    if C.dim() == 2:
        Mt = M.t().contiguous()
        left, right = (lambda v: v @ Mt), (lambda u: u @ M)
    else:
        left = lambda v: torch.bmm(M, v[:, :, None])[:, :, 0]  # noqa: E731
        right = lambda u: torch.bmm(u[:, None, :], M)[:, 0, :]  # noqa: E731
    v = torch.ones_like(b)
    for _ in range(iters):
        u = s / left(v)
        v = b / right(u)
    return (u[:, :, None] * M) * v[:, None, :], eps * u.log(), eps * v.log()


def _cost_of(c, g):
    C = torch.from_numpy(_costs(c)).cuda()
    if c.get("dense"):  # links that are up to a few per cent slower from problem to problem
        C = C * (1 + 0.01 * torch.randint(7, (c["B"], 1, 1), generator=g, device="cuda"))
    return C


def _marginals(c, g):
    """supply, demand [B][R] fp32."""
    N = c["tokens"] * c["top_k"] * c["R"]
    p = _shares(c, g)
    x = (N * p + (N * p * (1 - p)).sqrt() * torch.randn(p.shape, generator=g, device="cuda", dtype=torch.float64))
    x = x.round().clamp(min=0).long()
    top = p.argmax(1, keepdim=True)
    x.scatter_(1, top, (x.gather(1, top) + (N - x.sum(1, keepdim=True))).clamp(min=0))
    _, excess, spare, _ = _loads(c, x)
    return excess.float(), spare.float()


@dataclasses.dataclass
class State:
    case: dict
    args: tuple
    kept: dict  # outputs and workspace that the caller keeps


def prepare(case, seed):
    c, g = case, _gen(seed)
    B, R, E = c["B"], c["R"], c["E"]
    home = torch.from_numpy(_home(c).astype(np.int32)).cuda()

    def ws(nbytes):
        return torch.empty(max(int(nbytes), 1), dtype=torch.uint8, device="cuda")

    def new(*shape, dtype):
        return torch.empty(shape, dtype=dtype, device="cuda")

    i32, i64, f32, f64 = torch.int32, torch.int64, torch.float32, torch.float64
    if c["kind"] in ("step", "sched"):
        C = _costs(c)
        Bp, Ba = (torch.from_numpy(x).cuda() for x in taot.topology_pref(C))
    if c["kind"] == "step":
        return State(c, (_ids(c, g), home, torch.from_numpy(C).cuda(), E, c["eps"], c["iters"], c["K"], Bp, Ba), {})
    if c["kind"] == "loads":
        out = taot.Loads(new(B, R, E, dtype=i32), new(B, E, dtype=i64), new(B, R, dtype=i64), new(B, R, dtype=i64),
                         new(B, R, dtype=i64), new(B, E, dtype=i64), new(B, R, dtype=f32), new(B, R, dtype=f32),
                         new(B, dtype=f64), new(B, dtype=f64), new(B, dtype=i64), new(B, dtype=i32),
                         new(B, R, dtype=i32), new(B, R, dtype=i32), new(B, dtype=i32), new(B, dtype=i32))
        size = taot.workspace_bytes(B, R, E, 1)["plan_loads"]
        return State(c, (_ids(c, g), home, E), dict(out=out, workspace=ws(size)))
    if c["kind"] == "sink":
        a, b = _marginals(c, g)
        out = taot.Flow(new(B, R, R, dtype=f32), new(B, R, dtype=f32), new(B, R, dtype=f32), new(B, dtype=i32))
        size = taot.workspace_bytes(B, R, E, 1)["sinkhorn"]
        return State(c, (a, b, _cost_of(c, g), c["eps"], c["iters"], taot.SK_DENSE if c.get("dense") else 0),
                     dict(out=out, workspace=ws(size)))
    K = c["K"]
    n = _counts(c, g)
    x = n.sum(1, dtype=i64)
    load, excess, spare, mean = _loads(c, x)
    T = torch.empty((B, R, R), dtype=f32, device="cuda")
    for lo in range(0, B, 128):  # the hint of a short run of the same iteration
        T[lo:lo + 128] = _plan(excess[lo:lo + 128], spare[lo:lo + 128], torch.from_numpy(C).cuda(), c["eps"], 50)[0]
    out = taot.Schedule(new(B, R * K, dtype=i32), new(B, R * K, dtype=i64), new(B, R, R * K, dtype=i32),
                        new(B, dtype=i64), new(B, 2, dtype=i32), new(B, dtype=i32))
    size = taot.workspace_bytes(B, R, E, K)["round_schedule"]
    return State(c, (n, _spill(c, x, mean), spare, excess, x.sum(1).double() / E, home, T, Bp, Ba, K),
                 dict(out=out, workspace=ws(size)))


# ---- one pass ---------------------------------------------------------------

def run(state):
    kind = state.case["kind"]
    if kind == "step":
        p = taot.plan_step(*state.args)
        return [_fields(p.loads), _fields(p.flow), _fields(p.schedule)]
    call = dict(loads=taot.plan_loads, sink=taot.sinkhorn_batched, sched=taot.round_schedule)[kind]
    return _fields(call(*state.args, **state.kept))


def _fields(x):
    return [getattr(x, f.name) for f in dataclasses.fields(x)]


def work(case):
    """Inputs read once, outputs written once; for the iterations a multiply-add per rank and half-step
    (every entry of the cost matrix in the dense mode, which sweeps all of them)."""
    c = case
    B, R, E, N = c["B"], c["R"], c["E"], c["tokens"] * c["top_k"]
    loads = 4 * B * R * N + 4 * B * R * E + B * (16 * E + 40 * R)
    sink = 4 * B * R * R + 16 * B * R + 4 * R * R * (B if c.get("dense") else 1)
    flops = 4 * c.get("iters", 0) * B * R * (R if c.get("dense") else 1)
    sched = 4 * B * R * R * c.get("K", 0) + 4 * B * R * R + 4 * B * R * E + 24 * B * R + 16 * R * R
    if c["kind"] == "step":
        return {"bytes": loads + sink + sched, "flops": flops}
    return {"bytes": dict(loads=loads, sink=sink, sched=sched)[c["kind"]], "flops": flops}


def tolerance(case):
    if case["kind"] == "sink":
        # four times what 32-bit scalings are off the 64-bit iterate over these ranges (T: 2.5e-6 and 2e-5)
        return {"rel": 1e-5, "max": 8e-5}
    if case["kind"] == "step":
        # as above (one supply row: g is off by 3e-6 from the shift that nothing damps); the hint's
        # rounding decides between ranks that score alike, which is rare here
        return {"rel": 1.2e-5, "max": 8e-5, "differ": 0.002}
    return "exact"


def _exact_loads(c, ids):
    B, R, E, N = c["B"], c["R"], c["E"], c["tokens"] * c["top_k"]
    n = torch.empty((B, R, E), dtype=torch.int64, device="cuda")
    row = E * torch.arange(R, device="cuda")[:, None]
    for b in range(B):
        n[b] = torch.bincount((ids[b].long() + row).reshape(-1), minlength=R * E).reshape(R, E)
    x = n.sum(1)
    load, excess, spare, mean = _loads(c, x)
    total = load.sum(1)
    rho = (R * load.max(1).values - total).double() / total.double()
    r = torch.arange(R, device="cuda").expand(B, R)

    def ranks(member):
        at = torch.where(member, r, torch.full_like(r, R)).sort(1).values
        return torch.where(at < R, at, torch.full_like(at, -1)).int(), member.sum(1).int()

    hot, hot_n = ranks(excess > 0)
    cold, cold_n = ranks(spare > 0)
    return [n.int(), x, load, excess, spare, _spill(c, x, mean), excess.double(), spare.double(), rho,
            total.double() / E, torch.zeros(B, dtype=torch.int64, device="cuda"),
            torch.zeros(B, dtype=torch.int32, device="cuda"), hot, cold, hot_n, cold_n]


def exact(case, seed):
    c = case
    if c["kind"] == "sched":
        return None  # whole numbers of a matching and an auction: compared as they are
    s = prepare(c, seed)
    if c["kind"] == "loads":
        return _exact_loads(c, s.args[0])
    if c["kind"] == "step":
        ids, _, C, _, eps, iters = s.args[:6]
        loads = _exact_loads(c, ids)
        return [loads, [*_plan(loads[6], loads[7], C, eps, iters), None], None]
    a, b, C, eps, iters = s.args[:5]
    s.kept.clear()
    if not c.get("dense"):
        return [*_plan(a, b, C, eps, iters), None]
    parts = [_plan(a[k:k + 16], b[k:k + 16], C[k:k + 16], eps, iters) for k in range(0, c["B"], 16)]
    return [*(torch.cat(x) for x in zip(*parts)), None]
