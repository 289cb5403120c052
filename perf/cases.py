"""Timed cases of the scoring path: what a placer or a distributor has the library do.

A case is a dict of plain values.  `prepare` draws its inputs on the GPU (the distributions of
`paper_2509_06362_amd.workloads`, from the seed alone) and loads the profile tables; `run` is one call
of the library through the binding, into output arrays that the caller owns, as a serving or placing
loop makes it.  Every array holds the C types' bit patterns (uint32 as int32 and so on).

Calls:
  assign     maaso_score_assign: the distributor over one placement (window 0: against the state as
             given; window n: the state advances every n requests)
  sweep      maaso_placement_sweep: satisfied requests of every candidate deployment
  score      maaso_placement_score: the placer's composite score of every candidate
  partition  maaso_resource_partition_requests: Alg. 2 over the growth chains of Alg. 1
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2509_06362_amd import binding, workloads

TICKS = 1 << 20                      # time unit of arrival_ticks and q_ticks: 2^-20 s
WEIGHTS = dict(alpha=4.0, beta=0.3, gamma_t=16384.0, gamma_l=2.0)
BATCHES = (4, 8, 16, 32, 64, 128, 256)

DEFAULTS = dict(
    call="sweep", n_cand=1, i_pad=32, n_req=1024, n_slo=3, b_cap=128,
    window=0, policy=0, tbt_mode=0, pen_kappa=0.0, latencies=False,
    layout="mixed",      # instances of a candidate: "four" | "mixed" | "budget" | "full"
    gpus=32,             # GPUs of a candidate with layout "budget"; of the cluster for `partition`
    lengths="loguniform",  # prompt and output lengths: "loguniform" | "lognormal" | "short"
    jitter=False,        # every profile entry scaled by its own factor in [0.9, 1.1]
    load="fresh",        # state of the instances: "empty" | "fresh" | "loaded" | "stressed"
    deadlines=1.0,       # scale of the classes' deadlines: tight ones are what tells candidates apart
    rate=2000.0,         # arrivals per second
    bursty=False,
)


def _case(name, **kw):
    c = dict(DEFAULTS)
    c.update(kw)
    if name is not None:
        c["name"] = name
    return c


def listed():
    return [
        # one routing decision batch on a four-instance deployment: the smallest call there is
        _case("distribute_tiny", call="assign", i_pad=4, n_req=1024, b_cap=64, layout="four"),
        # the distributor in the paper's wording (shortest queue among the capable instances, worst-case
        # throughput) over a backlog of odd size, with the latencies a dashboard wants
        _case("distribute_backlog", call="assign", i_pad=64, n_req=1_000_003, policy=1, tbt_mode=1,
              latencies=True, load="loaded"),
        # a long request log against four instances: bound by the request stream
        _case("distribute_stream", call="assign", i_pad=4, n_req=1 << 26, b_cap=64, layout="four"),
        # the online distributor: 64 instances, 1024 windows of 4096 requests
        _case("distribute_online", call="assign", i_pad=64, n_req=4_194_304, window=4096, load="empty"),
        # the online distributor with every request routed against the state all earlier ones left
        _case("distribute_by_request", call="assign", i_pad=64, n_req=16_384, window=1, load="empty"),
        # a placer comparing a handful of deployments on a short trace
        _case("sweep_small", n_cand=37, i_pad=13, n_req=1000, b_cap=64, load="stressed", deadlines=0.25),
        # candidate deployments of a 32-GPU cluster under load, ragged (4 to 32 instances)
        _case("sweep_budget", n_cand=4096, i_pad=32, n_req=65_536, layout="budget", gpus=32,
              load="stressed", deadlines=0.25),
        # many fresh candidates of a large cluster, measured (jittered) profiles, tight deadlines
        _case("sweep_large", n_cand=65_536, i_pad=32, n_req=16_384, layout="full", jitter=True,
              deadlines=0.0625),
        # skewed lengths, eight classes, 128 loaded instances, occupancy penalty
        _case("sweep_skewed", n_cand=8192, i_pad=128, n_req=131_072, n_slo=8, b_cap=256,
              lengths="lognormal", load="loaded", pen_kappa=0.5, layout="full"),
        # the same, capacity-aware: every candidate through windows of 4096 over bursty arrivals
        _case("sweep_capacity", n_cand=8192, i_pad=128, n_req=131_072, n_slo=8, b_cap=256,
              lengths="lognormal", load="loaded", pen_kappa=0.5, layout="full", window=4096,
              rate=5000.0, bursty=True),
        # the composite score with the paper's request-by-request simulation
        _case("score_by_request", call="score", n_cand=8192, i_pad=128, n_req=8192, n_slo=8, b_cap=256,
              lengths="lognormal", load="loaded", pen_kappa=0.5, layout="full", window=1,
              rate=5000.0, bursty=True),
        # Alg. 2 on 64 GPUs: 24 configurations' growth chains (720 deployments) against R_t, R_l and R
        _case("partition", call="partition", gpus=64, n_req=131_072, n_slo=2, window=256,
              lengths="short", rate=400.0),
    ]


def _log_int(rng, lo, hi):
    """Log-uniform whole number in [lo, hi]; odd in every other draw."""
    v = int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
    if rng.random() < 0.5:
        v |= 1
    return max(lo, min(hi, v))


def _seconds(c):
    """Rough time of a pass, for keeping drawn cases below the largest listed one."""
    triples = c["n_cand"] * c["i_pad"] * c["n_req"]
    if c["call"] == "partition":
        return 1e-4 + c["n_req"] / c["window"] * c["gpus"] * 1e-7 + c["gpus"] ** 2 * c["n_req"] * 1e-12
    if c["window"] == 0:
        return 1e-5 + triples / 2e13
    n_win = math.ceil(c["n_req"] / c["window"])
    if c["call"] == "assign":
        return n_win * (1e-6 if c["window"] <= 4 else 4e-6) + triples / 5e11
    return n_win * 1e-5 * max(1.0, c["n_cand"] / 1024.0) * c["i_pad"] / 128.0 + triples / 4e12


def draw(rng):
    what = rng.choice(["assign", "assign", "assign_windows", "sweep", "sweep", "sweep",
                       "sweep_windows", "score_windows", "partition"])
    while True:
        n_slo = rng.choice([1, 2, 3, 5, 8, 16])
        b_cap = rng.choice([64, 128, 256])
        common = dict(n_slo=n_slo, b_cap=b_cap, lengths=rng.choice(["loguniform", "lognormal", "short"]),
                      jitter=rng.random() < 0.5, load=rng.choice(["empty", "fresh", "loaded", "stressed"]),
                      pen_kappa=rng.choice([0.0, 0.5]), tbt_mode=rng.choice([0, 0, 1]),
                      rate=rng.choice([400.0, 2000.0, 5000.0]), bursty=rng.random() < 0.5,
                      layout=rng.choice(["mixed", "full"]))
        if what == "assign":
            c = _case(None, call="assign", i_pad=_log_int(rng, 1, 256), n_req=_log_int(rng, 100, 1 << 24),
                      policy=rng.choice([0, 0, 1]), latencies=rng.random() < 0.5, **common)
        elif what == "assign_windows":
            window = rng.choice([1, 2, _log_int(rng, 3, 64), _log_int(rng, 64, 32_768)])
            c = _case(None, call="assign", i_pad=_log_int(rng, 2, 256), window=window,
                      n_req=_log_int(rng, 1000, 1 << 22), policy=rng.choice([0, 0, 1]),
                      latencies=rng.random() < 0.3, **common)
        elif what == "sweep":
            # deadlines that the longest prompts miss on any instance, so that counts are no constants
            common.update(lengths=rng.choice(["loguniform", "lognormal"]),
                          deadlines=0.0625 if n_slo == 3 else 0.25)
            c = _case(None, n_cand=_log_int(rng, 2, 65_536), i_pad=_log_int(rng, 2, 256),
                      n_req=_log_int(rng, 300, 1 << 18), **common)
            if c["i_pad"] >= 32 and rng.random() < 0.4:
                c.update(layout="budget", gpus=rng.choice([8, 16, 32]), i_pad=32)
        elif what in ("sweep_windows", "score_windows"):
            window = rng.choice([1, _log_int(rng, 2, 64), _log_int(rng, 64, 1024), _log_int(rng, 1024, 16_384)])
            c = _case(None, call=what.split("_")[0], n_cand=_log_int(rng, 8, 16_384),
                      i_pad=_log_int(rng, 2, 256), n_req=_log_int(rng, 500, 1 << 17), window=window,
                      policy=rng.choice([0, 0, 0, 1]) if window > 32 else 0, **common)
        else:
            c = _case(None, call="partition", gpus=_log_int(rng, 8, 96), n_req=_log_int(rng, 4096, 131_072),
                      n_slo=2, window=_log_int(rng, 64, 1024), lengths="short",
                      rate=rng.choice([200.0, 400.0, 800.0]))
        # within what the context's workspace holds, and cheaper than the largest listed case
        if 4 * c["n_slo"] * c["n_req"] + 16 * c["n_cand"] * c["i_pad"] > 48 << 20 and c["call"] == "sweep":
            continue
        if _seconds(c) <= 0.02:
            return c


# ------------------------------------------------------------------------------------------------
# inputs
# ------------------------------------------------------------------------------------------------

def _tables(case, seed):
    jitter = workloads.rng_for(seed, 0) if case["jitter"] else None
    a, p, t = workloads.profile_tables(case["b_cap"], jitter_rng=jitter)
    k = case["n_slo"]
    if case["call"] == "partition":
        d_ttft, d_tbt = np.array([0.5, 10.0], np.float32), np.array([0.05, 0.2], np.float32)
    elif k == 3:
        d_ttft, d_tbt = workloads.slo_three_classes()
    else:  # geometric ladders 0.2 .. 60 s and 20 .. 300 ms
        x = np.arange(k, dtype=np.float64) / max(k - 1, 1)
        d_ttft, d_tbt = (0.2 * 300.0 ** x).astype(np.float32), (0.02 * 15.0 ** x).astype(np.float32)
    scale = np.float32(case["deadlines"])
    return a, p, t, d_ttft * scale, d_tbt * scale


def _lengths(case, gen, n):
    def log_uniform(lo, hi):
        u = torch.rand(n, generator=gen, device="cuda", dtype=torch.float32).double()
        v = torch.exp(math.log(lo) + u * math.log((hi + 1) / lo)).floor_()
        return v.clamp_(lo, hi).to(torch.int32)

    def log_normal():
        v = torch.randn(n, generator=gen, device="cuda").mul_(1.5).add_(6.0).exp_().round_()
        return v.clamp_(1, 32768).to(torch.int32)

    if case["lengths"] == "lognormal":
        return log_normal(), log_normal()
    if case["lengths"] == "short":
        return log_uniform(16, 2048), log_uniform(8, 512)
    return log_uniform(16, 8192), log_uniform(8, 8192)


def _arrivals(case, gen, n):
    gaps = torch.empty(n, device="cuda", dtype=torch.float64).exponential_(1.0, generator=gen)
    rate = case["rate"]
    if case["bursty"]:  # blocks of 256 requests with a gamma-distributed (shape 0.3) rate of their own
        nb = (n + 255) // 256
        u = torch.rand(nb, generator=gen, device="cuda", dtype=torch.float64).clamp_min_(1e-9)
        e = torch.rand(nb, generator=gen, device="cuda", dtype=torch.float64).clamp_min_(1e-9)
        m = (u ** (1 / 0.3)) * (1.0 - torch.log(e)) / 0.3  # heavy near zero, mean of order one
        gaps = gaps / m.clamp_min_(1e-3).repeat_interleave(256)[:n]
    ticks = torch.cumsum(gaps * (TICKS / rate), 0).floor_().clamp_(max=2.0 ** 32 - 1).to(torch.int64)
    return torch.where(ticks >= 1 << 31, ticks - (1 << 32), ticks).to(torch.int32)


def _placements(case, gen):
    C, I = case["n_cand"], case["i_pad"]
    rand = lambda *s: torch.rand(*s, generator=gen, device="cuda")
    n_inst = torch.full((C,), I, dtype=torch.int64, device="cuda")
    batches = torch.tensor([b for b in BATCHES if b <= case["b_cap"]], device="cuda")
    if case["layout"] == "four":
        tp = torch.arange(I, device="cuda").expand(C, I) % 4
        B = (8 << tp).to(torch.int64)
    else:
        tp = torch.randint(0, 4, (C, I), generator=gen, device="cuda")
        B = batches[torch.randint(0, len(batches), (C, I), generator=gen, device="cuda")]
        if case["layout"] == "budget":  # degrees drawn among those that still fit until the GPUs are used
            left = torch.full((C,), case["gpus"], dtype=torch.int64, device="cuda")
            n_inst.zero_()
            for j in range(I):
                fit = torch.log2(left.clamp(1, 8).double()).floor().long() + 1
                t = torch.minimum((rand(C) * fit).long(), fit - 1)
                live = left > 0
                tp[:, j] = torch.where(live, t, torch.zeros_like(t))
                n_inst += live
                left -= torch.where(live, 1 << t, torch.zeros_like(t))
        elif case["layout"] == "mixed" and C > 1:  # ragged candidates
            n_inst = torch.randint(1, I + 1, (C,), generator=gen, device="cuda")
    valid = torch.arange(I, device="cuda")[None, :] < n_inst[:, None]
    scale = {"empty": 0.0, "fresh": 1.0, "loaded": 1.25, "stressed": 2.0}[case["load"]]
    occ = (rand(C, I) * B * scale).floor_().to(torch.int64)
    if case["load"] == "loaded":
        q = torch.randint(0, 1 << 19, (C, I), generator=gen, device="cuda")
    elif case["load"] == "stressed":
        q = (2.0 ** (14.0 + 9.0 * rand(C, I))).to(torch.int64)
    else:
        q = torch.zeros(C, I, dtype=torch.int64, device="cuda")
    zero = torch.zeros_like(occ)
    return dict(n_cand=C, i_pad=I, n_inst=n_inst.to(torch.int32),
                tp_idx=torch.where(valid, tp, zero).to(torch.uint8).contiguous(),
                max_batch=torch.where(valid, B, zero + 1).to(torch.int16).contiguous(),
                occ=torch.where(valid, occ, zero).to(torch.int32).contiguous(),
                q_ticks=torch.where(valid, q, zero).contiguous())


def _chains(case):
    """Growth chains of Alg. 1: 1, 2, ... identical fresh instances of every (strategy, batch size)."""
    w = workloads.partition_case(n_req=1)
    tp, b = workloads.all_configs()
    cw, offs = workloads.growth_chains(w, tp, b, case["gpus"])
    up = lambda x, v: torch.from_numpy(np.array(x).view(v)).cuda()
    pl = dict(n_cand=cw.n_cand, i_pad=cw.i_pad, n_inst=up(cw.n_inst, np.int32), tp_idx=up(cw.tp_idx, np.uint8),
              max_batch=up(cw.max_batch, np.int16), occ=up(cw.occ, np.int32), q_ticks=up(cw.q_ticks, np.int64))
    return pl, up(offs, np.int32)


def _inputs(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed * 7919 + 17)
    n = case["n_req"]
    prompt, out = _lengths(case, gen, n)
    rq = dict(n_req=n, prompt_len=prompt, out_len=out,
              slo_class=torch.randint(0, case["n_slo"], (n,), generator=gen, device="cuda", dtype=torch.uint8))
    if case["window"]:
        rq["arrival_ticks"] = _arrivals(case, gen, n)
    pl, offsets = _chains(case) if case["call"] == "partition" else (_placements(case, gen), None)
    prm = dict(s_bar=float(out.double().mean().float()), pen_kappa=case["pen_kappa"],
               tbt_mode=case["tbt_mode"], window=case["window"], policy=case["policy"])
    return rq, pl, offsets, prm


def prepare(case, seed):
    a, p, t, d_ttft, d_tbt = _tables(case, seed)
    rq, pl, offsets, prm = _inputs(case, seed)
    ctx = binding.maaso_profile_tables_load(4, case["b_cap"], a, p, t, d_ttft, d_tbt,
                                            tp_degree=workloads.TP_DEGREES)
    n, C = case["n_req"], pl["n_cand"]
    empty = lambda m, dt: torch.empty(m, dtype=dt, device="cuda")
    i32, f32 = torch.int32, torch.float32
    if case["call"] == "assign":
        out = dict(chosen=empty(n, i32), slack=empty(n, f32), n_satisfied=empty(1, torch.int64))
        if case["latencies"]:
            out.update(ttft=empty(n, f32), tbt=empty(n, f32), e2e=empty(n, f32))
    elif case["call"] == "sweep":
        out = dict(sat_count=empty(C, i32), sat_ratio=empty(C, f32), best_cand=empty(1, i32))
    elif case["call"] == "score":
        out = dict(sat_count=empty(C, i32), best_cand=empty(1, i32), score=empty(C, f32),
                   phi_s=empty(C, f32), phi_t=empty(C, f32), phi_l=empty(C, f32))
    else:
        G = case["gpus"] + 1
        sizes = dict(prompt_len_split=n, out_len_split=n, slo_class_split=n, arrival_ticks_split=n,
                     n_tight=1, partition=6, phi_opt=1)
        out = {name: empty(sizes.get(name, G if name.endswith("_star") else C), getattr(torch, dt))
               for name, dt in binding.PARTITION_WORK_FIELDS}
    return dict(call=case["call"], window=case["window"], gpus=case["gpus"], ctx=ctx, rq=rq, pl=pl,
                offsets=offsets, prm=prm, out=out)


def run(state):
    ctx, rq, pl, prm, out = (state[k] for k in ("ctx", "rq", "pl", "prm", "out"))
    if state["call"] == "assign":
        if not state["window"]:
            binding.maaso_score_assign(ctx, **pl, **rq, **prm, **out)
            return out
        # the windowed form advances the instances' state in place: the copy that goes in is returned
        live = dict(occ=pl["occ"].clone(), q_ticks=pl["q_ticks"].clone())
        binding.maaso_score_assign(ctx, **{**pl, **live}, **rq, **prm, **out)
        return {**out, **live}
    if state["call"] == "sweep":
        binding.maaso_placement_sweep(ctx, **pl, **rq, **prm, **out)
    elif state["call"] == "score":
        binding.maaso_placement_score(ctx, **pl, **rq, **prm, **WEIGHTS, **out)
    else:
        binding.maaso_resource_partition_requests(
            ctx, **pl, chain_offsets=state["offsets"], n_gpus=state["gpus"], **rq, tight_classes=1,
            **prm, **WEIGHTS, work=out)
    return out


# ------------------------------------------------------------------------------------------------
# what a pass cannot do without
# ------------------------------------------------------------------------------------------------

def work(case):
    """Inputs read once, outputs written once; the profile evaluation of every instance slot (about 12
    operations) at every window, and one evaluated triple (12 operations) per request and, where the
    state advances, per candidate.  A lower bound: the instances a request is compared with are left
    out, since a placement may settle them for all requests at once."""
    n, I = case["n_req"], case["i_pad"]
    if case["call"] == "partition":
        n_chain = len(workloads.all_configs()[0])
        C = sum(case["gpus"] // int(d) for d in workloads.TP_DEGREES) * (n_chain // 4)
        slots = sum((case["gpus"] // int(d)) * (case["gpus"] // int(d) + 1) // 2
                    for d in workloads.TP_DEGREES) * (n_chain // 4)
        # the split reads and writes 13 bytes a request; three request sets, 2 n requests in all
        return {"bytes": 26 * n + 15 * C * case["gpus"] + 24 * C,
                "flops": 12 * (2 * n * C + slots * 2 * math.ceil(n / case["window"]))}
    C = case["n_cand"]
    n_win = math.ceil(n / case["window"]) if case["window"] else 1
    bytes_in = (9 + (4 if case["window"] else 0)) * n + 15 * C * I + 4 * C
    if case["call"] == "assign":
        return {"bytes": bytes_in + (8 + (12 if case["latencies"] else 0)) * n + 8 + (12 * I if case["window"] else 0),
                "flops": 12 * (n + I * n_win)}
    bytes_out = (8 if case["call"] == "sweep" else 20) * C + 4
    scored = n * C if case["window"] else n
    return {"bytes": bytes_in + bytes_out, "flops": 12 * (scored + C * I * n_win)}


def tolerance(case):
    # One IEEE binary32 operation per operation of the model, in a fixed order, and integer sums: the
    # results do not depend on how a kernel tiles or schedules the work.
    return "exact"


# ------------------------------------------------------------------------------------------------
# the same in 64 bits, plain torch
# ------------------------------------------------------------------------------------------------

def _staged64(case, seed, pl, prm):
    a, p, t, d_ttft, d_tbt = (torch.from_numpy(x).cuda().double() for x in _tables(case, seed))
    tp, B = pl["tp_idx"].long(), pl["max_batch"].long() & 0xffff
    occ, q = pl["occ"].long(), pl["q_ticks"].double()
    w = B if prm["tbt_mode"] else torch.minimum(occ + 1, B)
    pen = 1.0 + prm["pen_kappa"] * (4 * w - 3 * B).clamp_min(0).double() / B
    tbt = t[tp, w] * pen
    wait = q / TICKS + (occ + 1 - B).clamp_min(0).double() / B * prm["s_bar"] * tbt
    valid = torch.arange(pl["i_pad"], device="cuda")[None, :] < pl["n_inst"].long()[:, None]
    wait = torch.where(valid, wait, torch.full_like(wait, math.inf))
    return a[tp, w], p[tp, w], tbt, wait, d_ttft, d_tbt


def exact(case, seed):
    """Static calls only: a windowed run rounds its state to whole ticks and whole requests at every
    window, so it has no 64-bit value to approach.  Chosen instances and counts are whole numbers."""
    if case["window"] or case["call"] not in ("assign", "sweep"):
        return None
    rq, pl, _, prm = _inputs(case, seed)
    a, p, tbt, wait, d_ttft, d_tbt = _staged64(case, seed, pl, prm)
    if case["call"] == "sweep":
        if pl["n_cand"] * pl["i_pad"] * case["n_slo"] > 1 << 26:
            return None
        count = torch.zeros(pl["n_cand"], dtype=torch.int64, device="cuda")
        for k in range(case["n_slo"]):
            lens = rq["prompt_len"][rq["slo_class"] == k].double().sort().values
            top = ((d_ttft[k] - wait) - a) / p  # longest prompt an instance serves in time
            top = torch.where(tbt <= d_tbt[k], top, torch.full_like(top, -1.0)).max(dim=1).values
            count += torch.searchsorted(lens, top, right=True)
        return dict(sat_count=None, sat_ratio=count.double() / case["n_req"], best_cand=None)
    if case["n_req"] * case["i_pad"] > 1 << 28:
        return None
    best = []
    for lo in range(0, case["n_req"], 1 << 18):
        s = slice(lo, lo + (1 << 18))
        L, S = rq["prompt_len"][s].double()[:, None], rq["out_len"][s].double()[:, None]
        k = rq["slo_class"][s].long()
        Dt, Db = d_ttft[k][:, None], d_tbt[k][:, None]
        De = Dt + S * Db
        ttft = wait + (a + p * L)
        e2e = ttft + S * tbt
        slack = torch.minimum(torch.minimum((Dt - ttft) / Dt, (Db - tbt) / Db), (De - e2e) / De)
        if prm["policy"]:  # among the capable instances the shortest queue, lowest index on ties
            order = torch.argsort(pl["occ"][0], stable=True)
            rank = torch.empty_like(order)
            rank[order] = torch.arange(len(order), device="cuda")
            key = torch.where(slack >= 0, 1000.0 - rank.double(), slack)
            slack = slack.gather(1, key.argmax(dim=1, keepdim=True))
        best.append(slack.max(dim=1).values)
    out = dict(chosen=None, slack=torch.cat(best), n_satisfied=None)
    if case["latencies"]:
        out.update(ttft=None, tbt=None, e2e=None)
    return out
