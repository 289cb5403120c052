"""Windows of a few requests, one instance per lane: the sweep, the score and the distributor against the CPU
oracle where their two forms meet (queues and slots that fit 32 bits and the tables, and ones that do not), at one
row of slots per lane and several, at four and eight candidates a block, over arrivals so close that nothing
completes between two windows, so far apart that something always does, in bursts, and in chunks of both kinds in turn; service
times of zero; slots and requests that are flagged."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

import oracle  # noqa: E402
from paper_2509_06362_amd import binding, workloads as W  # noqa: E402
from tests.test_gpu_windowed_sweep import check_against_oracle  # noqa: E402


def workload(n_cand, i_pad, n_req, variant, gaps, **kw):
    kw = dict(dict(n_slo=3, b_cap=64, pen_kappa=0.5), **kw)
    w = W.random_small(n_cand * 3 + i_pad + n_req, n_cand, i_pad, n_req, **kw)
    i = np.arange(n_req, dtype=np.uint64)
    ticks = {"close": i * 300, "far": i * 900_001, "bursts": i * 100 + i // 37 * (11 << 20)}[gaps]
    w = W.replace(w, arrival_ticks=ticks.astype(np.uint32))
    if variant == "long":       # deadlines and queues beyond 32-bit ticks
        w = W.replace(w, d_ttft=w.d_ttft * np.float32(1000.0), q_ticks=w.q_ticks * np.uint64(300),
                      prompt_len=w.prompt_len * np.uint32(700))
    elif variant == "wide":     # one queue of 2^32 ticks and more
        q = w.q_ticks.copy()
        q[:, -1] = np.uint64(5 << 32)
        w = W.replace(w, q_ticks=q, n_inst=np.full_like(w.n_inst, i_pad))
    elif variant == "full":     # batches past their cap
        w = W.replace(w, occ=(w.max_batch.astype(np.int32) + np.arange(i_pad, dtype=np.int32) % 3))
    return w


CASES = [
    (5, 1, 1, 130, "mixed", "close"), (5, 64, 1, 200, "mixed", "bursts"), (6, 65, 1, 129, "full", "far"),
    (3, 128, 1, 150, "long", "bursts"), (3, 129, 1, 100, "mixed", "bursts"), (2, 256, 1, 190, "full", "close"),
    (1030, 20, 1, 70, "full", "bursts"), (1026, 100, 1, 66, "mixed", "far"), (1025, 9, 2, 65, "wide", "bursts"),
    (7, 33, 2, 131, "full", "bursts"), (4, 70, 3, 128, "mixed", "far"), (4, 200, 2, 121, "wide", "close"),
    (2570, 40, 12, 100, "full", "bursts"), (4, 256, 4, 64, "full", "far"),
    # the longest windows of a line, and a request more (more candidates than a block each is used for)
    (2561, 8, 12, 73, "full", "bursts"), (2561, 16, 16, 81, "mixed", "far"), (2561, 24, 20, 101, "long", "bursts"),
    (2561, 40, 24, 130, "wide", "close"), (2561, 40, 25, 130, "full", "bursts"), (2561, 129, 28, 60, "full", "far"),
    # deadlines beyond 32-bit ticks: the general form's own longest windows, and a request more
    (2561, 7, 6, 40, "long", "bursts"), (2561, 8, 10, 70, "long", "bursts"), (2561, 33, 14, 90, "long", "far"),
    (2561, 33, 15, 90, "long", "bursts"), (2561, 60, 16, 130, "long", "bursts"), (2561, 100, 19, 90, "long", "far"),
    (2561, 130, 20, 70, "long", "bursts"), (2561, 200, 25, 60, "long", "close"),
]


@pytest.mark.parametrize("n_cand,i_pad,window,n_req,variant,gaps", CASES)
@pytest.mark.parametrize("kw", [{}, dict(pen_kappa=0.0, tbt_mode=1)])
def test_sweep_and_score(n_cand, i_pad, window, n_req, variant, gaps, kw):
    kw = dict(kw)
    mode = kw.pop("tbt_mode", 0)
    w = W.replace(workload(n_cand, i_pad, n_req, variant, gaps, **kw), tbt_mode=mode)
    check_against_oracle(w, window, f"short windows {variant} {gaps} {kw}")


@pytest.mark.parametrize("i_pad,window,n_req,variant,gaps", [
    (1, 1, 65, "mixed", "close"), (3, 1, 64, "full", "far"), (64, 1, 333, "mixed", "bursts"), (64, 1, 300, "full", "close"),
    (65, 1, 200, "full", "bursts"), (128, 1, 200, "long", "bursts"), (200, 1, 260, "full", "bursts"), (64, 1, 128, "wide", "far"),
    (40, 2, 127, "full", "bursts"), (64, 4, 256, "full", "far"), (100, 3, 200, "mixed", "bursts"), (256, 2, 130, "full", "close"),
    (64, 4, 255, "wide", "bursts"), (10, 1, 1, "mixed", "close"),
    # the longest windows that one wavefront takes, and one request more
    (64, 10, 205, "full", "bursts"), (64, 11, 205, "mixed", "bursts"), (65, 8, 200, "mixed", "far"), (128, 9, 200, "full", "bursts"),
    (129, 5, 130, "full", "bursts"), (256, 6, 130, "mixed", "close"), (33, 7, 140, "wide", "far"), (5, 9, 70, "long", "bursts"),
    (64, 8, 150, "long", "bursts"), (65, 6, 150, "long", "far"), (128, 7, 150, "long", "bursts"), (129, 4, 100, "long", "bursts"),
    (256, 5, 100, "long", "close"),
])
@pytest.mark.parametrize("mode,kappa", [(0, 0.5), (1, 0.0)])
def test_distributor(i_pad, window, n_req, variant, gaps, mode, kappa):
    w = W.replace(workload(2, i_pad, n_req, variant, gaps, pen_kappa=kappa), tbt_mode=mode)
    print(f"short windows I={i_pad} R={n_req} window={window} {variant} {gaps} mode={mode}", flush=True)
    dw = binding.DeviceWorkload(w)
    try:
        got = dw.assign(cand=1, window=window, latencies=True)
        torch.cuda.synchronize()
        ref = oracle.score_assign(w, cand=1, window=window)
        for key in ("chosen", "slack", "ttft", "tbt", "e2e"):
            assert np.array_equal(got[key].cpu().numpy(), ref[key], equal_nan=key != "chosen"), key
        assert int(got["n_satisfied"].item()) == ref["n_satisfied"]
        assert np.array_equal(got["occ"].cpu().numpy()[0], ref["occ"])
        assert np.array_equal(got["q_ticks"].cpu().numpy()[0].view(np.uint64), ref["q_ticks"])
        assert binding.maaso_ctx_device_status(dw.ctx) == 0
    finally:
        dw.close()


@pytest.mark.parametrize("i_pad,window,n_req", [(4, 5, 3), (4, 1, 3), (40, 1, 130), (64, 3, 128), (70, 1, 65), (100, 8, 90),
                                                (200, 1, 64), (130, 5, 12), (4, 60, 300)])
@pytest.mark.parametrize("mode", [0, 1])
@pytest.mark.parametrize("s_bar,tbt", [(1e-40, 1e-6), (1e-30, 1e-20)])
def test_nothing_completes_behind_the_last_window(i_pad, window, n_req, mode, s_bar, tbt):
    """A service time that is zero in binary32: all requests complete between two windows, however short the time, and
    none behind the last one, where no time passes."""
    w = workload(2, i_pad, n_req, "full", "close", n_slo=3)
    w = W.replace(w, n_inst=np.full_like(w.n_inst, i_pad), s_bar=np.float32(s_bar), tbt=np.full_like(w.tbt, tbt), tbt_mode=mode)
    print(f"zero service time I={i_pad} R={n_req} window={window} mode={mode} s_bar={s_bar}", flush=True)
    dw = binding.DeviceWorkload(w)
    try:
        got = dw.assign(cand=1, window=window)
        torch.cuda.synchronize()
        ref = oracle.score_assign(w, cand=1, window=window)
        assert n_req > window or int(ref["occ"].sum()) == int(w.occ[1].sum()) + ref["n_satisfied"] > 0
        for key in ("chosen", "slack"):
            assert np.array_equal(got[key].cpu().numpy(), ref[key]), key
        assert int(got["n_satisfied"].item()) == ref["n_satisfied"]
        assert np.array_equal(got["occ"].cpu().numpy()[0], ref["occ"])
        assert np.array_equal(got["q_ticks"].cpu().numpy()[0].view(np.uint64), ref["q_ticks"])
    finally:
        dw.close()


def safe_ticks(s_bar, tbt, run):
    """row_safe_ticks for windows of one request."""
    f = np.float32
    return int(f(f(s_bar) * f(tbt)) / f(run) * f(1048576.0 * (1.0 - 2.0 ** -10)))


@pytest.mark.parametrize("latencies", [True, False])
@pytest.mark.parametrize("mode,kappa", [(0, 0.5), (0, 0.0), (1, 0.5)])
@pytest.mark.parametrize("i_pad,tail", [(64, 17), (5, 64), (23, 1)])
def test_chain_and_completing_steps_in_turn(i_pad, tail, mode, kappa, latencies):
    """One request per window on up to 64 slots: chunks of 64 requests in which nothing can complete, which take the chain,
    and chunks with gaps in which requests do, in turn.  The instances start empty and the gaps are shorter than the
    service time of a single request, so what completes does so for the requests that the chain admitted."""
    chunks = "CLCCLLCLC"
    n_req = 64 * (len(chunks) - 1) + tail
    w = W.random_small(i_pad + tail, 1, i_pad, n_req, n_slo=3, b_cap=64, pen_kappa=kappa, queued=False)
    w = W.replace(w, n_inst=np.full_like(w.n_inst, i_pad), occ=np.zeros_like(w.occ), tbt_mode=mode,
                  max_batch=np.maximum(w.max_batch, 32).astype(np.uint16), prompt_len=np.minimum(w.prompt_len, 64).astype(np.uint32),
                  d_tbt=w.d_tbt * np.float32(4.0))
    least = float(w.tbt[:, 1:].min())
    alone = safe_ticks(w.s_bar, least, 1)
    gap = np.full(n_req, 300, dtype=np.uint64)
    for k, c in enumerate(chunks):
        if c == "L":
            at = 64 * k + np.array([0, 1, 20, 31, 62, 63])[k % 3:]
            gap[at] = np.uint64(alone * 9 // 10)
    assert 300 < safe_ticks(w.s_bar, least, 64) <= safe_ticks(w.s_bar, least, 32) < alone * 9 // 10  # chain; steps
    w = W.replace(w, arrival_ticks=(np.cumsum(gap) - gap).astype(np.uint32))
    print(f"chain and steps I={i_pad} R={n_req} mode={mode} kappa={kappa} latencies={latencies}", flush=True)
    ref = oracle.score_assign(w, cand=0, window=1)
    assert 0 < int(ref["occ"].sum()) < ref["n_satisfied"] // 2  # requests completed
    dw = binding.DeviceWorkload(w)
    try:
        got = dw.assign(window=1, latencies=latencies)
        torch.cuda.synchronize()
        for key in ("chosen", "slack") + (("ttft", "tbt", "e2e") if latencies else ()):
            assert np.array_equal(got[key].cpu().numpy(), ref[key], equal_nan=key != "chosen"), key
        assert int(got["n_satisfied"].item()) == ref["n_satisfied"]
        assert np.array_equal(got["occ"].cpu().numpy()[0], ref["occ"])
        assert np.array_equal(got["q_ticks"].cpu().numpy()[0].view(np.uint64), ref["q_ticks"])
        assert binding.maaso_ctx_device_status(dw.ctx) == 0
    finally:
        dw.close()


@pytest.mark.parametrize("i_pad,window,n_req", [(64, 1, 200), (64, 3, 150), (40, 10, 205), (65, 4, 130), (128, 8, 200), (130, 2, 90),
                                                (256, 5, 130), (100, 1, 130)])
@pytest.mark.parametrize("latencies", [True, False])
def test_flagged_slots_and_requests(i_pad, window, n_req, latencies):
    """Slots outside the tables, a negative occupancy and requests of an unknown class, at the short windows of every
    number of slots per lane: one wavefront and the persistent kernel give the same, and the oracle's values where it
    has any (a slot that nobody can be admitted to stands for one outside the tables, an endless prompt for an unknown
    class)."""
    w = workload(1, i_pad, n_req, "mixed", "bursts")
    tp, B, q = w.tp_idx.copy(), w.max_batch.copy(), w.q_ticks.copy()
    out = [0, i_pad // 2]
    q[:, out] = np.uint64(1 << 50)
    odd = np.arange(5, n_req, 37)
    prompt, cls = w.prompt_len.copy(), w.slo_class.copy()
    prompt[odd] = 16777215
    w = W.replace(w, n_inst=np.full_like(w.n_inst, i_pad), prompt_len=prompt)
    ref = oracle.score_assign(W.replace(w, q_ticks=q), cand=0, window=window)
    assert (ref["slack"][odd] < 0).all() and ref["n_satisfied"] > 0
    tp[:, 0] = 9
    B[:, i_pad // 2] = 65
    cls[odd] = 200
    bad = W.replace(w, tp_idx=tp, max_batch=B, slo_class=cls)
    neg = bad.occ.copy()
    neg[:, i_pad - 1] = -3
    keys = ("chosen", "slack") + (("ttft", "tbt", "e2e") if latencies else ())
    for what, x in (("outside", bad), ("negative", W.replace(bad, occ=neg))):
        got = []
        for blocks in (0, 1):
            print(f"flagged {what} I={i_pad} window={window} R={n_req} blocks={blocks} latencies={latencies}", flush=True)
            dw = binding.DeviceWorkload(x)
            try:
                binding.maaso_ctx_set_launch_shape(dw.ctx, 0, 0, 0, blocks)
                g = dw.assign(window=window, latencies=latencies)
                torch.cuda.synchronize()
                got.append({k: g[k].cpu().numpy() for k in keys + ("occ", "q_ticks", "n_satisfied")})
                assert binding.maaso_ctx_device_status(dw.ctx) == 3
            finally:
                dw.close()
        for k in got[0]:
            assert np.array_equal(got[0][k], got[1][k], equal_nan=got[0][k].dtype.kind == "f"), (what, k)
        assert (got[0]["chosen"][odd] == -1).all() and np.isneginf(got[0]["slack"][odd]).all()
        if what == "outside":
            known = np.setdiff1d(np.arange(n_req), odd)
            for k in keys:
                assert np.array_equal(got[0][k][known], ref[k][known], equal_nan=k != "chosen"), k
            assert int(got[0]["n_satisfied"].item()) == ref["n_satisfied"]
            inside = np.setdiff1d(np.arange(i_pad), out)
            assert np.array_equal(got[0]["occ"][0][inside], ref["occ"][inside])
            assert np.array_equal(got[0]["q_ticks"][0].view(np.uint64)[inside], ref["q_ticks"][inside])


@pytest.mark.parametrize("n_cand,b_cap", [(2561, 511), (4300, 511), (4300, 64), (6000, 255)])
@pytest.mark.parametrize("window", [1, 3])
def test_wavefronts_per_block(n_cand, b_cap, window):
    """Blocks of four wavefronts and of eight: which spread better, and tables that leave room for fewer than eight
    blocks of four on a compute unit."""
    check_against_oracle(workload(n_cand, 3, 20, "full", "bursts", b_cap=b_cap), window, f"blocks b_cap={b_cap}")
