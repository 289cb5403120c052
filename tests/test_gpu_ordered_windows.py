"""Windows laid out by class and prompt length, against the CPU oracle: sizes around the batches (16 and 64
requests), the groups of 256 and the segments of 4096 requests, empty and single classes, ties on the between-token margin, prefills
beyond eight seconds, classes out of range, and a stream that takes more than one round of launches."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

import oracle  # noqa: E402
from paper_2509_06362_amd import binding, workloads as W  # noqa: E402

WEIGHTS = (4.0, 0.3, 2048.0, 1.0)


def variant_of(w, variant):
    """`alike`: instances of one kind that differ in their queues alone (ties); `long`: prefills of up to a minute against
    deadlines of minutes; `one class`; `one length`; `zeros`: prompts and outputs of length 0 among the others."""
    rng = W.rng_for(w.seed, 11)
    if variant == "alike":
        one = lambda x: np.ascontiguousarray(np.broadcast_to(x[:, :1], x.shape))
        w = W.replace(w, tp_idx=one(w.tp_idx), max_batch=one(w.max_batch), occ=np.zeros_like(w.occ),
                      q_ticks=w.q_ticks % np.uint64(1 << 18))
    elif variant == "long":
        w = W.replace(w, d_ttft=np.minimum(w.d_ttft * np.float32(20.0), np.float32(400.0)),
                      prompt_len=w.prompt_len * np.uint32(60))
    elif variant == "one class":
        w = W.replace(w, slo_class=np.full_like(w.slo_class, w.d_ttft.size - 1))
    elif variant == "one length":
        w = W.replace(w, prompt_len=np.full_like(w.prompt_len, 777))
    elif variant == "zeros":
        z = rng.random(w.n_req) < 0.3
        w = W.replace(w, prompt_len=np.where(z, 0, w.prompt_len).astype(np.uint32),
                      out_len=np.where(z[::-1], 0, w.out_len).astype(np.uint32))
    return w


# candidates and windows enough for the laid-out form (tests/test_window_rules.py checks that), under the shortest-queue rule too from
# 400 candidates on
SWEEPS = [
    (1001, 3, 3, 257, 3900, "mixed", 0), (1000, 2, 1, 300, 4600, "alike", 0),
    (1003, 5, 16, 271, 4110, "mixed", 1), (1003, 5, 16, 272, 4200, "mixed", 0),   # 32 batches of 16, and one group more
    (1000, 4, 8, 399, 6100, "alike", 0), (1000, 4, 8, 400, 6100, "mixed", 0),
    (1002, 3, 3, 479, 7300, "long", 0), (1002, 3, 3, 480, 7300, "one class", 1), (1000, 3, 2, 512, 7900, "zeros", 0),
    (1000, 70, 3, 500, 7600, "mixed", 0), (1000, 130, 3, 300, 2200, "alike", 0),  # two and four slots a lane
    (1001, 131, 2, 600, 3300, "mixed", 1),
    (400, 3, 3, 2048, 30_727, "one length", 0), (400, 5, 5, 4095, 61_428, "mixed", 0), (64, 4, 3, 4096, 126_977, "long", 0),
    (65, 4, 16, 4097, 127_010, "zeros", 0), (64, 140, 3, 16_390, 49_181, "alike", 0), (4100, 2, 3, 256, 3900, "mixed", 0),
    # with the sums of batches worked out ahead
    (400, 40, 3, 2048, 30_727, "long", 0), (400, 40, 3, 2048, 30_727, "mixed", 1), (64, 33, 16, 4100, 127_103, "one length", 0),
    (64, 70, 2, 4500, 139_505, "alike", 0), (64, 4, 3, 16_384, 49_652, "mixed", 1),
    (4100, 3, 3, 5000, 4500, "mixed", 0),                                         # one window, shorter than its size
]
# the same in a few windows, most of which other kernels take
FEW_WINDOWS = [
    (1001, 3, 3, 257, 600, "mixed", 0), (1000, 2, 1, 300, 901, "alike", 0), (1003, 5, 16, 320, 700, "mixed", 0),
    (1000, 4, 8, 384, 800, "alike", 0), (1000, 4, 8, 385, 800, "mixed", 0),
    (1002, 3, 3, 464, 930, "long", 0), (1002, 3, 3, 465, 940, "one class", 0), (1000, 3, 2, 512, 1024, "zeros", 0),
    (1000, 70, 3, 500, 700, "mixed", 0), (1000, 130, 3, 300, 400, "alike", 0),
    (400, 3, 3, 2048, 4100, "one length", 0), (64, 5, 5, 4095, 8190, "mixed", 0), (64, 4, 3, 4096, 8193, "long", 0),
    (65, 4, 16, 4097, 9000, "zeros", 0), (64, 140, 3, 8200, 8300, "alike", 0), (4100, 2, 3, 256, 300, "mixed", 0),
    (400, 40, 3, 2048, 4100, "long", 0), (64, 33, 16, 4100, 8300, "one length", 0), (64, 70, 2, 2500, 5100, "alike", 0),
    (64, 4, 3, 16_384, 16_900, "mixed", 0), (1000, 3, 3, 5000, 300, "mixed", 0),
]


@pytest.mark.parametrize("n_cand,i_pad,n_slo,window,n_req,variant,mode", SWEEPS + FEW_WINDOWS)
def test_sweep_and_score(n_cand, i_pad, n_slo, window, n_req, variant, mode):
    w = variant_of(W.random_small(n_cand + 31 * i_pad + window, n_cand, i_pad, n_req, n_slo=n_slo, b_cap=64, pen_kappa=0.5,
                                  jitter=variant != "alike"), variant)
    w = W.replace(w, tbt_mode=mode)
    for policy in (0, 1):
        wp = W.replace(w, policy=policy)
        print(f"laid out C={n_cand} I={i_pad} K={n_slo} window={window} R={n_req} {variant} mode={mode} policy={policy}", flush=True)
        dw = binding.DeviceWorkload(wp)
        try:
            cnt, _, best = dw.sweep(window=window)
            sc = dw.score(*WEIGHTS, window=window)
            torch.cuda.synchronize()
            ref = oracle.placement_score(wp, *WEIGHTS, window=window)
            assert np.array_equal(cnt.cpu().numpy().view(np.uint32), ref["sat_count"])
            assert int(best.item()) == int(np.argmax(ref["sat_count"]))
            for k in ("sat_count", "phi_s", "phi_t", "phi_l", "score"):
                got = sc[k].cpu().numpy()
                assert np.array_equal(got.view(np.uint32) if k == "sat_count" else got, ref[k]), k
            assert binding.maaso_ctx_device_status(dw.ctx) == 0
        finally:
            dw.close()


def check_assign(w, window, latencies, out_of_range=False):
    dw = binding.DeviceWorkload(w)
    try:
        print(f"laid-out assign I={w.i_pad} R={w.n_req} window={window} policy={w.policy}", flush=True)
        got = dw.assign(window=window, latencies=latencies)
        torch.cuda.synchronize()
        assert binding.maaso_ctx_device_status(dw.ctx) == (1 if out_of_range else 0)
        ref = oracle.score_assign(w, window=window)
        for k in ("chosen", "slack") + (("ttft", "tbt", "e2e") if latencies else ()):
            assert np.array_equal(got[k].cpu().numpy(), ref[k], equal_nan=True), k
        assert int(got["n_satisfied"].item()) == ref["n_satisfied"]
        assert np.array_equal(got["occ"].cpu().numpy()[0], ref["occ"])
        assert np.array_equal(got["q_ticks"].cpu().numpy()[0].view(np.uint64), ref["q_ticks"])
    finally:
        dw.close()


DISTRIBUTORS = [
    (2, 3, 11, 500, 0, "mixed"), (1, 1, 64, 1000, 0, "alike"), (4, 3, 48, 999, 0, "mixed"), (8, 3, 128, 1300, 0, "mixed"),
    (8, 16, 4096, 9001, 0, "long"), (16, 3, 512, 2600, 0, "mixed"), (16, 3, 1001, 5000, 0, "alike"), (8, 8, 8190, 122_853, 0, "one length"),
    (4, 3, 16_384, 114_689, 0, "mixed"), (32, 5, 2048, 129_033, 0, "zeros"), (64, 3, 4097, 520_324, 0, "mixed"),
    (100, 3, 4096, 520_193, 0, "mixed"), (256, 3, 8192, 2_088_961, 0, "mixed"),
    (2, 3, 11, 300, 1, "mixed"), (8, 3, 11, 300, 1, "mixed"), (16, 3, 32, 330, 1, "mixed"), (20, 3, 64, 700, 1, "mixed"),
    (64, 3, 64, 700, 1, "mixed"), (100, 8, 128, 393, 1, "alike"), (256, 3, 333, 2000, 1, "mixed"), (200, 16, 4096, 12_293, 1, "long"),
    (3, 3, 8192, 16_000, 1, "one class"),
]
# short streams, most of which the persistent kernel takes
SHORT_STREAMS = [
    (8, 3, 48, 999, 0, "mixed"), (40, 5, 2048, 7000, 0, "zeros"), (64, 3, 4097, 12_500, 0, "mixed"), (64, 8, 16_384, 20_000, 0, "one length"),
    (100, 3, 4096, 9000, 0, "mixed"), (256, 3, 8192, 17_000, 0, "mixed"), (16, 3, 11, 300, 1, "mixed"), (64, 3, 16, 330, 1, "mixed"),
    (100, 8, 32, 700, 1, "alike"), (200, 16, 4096, 9000, 1, "long"), (3, 3, 16_384, 16_000, 1, "one class"),
]


@pytest.mark.parametrize("i_pad,n_slo,window,n_req,policy,variant", DISTRIBUTORS + SHORT_STREAMS)
def test_distributor(i_pad, n_slo, window, n_req, policy, variant):
    half = n_req > 2_000_000  # (arrivals are 32-bit ticks: twice the requests at twice the rate)
    w = W.random_small(7 * i_pad + window, 1, i_pad, (n_req + 1) // 2 if half else n_req, n_slo=n_slo, b_cap=64, jitter=variant != "alike")
    if half:
        a = w.arrival_ticks // np.uint32(2)
        w = W.replace(w, **{k: np.tile(getattr(w, k), 2)[:n_req] for k in ("prompt_len", "out_len", "slo_class")},
                      arrival_ticks=np.concatenate([a, a + a[-1]])[:n_req])
    w = variant_of(w, variant)
    w = W.replace(w, policy=policy, n_inst=np.full_like(w.n_inst, max(1, i_pad - 1)))
    check_assign(w, window, latencies=policy == 1 or i_pad % 16 == 0)
    # no instances at all, then requests of a class that does not exist (given to nobody)
    check_assign(W.replace(w, n_inst=np.zeros_like(w.n_inst)), window, latencies=True)
    cls = w.slo_class.copy()
    cls[:: 7] = 200
    dw = binding.DeviceWorkload(W.replace(w, slo_class=cls))
    try:
        got = dw.assign(window=window)
        torch.cuda.synchronize()
        assert binding.maaso_ctx_device_status(dw.ctx) == 1
        binding.maaso_ctx_set_launch_shape(dw.ctx, 0, 0, 0, 2)  # the persistent kernel, on the state as it was given
        exp = binding.DeviceWorkload(W.replace(w, slo_class=cls))
        binding.maaso_ctx_set_launch_shape(exp.ctx, 0, 0, 0, 2)
        ref = exp.assign(window=window)
        torch.cuda.synchronize()
        assert (got["chosen"][:: 7] == -1).all()
        for k in ("chosen", "slack", "n_satisfied", "occ", "q_ticks"):
            assert torch.equal(got[k], ref[k]), k
        exp.close()
    finally:
        dw.close()


FLAGGED = [(8, 128, 700, 0), (16, 512, 2600, 0), (32, 2048, 129_100, 0), (8, 11, 200, 1), (64, 64, 700, 1), (100, 128, 400, 1), (256, 128, 1000, 1)]


@pytest.mark.parametrize("i_pad,window,n_req,policy", FLAGGED)
@pytest.mark.parametrize("mode,kappa", [(0, 0.5), (1, 0.0)])
@pytest.mark.parametrize("pause", [0, 4 << 20])
def test_distributor_with_flagged_slots(i_pad, window, n_req, policy, mode, kappa, pause):
    """Slots outside the tables, and occupancies below zero that time brings back, with a batch cap of one, one that the next
    window's batch is at once, and one that it grows to: as the persistent kernel, which evaluates every slot at every window."""
    w = W.random_small(5 * i_pad + window, 1, i_pad, n_req, n_slo=3, b_cap=64, pen_kappa=kappa)
    i = np.arange(n_req, dtype=np.uint64)
    tp, B, occ, q = w.tp_idx.copy(), w.max_batch.copy(), w.occ.copy(), w.q_ticks.copy()
    back = [1, 2, 3, i_pad - 1]  # slots that come back
    q[:, 5:] += np.uint64(60 << 20)  # most others are busy
    B[:, back], occ[:, back], q[:, back] = [1, 8, 64, 16], [-3, -5, -2, -3], 0
    tp[:, 0], B[:, i_pad // 2] = 9, 65
    w = W.replace(w, policy=policy, tbt_mode=mode, tp_idx=tp, max_batch=B, occ=occ, q_ticks=q, n_inst=np.full_like(w.n_inst, i_pad),
                  arrival_ticks=(i * 300 + i // window * np.uint64(pause)).astype(np.uint32))
    got = []
    for blocks in (0, 1):
        print(f"flagged slots I={i_pad} window={window} R={n_req} policy={policy} mode={mode} pause={pause} blocks={blocks}", flush=True)
        dw = binding.DeviceWorkload(w)
        try:
            binding.maaso_ctx_set_launch_shape(dw.ctx, 0, 0, 0, blocks)
            got.append(dw.assign(window=window))
            torch.cuda.synchronize()
            assert binding.maaso_ctx_device_status(dw.ctx) == 2
        finally:
            dw.close()
    assert np.isin(got[1]["chosen"].cpu().numpy(), back).any()
    for k in got[0]:
        assert np.array_equal(got[0][k].cpu().numpy(), got[1][k].cpu().numpy(), equal_nan=got[0][k].is_floating_point()), k


def test_distributor_overloaded_then_idle():
    """Queues of minutes build up in the first windows, most windows admit nothing, and pauses let the instances admit
    again: windows are skipped, and taken up again, in every order."""
    for seed, rate in ((3, 3000.0), (4, 60.0), (5, 900.0)):
        w = W.random_small(seed, 1, 8, 40_000, b_cap=16, queued=False)
        gaps = W.rng_for(seed, 5).exponential(1.0 / rate, size=w.n_req)
        gaps[:: 6000] += 200.0
        ticks = np.minimum(np.cumsum(gaps) * (1 << 20), 2.0 ** 32 - 1).astype(np.uint32)
        w = W.replace(w, arrival_ticks=ticks, n_inst=np.full_like(w.n_inst, 8))
        for policy in (0, 1):
            check_assign(W.replace(w, policy=policy), 128, latencies=False)


def test_distributor_in_rounds():
    """More windows than the workspace takes at a time: the state, and the count, go from one round to the next."""
    n = 11 * 9000 + 5
    w = W.random_small(12, 1, 2, n, n_slo=16, b_cap=32)
    w = W.replace(w, n_inst=np.full_like(w.n_inst, 2))
    # a window of 11 requests of sixteen classes takes 16 batches of 64 places and their bounds
    assert 9000 * 16 * (64 * 8 + 16) > 64 << 20
    check_assign(w, 11, latencies=True)


def test_distributor_unaligned_arrays_and_state_alone():
    """Arrays at odd addresses (one request per thread), and a call that asks for the count alone."""
    w = W.random_small(21, 1, 8, 4001, b_cap=32)
    w = W.replace(w, n_inst=np.full_like(w.n_inst, 8))
    ref = oracle.score_assign(w, window=128)
    dw = binding.DeviceWorkload(w)
    try:
        up = lambda x, v: torch.from_numpy(np.concatenate([np.zeros(1, x.dtype), x]).view(v)).cuda()[1:]
        rq = dict(n_req=w.n_req, prompt_len=up(w.prompt_len, np.int32), out_len=up(w.out_len, np.int32),
                  slo_class=up(w.slo_class, np.uint8), arrival_ticks=up(w.arrival_ticks, np.int32))
        pl = lambda: dict(n_cand=1, i_pad=8, n_inst=dw.n_inst, tp_idx=dw.tp_idx, max_batch=dw.max_batch,
                          occ=dw.occ.clone(), q_ticks=dw.q_ticks.clone())
        prm = dict(dw.param_args(), window=128)
        chosen = torch.empty(w.n_req + 1, dtype=torch.int32, device="cuda")[1:]
        count = torch.empty(1, dtype=torch.int64, device="cuda")
        binding.maaso_score_assign(dw.ctx, **pl(), **rq, **prm, chosen=chosen, n_satisfied=count)
        torch.cuda.synchronize()
        assert np.array_equal(chosen.cpu().numpy(), ref["chosen"]) and int(count.item()) == ref["n_satisfied"]
        live = pl()
        binding.maaso_score_assign(dw.ctx, **live, **rq, **prm, n_satisfied=count.zero_())
        torch.cuda.synchronize()
        assert int(count.item()) == ref["n_satisfied"]
        assert np.array_equal(live["occ"].cpu().numpy()[0], ref["occ"])
    finally:
        dw.close()


def test_captured_sweep_keeps_off_the_workspace():
    """A windowed sweep captured in a graph replays beside other calls of the context, which use its workspace."""
    w = W.random_small(33, 1200, 6, 4800, b_cap=32)
    dw = binding.DeviceWorkload(w)
    try:
        s = torch.cuda.Stream()
        eager = dw.sweep(window=300, stream=s)
        torch.cuda.synchronize()
        out = tuple(torch.empty_like(x) for x in eager)
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=s):
            dw.sweep(out=out, stream=s, window=300)
        for _ in range(3):
            for x in out:
                x.zero_()
            torch.cuda.synchronize()
            g.replay()
            dw.sweep(stream=s)  # static: its lengths are in the workspace
            torch.cuda.synchronize()
            for x, y in zip(out, eager):
                assert torch.equal(x, y)
    finally:
        dw.close()


def test_windowed_sweep_keeps_off_a_workspace_that_others_need():
    """Beside a captured static sweep that replays, and behind a profiled distributor call whose figures are read later."""
    w = W.random_small(33, 1200, 6, 9000, b_cap=32)
    dw = binding.DeviceWorkload(w)
    try:
        pl = dict(n_cand=1, i_pad=6, n_inst=dw.n_inst[:1], tp_idx=dw.tp_idx[:1], max_batch=dw.max_batch[:1],
                  occ=dw.occ[:1].clone(), q_ticks=dw.q_ticks[:1].clone())
        binding.maaso_ctx_window_profile(dw.ctx, True)
        binding.maaso_score_assign(dw.ctx, **pl, **dw.request_args(), **{**dw.param_args(), "policy": 0}, window=3000,
                                   arrival_ticks=dw.arrival_ticks, n_satisfied=torch.zeros(1, dtype=torch.int64, device="cuda"))
        before = binding.maaso_ctx_window_phases(dw.ctx)
        assert before["windows"] == 3
        windowed = dw.sweep(window=300)
        torch.cuda.synchronize()
        assert binding.maaso_ctx_window_phases(dw.ctx) == before
        binding.maaso_ctx_window_profile(dw.ctx, False)

        s = torch.cuda.Stream()
        static = dw.sweep(stream=s)
        torch.cuda.synchronize()
        out = tuple(torch.empty_like(x) for x in static)
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=s):
            dw.sweep(out=out, stream=s)
        for _ in range(3):
            for x in out:
                x.zero_()
            torch.cuda.synchronize()
            with torch.cuda.stream(s):
                g.replay()
            again = dw.sweep(window=300)
            torch.cuda.synchronize()
            for x, y in zip(out + again, static + windowed):
                assert torch.equal(x, y)
    finally:
        dw.close()


def laid_out_sweep_us(dw, window):
    dw.sweep(window=window)
    best = float("inf")
    for _ in range(6):
        t0, t1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        t0.record()
        dw.sweep(window=window)
        t1.record()
        torch.cuda.synchronize()
        best = min(best, t0.elapsed_time(t1) * 1e3)
    return best


def test_a_capture_leaves_later_sweeps_as_fast():
    """Captured static sweeps and distributors, of whatever size, and a distributor's profile that is still to be read cost later windowed
    sweeps nothing (without their windows laid out they take some three times as long)."""
    w = W.random_small(34, 4000, 32, 40_960, b_cap=32)
    dw = binding.DeviceWorkload(w)
    try:
        before = laid_out_sweep_us(dw, 4096)
        s = torch.cuda.Stream()
        out = dw.sweep(stream=s)
        torch.cuda.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=s):
            dw.sweep(out=out, stream=s)
        captured = laid_out_sweep_us(dw, 4096)
        pl = dict(n_cand=1, i_pad=32, n_inst=dw.n_inst[:1], tp_idx=dw.tp_idx[:1], max_batch=dw.max_batch[:1],
                  occ=dw.occ[:1].clone(), q_ticks=dw.q_ticks[:1].clone())
        binding.maaso_ctx_window_profile(dw.ctx, True)
        binding.maaso_score_assign(dw.ctx, **pl, **dw.request_args(), **{**dw.param_args(), "policy": 0}, window=3000,
                                   arrival_ticks=dw.arrival_ticks, n_satisfied=torch.zeros(1, dtype=torch.int64, device="cuda"))
        profiled = laid_out_sweep_us(dw, 4096)
        binding.maaso_ctx_window_profile(dw.ctx, False)
        # a distributor of 9,000,000 requests, which takes as much of the workspace as there is
        n = 9_000_000
        many = dict(n_req=n, slo_class=dw.request_args()["slo_class"].repeat(220)[:n], prompt_len=dw.request_args()["prompt_len"].repeat(220)[:n],
                    out_len=dw.request_args()["out_len"].repeat(220)[:n])
        arrival = torch.arange(n, dtype=torch.int32, device="cuda") * 200
        count = torch.zeros(1, dtype=torch.int64, device="cuda")
        torch.cuda.synchronize()
        g2 = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g2, stream=s):
            binding.maaso_score_assign(dw.ctx, **pl, **many, **{**dw.param_args(), "policy": 0}, window=4096, arrival_ticks=arrival,
                                       n_satisfied=count, stream=s)
        filled = laid_out_sweep_us(dw, 4096)
        print(f"windowed sweep: {before:.0f} us, behind a capture {captured:.0f}, with a profile held {profiled:.0f}, behind a capture that "
              f"fills the workspace {filled:.0f}", flush=True)
        assert captured < 1.5 * before and profiled < 1.5 * before and filled < 1.5 * before
    finally:
        dw.close()


@pytest.mark.parametrize("i_pad,window,policy", [(2, 64, 0), (6, 1024, 0), (32, 256, 1)])
def test_captured_distributor_replays_beside_other_calls(i_pad, window, policy):
    """The laid-out distributor, captured: every replay gives the eager result, with windowed sweeps laid out in between."""
    w = W.random_small(35 + i_pad, 1200, i_pad, 9000, b_cap=32)
    w = W.replace(w, policy=policy, n_inst=np.full_like(w.n_inst, i_pad))
    dw = binding.DeviceWorkload(w)
    try:
        start = dict(occ=dw.occ[:1].clone(), q_ticks=dw.q_ticks[:1].clone())
        live = {k: v.clone() for k, v in start.items()}
        out = dict(chosen=torch.empty(w.n_req, dtype=torch.int32, device="cuda"), slack=torch.empty(w.n_req, device="cuda"),
                   n_satisfied=torch.empty(1, dtype=torch.int64, device="cuda"))
        s = torch.cuda.Stream()

        def call():
            binding.maaso_score_assign(dw.ctx, n_cand=1, i_pad=i_pad, n_inst=dw.n_inst[:1], tp_idx=dw.tp_idx[:1],
                                       max_batch=dw.max_batch[:1], **live, **dw.request_args(), **dw.param_args(), window=window,
                                       arrival_ticks=dw.arrival_ticks, **out, stream=s)

        call()
        torch.cuda.synchronize()
        eager = {k: v.clone() for k, v in {**out, **live}.items()}
        ref = oracle.score_assign(w, window=window)
        assert np.array_equal(eager["chosen"].cpu().numpy(), ref["chosen"])
        windowed = [x.clone() for x in dw.sweep(window=300)]
        torch.cuda.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=s):
            call()
        for _ in range(3):
            for k, v in start.items():
                live[k].copy_(v)
            for v in out.values():
                v.zero_()
            torch.cuda.synchronize()
            with torch.cuda.stream(s):
                g.replay()
            again = dw.sweep(window=300)
            torch.cuda.synchronize()
            for k, v in {**out, **live}.items():
                assert torch.equal(v, eager[k]), k
            for x, y in zip(again, windowed):
                assert torch.equal(x, y)
    finally:
        dw.close()
