"""Parity of the HIP path (through the C-ABI) with the CPU oracle, element by element.

Bar: integer outputs (chosen instance, satisfied counts, best candidate, final occupancy and queue
ticks) bit-exact; binary32 slack and latencies within 1e-5 relative - in practice they are asserted
bit-identical, because both sides perform the same sequence of IEEE operations.  A differing chosen
instance would be tolerated only where the oracle's slacks of the two instances differ by less than
1e-5 relative (check_assign reports how many such requests there are; none are expected).
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

import oracle  # noqa: E402
from paper_2509_06362_amd import binding, workloads as W  # noqa: E402

REL = 1e-5


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a GPU (run with -m 'not gpu' on CPU-only machines)")
    binding.load_library()


def u32(t):
    return t.cpu().numpy().view(np.uint32)


def oracle_counts(w, cands, window=0, threads=8):
    """Satisfied counts of the listed candidates from the triple oracle (static, or windowed with
    window > 0): independent single-threaded oracle calls, one candidate each, run side by side."""
    from concurrent.futures import ThreadPoolExecutor

    def one(c):
        if window:
            return int(oracle.placement_sweep_windowed(w, window=window, c_begin=c, c_end=c + 1)["sat_count"][c])
        return int(oracle.placement_sweep(w, c, c + 1)["sat_count"][c])
    with ThreadPoolExecutor(max_workers=threads) as pool:
        return np.array(list(pool.map(one, cands)), np.uint32)


def check_sweep(w, shapes=((0, 0, 0),), sampled=None, threshold=False):
    """GPU sweep vs the triple oracle (all candidates, or `sampled` ones) and optionally vs the
    threshold-count route on all candidates.  `shapes`: settings of the sweep's three shape knobs, which
    set what its workspace is charged with and must change nothing else."""
    dw = binding.DeviceWorkload(w)
    try:
        ref = None
        if sampled is None:
            ref = oracle.placement_sweep(w)
        thr = oracle.threshold_sweep(w) if threshold else None
        for q, group, bq in shapes:
            binding.maaso_ctx_set_launch_shape(dw.ctx, q, group, bq, 0)
            print(f"sweep {w.name} C={w.n_cand} I={w.i_pad} R={w.n_req} q={q} group={group} bq={bq}",
                  flush=True)
            cnt, ratio, best = dw.sweep()
            torch.cuda.synchronize()
            cnt, ratio, best = u32(cnt), ratio.cpu().numpy(), int(u32(best)[0])
            if ref is not None:
                assert np.array_equal(cnt, ref["sat_count"])
                assert np.array_equal(ratio, ref["sat_ratio"])
                assert best == ref["best_cand"]
            if thr is not None:
                assert np.array_equal(cnt, thr)
                assert best == int(np.argmax(thr))
                if w.n_req:
                    assert np.array_equal(ratio, (thr.astype(np.float32) / np.float32(w.n_req)))
            if sampled is not None:
                ref_s = oracle_counts(w, sampled)
                bad = np.nonzero(cnt[sampled] != ref_s)[0]
                assert bad.size == 0, f"candidates {[sampled[i] for i in bad[:8]]}"
                assert np.array_equal(ratio[sampled], ref_s.astype(np.float32) / np.float32(max(w.n_req, 1)))
            assert binding.maaso_ctx_device_status(dw.ctx) == 0
        return cnt
    finally:
        dw.close()


def check_assign(w, cand=0, window=None, window_blocks=0, latencies=True, tbt_mode=None, ref=None):
    dw = binding.DeviceWorkload(w)
    try:
        binding.maaso_ctx_set_launch_shape(dw.ctx, 0, 0, 0, window_blocks)
        print(f"assign {w.name} I={w.i_pad} R={w.n_req} window={window} blocks={window_blocks}", flush=True)
        got = dw.assign(cand=cand, window=window, latencies=latencies, tbt_mode=tbt_mode)
        torch.cuda.synchronize()
        assert binding.maaso_ctx_device_status(dw.ctx) == 0
        if ref is None:
            ref = oracle.score_assign(w, cand=cand, window=window, tbt_mode=tbt_mode)
        chosen = got["chosen"].cpu().numpy()
        slack = got["slack"].cpu().numpy()
        diff = np.nonzero(chosen != ref["chosen"])[0]
        if diff.size:  # tolerated only for near-ties; with identical arithmetic there are none
            a, b = slack[diff], ref["slack"][diff]
            assert (np.abs(a - b) <= REL * np.maximum(1.0, np.abs(b))).all(), diff[:10]
            pytest.fail(f"{diff.size} requests chose another instance within tolerance - "
                        "the two sides are expected to agree exactly")
        assert np.array_equal(slack, ref["slack"])
        fin = np.isfinite(ref["slack"])
        assert np.allclose(slack[fin], ref["slack"][fin], rtol=REL, atol=0)
        if latencies:
            for k in ("ttft", "tbt", "e2e"):
                assert np.array_equal(got[k].cpu().numpy(), ref[k], equal_nan=True), k
        assert int(got["n_satisfied"].item()) == ref["n_satisfied"]
        assert np.array_equal(got["occ"].cpu().numpy()[0], ref["occ"])
        assert np.array_equal(got["q_ticks"].cpu().numpy()[0].view(np.uint64), ref["q_ticks"])
        near = int((np.abs(ref["slack"][fin]) < REL).sum())
        print(f"  ok; requests within {REL} of a deadline: {near}", flush=True)
        return got
    finally:
        dw.close()


# ------------------------------------------------------------------------------------------------
# placer sweep
# ------------------------------------------------------------------------------------------------

@pytest.mark.parametrize("seed,n_cand,i_pad,n_req,n_slo", [
    (1, 37, 16, 3000, 3),       # ragged n_inst incl. empty candidates, ragged request tail
    (2, 200, 32, 5000, 3),
    (3, 9, 1, 700, 1),          # one slot, one class
    (4, 70, 48, 2500, 5),       # i_pad that does not divide the block
    (5, 24, 128, 1500, 8),
    (6, 10, 256, 900, 16),      # the limits: 256 slots, 16 classes
    (7, 130, 7, 64, 2),         # fewer requests than one wavefront tile
])
def test_sweep_small_irregular(seed, n_cand, i_pad, n_req, n_slo):
    w = W.random_small(seed, n_cand, i_pad, n_req, n_slo=n_slo, pen_kappa=0.5 if seed % 2 else 0.0)
    spread = 0
    for v in (w, W.stressed(w, seed=seed, deadline_scale=0.25),
              W.stressed(w, seed=seed, deadline_scale=0.03)):
        cnt = check_sweep(v, shapes=((0, 0, 0), (2, 1, 1), (4, 3, 2), (8, 64, 5), (16, 7, 100)), threshold=True)
        spread = max(spread, len(np.unique(cnt)))
    assert spread > 1, "no variant discriminates between candidates"


def test_sweep_edge_cases():
    w = W.random_small(11, 5, 8, 300)
    check_sweep(W.replace(w, n_inst=np.zeros(5, np.uint32)))                 # nothing can be served
    check_sweep(w.with_requests(0, 0))                                       # no requests
    check_sweep(w.with_requests(0, 1))                                       # one request
    check_sweep(w.with_candidates(2, 3))                                     # one candidate
    one_class = W.replace(w, slo_class=np.full(300, 2, np.uint8))            # two classes unused
    check_sweep(one_class, threshold=True)
    worst = W.replace(w, tbt_mode=1)
    check_sweep(worst, threshold=True)


def test_sweep_is_deterministic_and_leaves_inputs_alone():
    w = W.stressed(W.config1(n_cand=300, n_req=6000), seed=5)
    dw = binding.DeviceWorkload(w)
    a = [t.clone() for t in dw.sweep()]
    b = dw.sweep()
    torch.cuda.synchronize()
    for x, y in zip(a, b):
        assert torch.equal(x, y)
    assert np.array_equal(dw.occ.cpu().numpy(), w.occ)
    assert np.array_equal(dw.q_ticks.cpu().numpy().view(np.uint64), w.q_ticks)
    dw.close()


@pytest.mark.parametrize("make", [
    lambda: W.config0(),
    lambda: W.config1(n_cand=512, n_req=8192),
    lambda: W.config3(n_cand=512, n_req=4000),
    lambda: W.config4(n_cand=48, n_req=6000),
])
def test_sweep_config_shapes_reduced(make):
    w = make()
    check_sweep(w, threshold=True)
    cnt = check_sweep(W.stressed(w, seed=7), threshold=True)
    assert w.n_cand == 1 or len(np.unique(cnt)) > 1


@pytest.mark.parametrize("cfg,n_sample", [(1, 4096), (3, 4096), (4, 512)])
def test_sweep_full_size(cfg, n_sample):
    """Full configuration sizes in the default launch shape (the one the benchmark times), plain and
    stressed: against the triple oracle every candidate of config 1, 4096 seeded candidates of
    config 3 and 512 of config 4 (the oracle needs 76 ms per candidate there); and every candidate
    against the threshold-count route."""
    w = W.CONFIGS[cfg]()
    rng = np.random.default_rng(cfg)
    for v in (w, W.stressed(w, seed=cfg)):
        sampled = sorted(rng.choice(v.n_cand, size=n_sample, replace=False).tolist())
        cnt = check_sweep(v, sampled=sampled, threshold=True)
        assert cnt.max() <= v.n_req
    assert len(np.unique(cnt)) > 10


# ------------------------------------------------------------------------------------------------
# placer sweep, capacity-aware (windowed)
# ------------------------------------------------------------------------------------------------

def check_sweep_windowed(w, window, sampled=None):
    dw = binding.DeviceWorkload(w)
    try:
        print(f"windowed sweep {w.name} C={w.n_cand} I={w.i_pad} R={w.n_req} window={window}", flush=True)
        cnt, ratio, best = dw.sweep(window=window)
        torch.cuda.synchronize()
        cnt, ratio, best = u32(cnt), ratio.cpu().numpy(), int(u32(best)[0])
        assert binding.maaso_ctx_device_status(dw.ctx) == 0
        if sampled is None:
            ref = oracle.placement_sweep_windowed(w, window=window)
            assert np.array_equal(cnt, ref["sat_count"])
            assert np.array_equal(ratio, ref["sat_ratio"])
            assert best == ref["best_cand"]
        else:
            ref_s = oracle_counts(w, sampled, window=window)
            bad = np.nonzero(cnt[sampled] != ref_s)[0]
            assert bad.size == 0, f"candidates {[sampled[i] for i in bad[:8]]}"
            assert np.array_equal(ratio[sampled], ref_s.astype(np.float32) / np.float32(max(w.n_req, 1)))
            assert best == int(np.argmax(cnt))
        assert np.array_equal(dw.occ.cpu().numpy(), w.occ)            # the caller's state is untouched
        return cnt
    finally:
        dw.close()


@pytest.mark.parametrize("seed,n_cand,i_pad,n_req,n_slo,window", [
    (61, 30, 16, 3000, 3, 256), (62, 12, 1, 700, 1, 64), (63, 9, 48, 2500, 5, 1000),
    (64, 6, 128, 1500, 8, 100), (65, 4, 256, 900, 16, 333), (66, 20, 7, 300, 2, 1),
    (67, 10, 32, 2000, 3, 5000),
])
def test_windowed_sweep_small_irregular(seed, n_cand, i_pad, n_req, n_slo, window):
    w = W.random_small(seed, n_cand, i_pad, n_req, n_slo=n_slo, pen_kappa=0.5 if seed % 2 else 0.0)
    spread = 0
    for v in (w, W.stressed(w, seed=seed, deadline_scale=0.25),
              W.stressed(w, seed=seed, deadline_scale=0.03)):
        cnt = check_sweep_windowed(v, window)
        spread = max(spread, len(np.unique(cnt)))
    assert spread > 1


@pytest.mark.parametrize("seed,n_cand,i_pad,n_req,n_slo", [
    (161, 9, 1, 65, 1), (162, 7, 64, 1000, 3), (163, 5, 65, 63, 2), (164, 6, 128, 700, 8),
    (165, 3, 200, 64, 16), (166, 5, 256, 513, 3), (167, 13, 20, 1, 2), (168, 4, 31, 2, 3),
])
def test_sweep_request_by_request(seed, n_cand, i_pad, n_req, n_slo):
    """Windows of one request (every request meets the state left by all earlier ones) run in a
    kernel of their own - one wavefront per candidate, lanes = instances: counts, scores, request
    sets and the flags for out-of-range elements against the oracle's distributor at window 1."""
    w = W.random_small(seed, n_cand, i_pad, n_req, n_slo=n_slo, pen_kappa=0.5 if seed % 2 else 0.0)
    w = W.replace(w, arrival_ticks=W.poisson_arrivals(W.rng_for(seed, 3), 300.0, n_req))
    seen = set()
    for v in (w, W.stressed(w, seed=seed, deadline_scale=0.25), W.replace(w, tbt_mode=1)):
        seen.update(check_sweep_windowed(v, 1).tolist())
        check_score(v, 1, weights=SCORE_WEIGHTS[:2])
    assert len(seen) > 1 or n_req <= 2
    if n_req >= 64:
        v = W.stressed(w, seed=seed, deadline_scale=0.25)
        m = n_req // 3
        dw = binding.DeviceWorkload(v)
        try:
            alpha, beta, gt, gl = SCORE_WEIGHTS[0]
            outs = dw.score_sets([(0, m), (m, n_req), (0, n_req)], alpha, beta, gt, gl, window=1)
            torch.cuda.synchronize()
            for (lo, hi), out in zip([(0, m), (m, n_req), (0, n_req)], outs):
                ref = oracle.placement_score(v.with_requests(lo, hi), alpha, beta, gt, gl, window=1)
                for k in ("sat_count", "phi_s", "phi_t", "phi_l", "score"):
                    got = u32(out[k]) if out[k].dtype == torch.int32 else out[k].cpu().numpy()
                    assert np.array_equal(got, ref[k]), (k, lo, hi)
            assert binding.maaso_ctx_device_status(dw.ctx) == 0
        finally:
            dw.close()


def test_sweep_request_by_request_flags_out_of_range_elements():
    """A request of an unknown class is never admitted (time still passes after it) and an instance
    outside the tables is absent: the counts are those of the oracle on a stream where these requests
    are hopeless ones of a valid class and that instance is one nobody can use."""
    w = W.random_small(169, 4, 8, 300)
    w = W.replace(w, n_inst=np.full(4, 8, np.uint32),
                  arrival_ticks=W.poisson_arrivals(W.rng_for(169, 3), 300.0, 300))
    rows = [3, 77, 299]
    bad_cls = w.slo_class.copy(); bad_cls[rows] = 9
    bad_tp = w.tp_idx.copy(); bad_tp[1, 2] = 200
    dw = binding.DeviceWorkload(W.replace(w, slo_class=bad_cls, tp_idx=bad_tp))
    try:
        cnt, _, _ = dw.sweep(window=1)
        torch.cuda.synchronize()
        assert binding.maaso_ctx_device_status(dw.ctx) == 3
    finally:
        dw.close()
    hopeless = w.prompt_len.copy(); hopeless[rows] = 16777215        # minutes of prefill: never admitted
    unusable = w.q_ticks.copy(); unusable[1, 2] = 1 << 45            # a year of queued prefill
    ref = oracle.placement_sweep_windowed(W.replace(w, prompt_len=hopeless, q_ticks=unusable), window=1)
    assert np.array_equal(u32(cnt), ref["sat_count"])
    assert 0 < int(ref["sat_count"].min()) and int(ref["sat_count"].max()) < 300


@pytest.mark.parametrize("policy", [0, 1])
def test_windowed_sweep_repeats_exactly(policy):
    """Short windows, many of them, repeated on fresh contexts: every call must give the oracle's
    counts.  (Guards the publication of the per-window LDS sums: unused-result LDS atomics need an
    explicit wait before the barrier, without it single candidates came out differently from call to
    call.)"""
    w = W.random_small(161, 30, 16, 3000, n_slo=3, pen_kappa=0.5)
    w = W.replace(w, policy=policy, occ=(w.occ // 3).astype(np.int32))
    ref = oracle.placement_sweep_windowed(w, window=256)["sat_count"]
    for trial in range(3):
        dw = binding.DeviceWorkload(w)
        try:
            for rep in range(6):
                cnt, _, _ = dw.sweep(window=256)
                torch.cuda.synchronize()
                assert np.array_equal(u32(cnt), ref), (trial, rep)
        finally:
            dw.close()


def test_windowed_sweep_one_window_equals_static_sweep():
    w = W.stressed(W.config1(n_cand=64, n_req=4096), seed=9)
    w = W.replace(w, arrival_ticks=W.poisson_arrivals(W.rng_for(9, 3), 2000.0, 4096))
    a = check_sweep(w)
    b = check_sweep_windowed(w, 4096)
    assert np.array_equal(a, b)


def test_windowed_sweep_config4_shape():
    """Config 4 with its bursty arrivals, windows of 4096: reduced in full, full size on a sample."""
    small = W.config4(n_cand=24, n_req=16384)
    check_sweep_windowed(small, 4096)
    check_sweep_windowed(W.stressed(small, seed=4), 1024)
    full = W.config4()
    rng = np.random.default_rng(44)
    check_sweep_windowed(full, 4096, sampled=sorted(rng.choice(full.n_cand, 48, replace=False).tolist()))
    # request by request (the short-window kernel), and at its longest window for 128 instance slots
    check_sweep_windowed(full, 1, sampled=sorted(rng.choice(full.n_cand, 32, replace=False).tolist()))
    check_sweep_windowed(full, 16, sampled=sorted(rng.choice(full.n_cand, 32, replace=False).tolist()))


# ------------------------------------------------------------------------------------------------
# composite serving score (Sec. IV-D, Eq. 6-8)
# ------------------------------------------------------------------------------------------------
SCORE_WEIGHTS = ((4.0, 0.3, 512.0, 0.5), (10.0, 0.75, 1.0e5, 0.004), (0.0, 1.0, 2000.0, 3.0))


def check_score(w, window=0, weights=SCORE_WEIGHTS, sampled=None):
    """Every output of maaso_placement_score bit-identical to the oracle's: counts, the three
    indicators, the score and the best candidate."""
    dw = binding.DeviceWorkload(w)
    try:
        seen = set()
        for alpha, beta, gt, gl in weights:
            print(f"score {w.name} C={w.n_cand} I={w.i_pad} R={w.n_req} window={window} "
                  f"alpha={alpha} beta={beta} gamma_t={gt} gamma_l={gl}", flush=True)
            got = dw.score(alpha, beta, gt, gl, window=window)
            torch.cuda.synchronize()
            assert binding.maaso_ctx_device_status(dw.ctx) == 0
            got = {k: (u32(v) if v.dtype == torch.int32 else v.cpu().numpy()) for k, v in got.items()}
            if sampled is None:
                ref = oracle.placement_score(w, alpha, beta, gt, gl, window=window)
                for k in ("sat_count", "phi_s", "phi_t", "phi_l", "score"):
                    assert np.array_equal(got[k], ref[k]), k
                assert int(got["best_cand"][0]) == ref["best_cand"]
            else:
                for c in sampled:
                    one = oracle.placement_score(w, alpha, beta, gt, gl, window=window,
                                                 c_begin=c, c_end=c + 1)
                    for k in ("sat_count", "phi_s", "phi_t", "phi_l", "score"):
                        assert got[k][c] == one[k][c], (k, c)
                assert int(got["best_cand"][0]) == int(np.argmax(got["score"]))
            seen.update(got["score"].tolist())
        assert np.array_equal(dw.occ.cpu().numpy(), w.occ)
        return seen
    finally:
        dw.close()


@pytest.mark.parametrize("seed,n_cand,i_pad,n_req,n_slo,window", [
    (71, 30, 16, 3000, 3, 0), (72, 12, 1, 700, 1, 64), (73, 9, 48, 2500, 5, 1000),
    (74, 6, 128, 1500, 8, 0), (75, 4, 256, 900, 16, 333), (76, 20, 7, 300, 2, 1),
    (77, 10, 32, 2000, 3, 5000),
])
def test_score_small_irregular(seed, n_cand, i_pad, n_req, n_slo, window):
    w = W.random_small(seed, n_cand, i_pad, n_req, n_slo=n_slo, pen_kappa=0.5 if seed % 2 else 0.0)
    seen = set()
    for v in (w, W.stressed(w, seed=seed, deadline_scale=0.25),
              W.stressed(w, seed=seed, deadline_scale=0.03)):
        seen |= check_score(v, window)
    assert len(seen) > 3


def test_score_edge_cases():
    w = W.random_small(78, 5, 8, 400, n_slo=2)
    check_score(w.with_requests(0, 0))                                # no requests: every indicator 0
    check_score(W.replace(w, n_inst=np.zeros_like(w.n_inst)))         # no instances: nothing admitted
    hopeless = W.replace(w, d_ttft=np.full_like(w.d_ttft, 2.0 ** -20),
                         d_tbt=np.full_like(w.d_tbt, 2.0 ** -20))
    check_score(hopeless)                                             # nothing admitted anywhere
    check_score(hopeless, window=50)


def test_score_counts_match_the_sweeps():
    w = W.stressed(W.config1(n_cand=48, n_req=8192), seed=12)
    w = W.replace(w, arrival_ticks=W.poisson_arrivals(W.rng_for(12, 3), 1500.0, 8192))
    dw = binding.DeviceWorkload(w)
    try:
        for window in (0, 1024):
            cnt, _, _ = dw.sweep(window=window)
            got = dw.score(4.0, 0.3, 512.0, 0.5, window=window)
            torch.cuda.synchronize()
            assert torch.equal(cnt, got["sat_count"])
    finally:
        dw.close()


def test_score_config_shapes():
    check_score(W.config0(), weights=SCORE_WEIGHTS[:1])
    small = W.config4(n_cand=24, n_req=16384)
    check_score(small, window=4096, weights=SCORE_WEIGHTS[:2])
    check_score(W.stressed(small, seed=4), window=1024, weights=SCORE_WEIGHTS[:2])
    full = W.config4()
    rng = np.random.default_rng(45)
    picks = sorted(rng.choice(full.n_cand, 4, replace=False).tolist())
    check_score(full, window=4096, weights=SCORE_WEIGHTS[:1], sampled=picks)
    check_score(full, window=0, weights=SCORE_WEIGHTS[1:2], sampled=picks[:2])


@pytest.mark.parametrize("seed,n_cand,i_pad,n_req,window,cuts", [
    (81, 14, 24, 3000, 128, (0, 1100, 3000)),       # R_t, R_l and all of R, as Alg. 2 asks
    (82, 9, 64, 2600, 0, (0, 700, 2600)),           # static: the sets' single windows differ in size
    (83, 5, 8, 1500, 700, (0, 0, 1500)),            # an empty set among them
    (84, 21, 3, 900, 40, (0, 450, 900)),
])
def test_score_request_sets(seed, n_cand, i_pad, n_req, window, cuts):
    """One launch over several request sets (Alg. 2 scores every deployment against R_t, R_l and R)
    gives, set by set, the oracle's result for that set alone."""
    w = W.stressed(W.random_small(seed, n_cand, i_pad, n_req, n_slo=3, pen_kappa=0.5), seed=seed,
                   deadline_scale=0.2)
    a, m, b = cuts
    ranges = [(a, m), (m, b), (a, b), (m, m + (b - m) // 3)]
    alpha, beta, gt, gl = SCORE_WEIGHTS[0]
    dw = binding.DeviceWorkload(w)
    try:
        for n_sets in (4, 3, 1):
            print(f"score sets {w.name} C={n_cand} I={i_pad} R={n_req} window={window} "
                  f"ranges={ranges[:n_sets]}", flush=True)
            outs = dw.score_sets(ranges[:n_sets], alpha, beta, gt, gl, window=window)
            torch.cuda.synchronize()
            if n_sets == 4:
                outs4 = outs
            assert binding.maaso_ctx_device_status(dw.ctx) == 0
            for (lo, hi), out in zip(ranges, outs):
                ref = oracle.placement_score(w.with_requests(lo, hi), alpha, beta, gt, gl, window=window)
                for k in ("sat_count", "phi_s", "phi_t", "phi_l", "score"):
                    got = u32(out[k]) if out[k].dtype == torch.int32 else out[k].cpu().numpy()
                    assert np.array_equal(got, ref[k]), (k, lo, hi)
                assert int(u32(out["best_cand"])[0]) == ref["best_cand"]
        # the order in which the sets are given does not matter (the library runs the longest first)
        perm = [2, 0, 3, 1]
        outs_p = dw.score_sets([ranges[i] for i in perm], alpha, beta, gt, gl, window=window)
        torch.cuda.synchronize()
        for pos, i in enumerate(perm):
            for k in ("sat_count", "phi_s", "phi_t", "phi_l", "score", "best_cand"):
                assert torch.equal(outs_p[pos][k], outs4[i][k]), (k, i)
        assert np.array_equal(dw.occ.cpu().numpy(), w.occ)
    finally:
        dw.close()


def test_score_request_sets_rejects_bad_arguments():
    w = W.random_small(85, 3, 4, 200, n_slo=2)
    dw = binding.DeviceWorkload(w)
    try:
        with pytest.raises(binding.MaasoError):
            dw.score_sets([], 4.0, 0.3, 512.0, 0.5)
        with pytest.raises(binding.MaasoError):
            dw.score_sets([(0, 10)] * 5, 4.0, 0.3, 512.0, 0.5)
    finally:
        dw.close()


# ------------------------------------------------------------------------------------------------
# profiler: least-squares fit of the throughput-decay function (Sec. IV-B, Eq. 1)
# ------------------------------------------------------------------------------------------------
FIT_REL = 1e-6   # binary64 on both sides; the two log / exp implementations differ in the last place


@pytest.mark.parametrize("seed,noise,repeats,b_cap,levels", [
    (1, 0.0, 3, 128, (1, 2, 4, 8, 16, 32, 64, 128)), (2, 0.02, 3, 128, (1, 2, 4, 8, 16, 32, 64, 128)),
    (3, 0.05, 5, 64, (1, 3, 9, 27, 64)), (4, 0.1, 2, 256, (1, 2, 4, 8, 16, 32, 64, 128, 256)),
    (5, 0.002, 1, 16, (1, 2, 16)),
])
def test_profile_fit(seed, noise, repeats, b_cap, levels):
    off, lv, th, truth = W.throughput_samples(seed, levels=levels, repeats=repeats, noise=noise)
    ref_p, ref_t, ok = oracle.profile_fit(off, lv, th, b_cap)
    assert ok
    print(f"profile fit seed={seed} noise={noise} samples={len(lv)} b_cap={b_cap}", flush=True)
    params, tbt = binding.maaso_profile_fit(off, lv, th, b_cap)
    assert np.allclose(params[:, 0], ref_p[:, 0], rtol=FIT_REL)                    # T0
    assert np.allclose(params[:, 1], ref_p[:, 1], rtol=1e-5)                       # delta
    # eps is the flat direction of the residual: equal to grid resolution, not to rounding
    assert np.allclose(params[:, 2], ref_p[:, 2], rtol=1e-4)
    assert np.allclose(params[:, 3], ref_p[:, 3], rtol=1e-6, atol=1e-9)            # residual
    assert np.allclose(tbt[:, 1:], ref_t[:, 1:], rtol=FIT_REL) and np.isnan(tbt[:, 0]).all()
    # the fitted table drives the scoring path like any other
    w = W.config0()
    if b_cap >= w.b_cap:
        fitted = W.replace(w, tbt=np.ascontiguousarray(tbt[:, :w.b_cap + 1]))
        check_assign(fitted, window=0)


def test_profile_fit_error_paths():
    off, lv, th, _ = W.throughput_samples(7, levels=(1, 2, 4, 8), noise=0.0, truth=[[100.0, 0.3, 1.0]])
    with pytest.raises(binding.MaasoError) as e:                # F(b) <= 0 inside the table
        binding.maaso_profile_fit(off, lv, th, 64)
    assert e.value.status == -3
    params, tbt = e.value.partial
    ref_p, ref_t, ok = oracle.profile_fit(off, lv, th, 64)
    assert not ok and np.allclose(params[:, :3], ref_p[:, :3], rtol=1e-4)
    with pytest.raises(binding.MaasoError) as e:                # two samples for three parameters
        binding.maaso_profile_fit(np.array([0, 2], np.uint32), lv[:2], th[:2], 8)
    assert e.value.status == -3
    with pytest.raises(binding.MaasoError) as e:                # a level below 1
        binding.maaso_profile_fit(off, lv * 0.5, th, 8)
    assert e.value.status == -3
    with pytest.raises(binding.MaasoError) as e:
        binding.maaso_profile_fit(off, lv, th, 8, eps_lo=1.0, eps_hi=0.5)
    assert e.value.status == -1
    with pytest.raises(binding.MaasoError) as e:                # more cells than the kernels stage
        binding.maaso_profile_fit(off, lv, th, 4096)
    assert e.value.status == -2


# ------------------------------------------------------------------------------------------------
# placer's outer algorithms (Sec. IV-E): split by SLO, Alg. 1 bookkeeping, Alg. 2 partition scan
# ------------------------------------------------------------------------------------------------
@pytest.mark.parametrize("n_req,n_slo,mask,arrivals", [
    (0, 3, 0b1, True), (1, 2, 0b10, False), (4095, 5, 0b01001, True), (4096, 5, 0b11111, True),
    (4097, 5, 0, False), (70001, 16, 0xA5A5, True), (300000, 3, 0b100, True),
])
def test_split_by_slo(n_req, n_slo, mask, arrivals):
    w = W.random_small(81, 1, 4, max(n_req, 1), n_slo=n_slo).with_requests(0, n_req)
    arr = W.poisson_arrivals(W.rng_for(81, 3), 3000.0, n_req) if arrivals else None
    w = W.replace(w, arrival_ticks=arr)
    t, l = oracle.split_by_slo(w, mask)
    dw = binding.DeviceWorkload(w)
    try:
        print(f"split R={n_req} K={n_slo} mask={mask:#x}", flush=True)
        sp = dw.split_by_slo(mask)
        torch.cuda.synchronize()
        assert binding.maaso_ctx_device_status(dw.ctx) == 0
        n_t = int(sp["n_tight"].item())
        assert n_t == t.n_req
        for key, name in (("prompt_len_out", "prompt_len"), ("out_len_out", "out_len"),
                          ("slo_class_out", "slo_class"), ("arrival_ticks_out", "arrival_ticks")):
            if sp[key] is None:
                continue
            got = sp[key].cpu().numpy()
            got = got.view(np.uint32) if got.dtype == np.int32 else got
            assert np.array_equal(got[:n_t], getattr(t, name)), name
            assert np.array_equal(got[n_t:], getattr(l, name)), name
    finally:
        dw.close()


def chain_case(n_req, rate, n_gpus, seed, batch_set=(4, 32, 128), max_inst=256):
    w = W.partition_case(n_req=max(n_req, 1), rate=rate, seed=seed).with_requests(0, n_req)
    tp, b = W.all_configs(batch_set=list(batch_set))
    cw, offs = W.growth_chains(w, tp, b, n_gpus, max_inst=max_inst)
    return w, cw, offs, tp, b


def star_as_config(cand_star, offs):
    """Candidate indices of a chain layout -> (configuration, instance count), -1/0 where empty."""
    cfg = np.full(len(cand_star), -1, np.int64)
    cnt = np.zeros(len(cand_star), np.int64)
    for k, c in enumerate(cand_star):
        if c >= 0:
            cfg[k] = np.searchsorted(offs, c, side="right") - 1
            cnt[k] = c - offs[cfg[k]] + 1
    return cfg, cnt


@pytest.mark.parametrize("n_req,rate,n_gpus,window,max_inst", [
    (3000, 400.0, 32, 64, 256), (2000, 20.0, 16, 64, 256), (1500, 5.0, 16, 16, 256),
    (1200, 150.0, 12, 32, 5), (800, 900.0, 9, 0, 256), (0, 400.0, 8, 16, 256), (2500, 300.0, 70, 128, 256),
])
def test_ins_deploy_select_reproduces_the_sequential_greedy(n_req, rate, n_gpus, window, max_inst):
    """Scores from the oracle, bookkeeping on the GPU: Phi*[k] and I*[k] equal Alg. 1 run one
    deployment at a time."""
    w, cw, offs, tp, b = chain_case(n_req, rate, n_gpus, seed=20 + n_gpus, max_inst=max_inst)
    ref = oracle.ins_deploy(w, n_gpus, tp, b, *SCORE_WEIGHTS[0], window=window, max_inst=max_inst)
    scores = oracle.placement_score(cw, *SCORE_WEIGHTS[0], window=window)["score"]
    dw = binding.DeviceWorkload(cw)
    try:
        dev = dw.prompt_len.device
        phi = torch.empty(n_gpus + 1, dtype=torch.float32, device=dev)
        cand = torch.empty(n_gpus + 1, dtype=torch.int32, device=dev)
        print(f"select chains C={cw.n_cand} I={cw.i_pad} G={n_gpus} window={window}", flush=True)
        binding.maaso_ins_deploy_select(
            dw.ctx, n_cand=cw.n_cand, i_pad=cw.i_pad, n_inst=dw.n_inst, tp_idx=dw.tp_idx,
            score=torch.from_numpy(scores).to(dev),
            chain_offsets=torch.from_numpy(offs.view(np.int32)).to(dev), n_gpus=n_gpus,
            phi_star=phi, cand_star=cand)
        torch.cuda.synchronize()
        assert binding.maaso_ctx_device_status(dw.ctx) == 0
        assert np.array_equal(phi.cpu().numpy(), ref["phi_star"])
        cfg, cnt = star_as_config(cand.cpu().numpy(), offs)
        assert np.array_equal(cfg, ref["cfg_star"]) and np.array_equal(cnt, ref["cnt_star"])
    finally:
        dw.close()


def test_ins_deploy_select_without_chains_and_with_ties():
    """Every candidate eligible: per GPU count the largest positive score, lowest index on ties."""
    w = W.random_small(83, 700, 12, 10, n_slo=2)
    rng = np.random.default_rng(83)
    scores = (rng.integers(-2, 6, w.n_cand) * 0.25).astype(np.float32)   # many equal values, some <= 0
    k = np.array([int(w.tp_degree[w.tp_idx[c, :w.n_inst[c]]].sum()) for c in range(w.n_cand)])
    n_gpus = int(np.percentile(k, 80))                                   # some candidates do not fit
    phi_ref = np.zeros(n_gpus + 1, np.float32)
    cand_ref = np.full(n_gpus + 1, -1, np.int32)
    for c in range(w.n_cand):
        if k[c] <= n_gpus and scores[c] > phi_ref[k[c]]:
            phi_ref[k[c]], cand_ref[k[c]] = scores[c], c
    dw = binding.DeviceWorkload(w)
    try:
        dev = dw.prompt_len.device
        phi = torch.empty(n_gpus + 1, dtype=torch.float32, device=dev)
        cand = torch.empty(n_gpus + 1, dtype=torch.int32, device=dev)
        binding.maaso_ins_deploy_select(
            dw.ctx, n_cand=w.n_cand, i_pad=w.i_pad, n_inst=dw.n_inst, tp_idx=dw.tp_idx,
            score=torch.from_numpy(scores).to(dev), n_gpus=n_gpus, phi_star=phi, cand_star=cand)
        torch.cuda.synchronize()
        assert np.array_equal(phi.cpu().numpy(), phi_ref)
        assert np.array_equal(cand.cpu().numpy(), cand_ref)
        assert (cand_ref >= 0).sum() > 3
    finally:
        dw.close()


def test_resource_partition_scan():
    w = W.random_small(84, 1, 4, 10)
    dw = binding.DeviceWorkload(w)
    rng = np.random.default_rng(84)
    try:
        dev = dw.prompt_len.device
        part = torch.empty(6, dtype=torch.int32, device=dev)
        opt = torch.empty(1, dtype=torch.float32, device=dev)
        seen = set()
        for trial in range(60):
            n_gpus = int(rng.integers(0, 40)) if trial % 10 else 4096
            coarse = trial % 2 == 0   # coarse values: equal sums are common
            draw = (lambda n: (rng.integers(0, 6, n) * 0.5).astype(np.float32)) if coarse else \
                (lambda n: rng.random(n, dtype=np.float32) * 5)
            pt, pl = draw(n_gpus + 1), draw(n_gpus + 1)
            ph = None if trial % 3 == 0 else draw(n_gpus + 1) * np.float32(1.7)
            ct, cl, ch = (rng.integers(-1, 1000, n_gpus + 1).astype(np.int32) for _ in range(3))
            n = int(rng.integers(0, 50))
            n_l = int(rng.integers(0, n + 1))
            ref = oracle.resource_partition(n_gpus, pt, pl, ph, n_l, n)
            up = lambda a: None if a is None else torch.from_numpy(a).to(dev)  # noqa: E731
            binding.maaso_resource_partition(
                dw.ctx, n_gpus=n_gpus, phi_t_star=up(pt), phi_l_star=up(pl), phi_h_star=up(ph),
                cand_t_star=up(ct), cand_l_star=up(cl), cand_h_star=up(ch), n_req_l=n_l, n_req=n,
                partition=part, phi_opt=opt)
            torch.cuda.synchronize()
            got = part.cpu().numpy()
            assert got[:4].tolist() == [ref["g_t"], ref["g_l"], ref["heterogeneous"], ref["k_h"]], trial
            assert float(opt.item()) == ref["phi_opt"]
            if ref["heterogeneous"]:
                assert got[4] == ct[ref["g_t"]] and got[5] == cl[ref["g_l"]]
            else:
                assert got[5] == -1
                assert got[4] == (ch[ref["k_h"]] if (ph is not None and ref["phi_opt"] > 0) else -1)
            seen.add(ref["heterogeneous"])
        assert seen == {0, 1}
    finally:
        dw.close()


@pytest.mark.parametrize("n_req,rate,n_gpus,window,share", [
    (6000, 400.0, 32, 64, 0.5), (4000, 60.0, 24, 32, 0.2), (3000, 900.0, 16, 256, 0.8),
    (2000, 300.0, 12, 64, 1.0), (2000, 300.0, 12, 64, 0.0),
])
@pytest.mark.parametrize("one_call", [True, False])
def test_resource_partition_end_to_end(n_req, rate, n_gpus, window, share, one_call):
    """Alg. 2 against the oracle's sequential Alg. 1 + Alg. 2: as ONE library call that keeps |R_t| on
    the device (maaso_resource_partition_requests), and as the five separate calls with |R_t| read
    back by the host in between."""
    w = W.partition_case(n_req=n_req, rate=rate, seed=30 + n_gpus, tight_share=share)
    tp, b = W.all_configs(batch_set=[4, 16, 64])
    cw, offs = W.growth_chains(w, tp, b, n_gpus)
    wts = SCORE_WEIGHTS[0]
    r_t, r_l = oracle.split_by_slo(w, 0b1)
    ref = {tag: oracle.ins_deploy(ws, n_gpus, tp, b, *wts, window=window)
           for tag, ws in (("t", r_t), ("l", r_l), ("h", w))}
    part = oracle.resource_partition(n_gpus, ref["t"]["phi_star"], ref["l"]["phi_star"],
                                     ref["h"]["phi_star"], r_l.n_req, w.n_req)
    dw = binding.DeviceWorkload(cw)
    try:
        print(f"alg2 R={n_req} G={n_gpus} C={cw.n_cand} window={window} share={share}", flush=True)
        run = dw.resource_partition if one_call else dw.resource_partition_steps
        got = run(offs, 0b1, n_gpus, *wts, window=window)
        torch.cuda.synchronize()
        assert binding.maaso_ctx_device_status(dw.ctx) == 0
        assert int(got["n_tight"]) == r_t.n_req
        if one_call:
            for name, key in (("prompt_len", "prompt_len_split"), ("out_len", "out_len_split"),
                              ("arrival_ticks", "arrival_ticks_split")):
                both = np.concatenate([getattr(r_t, name), getattr(r_l, name)])
                assert np.array_equal(got[key].cpu().numpy().view(np.uint32), both), name
        for tag in ("t", "l", "h"):
            assert np.array_equal(got[f"phi_{tag}_star"].cpu().numpy(), ref[tag]["phi_star"]), tag
            cfg, cnt = star_as_config(got[f"cand_{tag}_star"].cpu().numpy(), offs)
            assert np.array_equal(cfg, ref[tag]["cfg_star"]) and np.array_equal(cnt, ref[tag]["cnt_star"])
        p = got["partition"].cpu().numpy()
        assert p[:4].tolist() == [part["g_t"], part["g_l"], part["heterogeneous"], part["k_h"]]
        assert float(got["phi_opt"].item()) == part["phi_opt"]
    finally:
        dw.close()


@pytest.mark.parametrize("window,homogeneous,share", [(0, True, 0.5), (64, False, 0.3), (0, False, 1.0),
                                                      (1, True, 0.6)])
def test_resource_partition_one_call_equals_the_five_calls(window, homogeneous, share):
    """Static scoring, no homogeneous fallback, an empty side, request-by-request windows: the one-call
    form writes what the step-by-step form writes, array by array."""
    w = W.partition_case(n_req=1500, rate=300.0, seed=44, tight_share=share)
    tp, b = W.all_configs(batch_set=[4, 16, 64])
    cw, offs = W.growth_chains(w, tp, b, 12)
    wts = SCORE_WEIGHTS[0]
    dw = binding.DeviceWorkload(cw)
    try:
        print(f"alg2 one call vs steps window={window} homogeneous={homogeneous} share={share}", flush=True)
        one = dw.resource_partition(offs, 0b1, 12, *wts, window=window, homogeneous=homogeneous)
        torch.cuda.synchronize()
        steps = dw.resource_partition_steps(offs, 0b1, 12, *wts, window=window, homogeneous=homogeneous)
        torch.cuda.synchronize()
        assert binding.maaso_ctx_device_status(dw.ctx) == 0
        assert int(one["n_tight"]) == steps["n_tight"]
        tags = ("t", "l", "h") if homogeneous else ("t", "l")
        for tag in tags:
            for key in (f"score_{tag}", f"phi_{tag}_star", f"cand_{tag}_star"):
                assert torch.equal(one[key], steps[key]), key
        assert torch.equal(one["partition"], steps["partition"])
        assert torch.equal(one["phi_opt"], steps["phi_opt"])
        assert torch.equal(one["prompt_len_split"], steps["split"]["prompt_len_out"])
        assert torch.equal(one["slo_class_split"], steps["split"]["slo_class_out"])
    finally:
        dw.close()


def test_resource_partition_at_bench_size():
    """The workload `bench.py --workload alg2` times (131,072 requests, 64 GPUs, 24 configurations ->
    720 deployments), whole pipeline against the sequential oracle."""
    import bench
    n_gpus, wts = bench.ALG2_GPUS, bench.ALG2_SCORE_WEIGHTS
    w = W.partition_case(n_req=131072, rate=400.0)
    tp, b = W.all_configs()
    cw, offs = W.growth_chains(w, tp, b, n_gpus)
    window = int(w.window)
    r_t, r_l = oracle.split_by_slo(w, 0b1)
    print("oracle: sequential Alg. 1 on R_t, R_l, R ...", flush=True)
    ref = {tag: oracle.ins_deploy(ws, n_gpus, tp, b, *wts, window=window)
           for tag, ws in (("t", r_t), ("l", r_l), ("h", w))}
    part = oracle.resource_partition(n_gpus, ref["t"]["phi_star"], ref["l"]["phi_star"],
                                     ref["h"]["phi_star"], r_l.n_req, w.n_req)
    dw = binding.DeviceWorkload(cw)
    try:
        print(f"alg2 full size C={cw.n_cand} I={cw.i_pad} R={cw.n_req}", flush=True)
        got = dw.resource_partition(offs, 0b1, n_gpus, *wts, window=window)
        torch.cuda.synchronize()
        assert binding.maaso_ctx_device_status(dw.ctx) == 0
        for tag in ("t", "l", "h"):
            assert np.array_equal(got[f"phi_{tag}_star"].cpu().numpy(), ref[tag]["phi_star"]), tag
            cfg, cnt = star_as_config(got[f"cand_{tag}_star"].cpu().numpy(), offs)
            assert np.array_equal(cfg, ref[tag]["cfg_star"]) and np.array_equal(cnt, ref[tag]["cnt_star"])
        p = got["partition"].cpu().numpy()
        assert p[:4].tolist() == [part["g_t"], part["g_l"], part["heterogeneous"], part["k_h"]]
        assert float(got["phi_opt"].item()) == part["phi_opt"]
    finally:
        dw.close()


def prune_on_gpu(ctx, dev, offsets, sat, lat, n_cand=None):
    n_cand = len(sat) if n_cand is None else n_cand
    keep = torch.full((len(sat),), 255, dtype=torch.uint8, device=dev)
    n_kept = torch.full((len(offsets) - 1,), -1, dtype=torch.int32, device=dev)
    binding.maaso_batch_size_prune(
        ctx, n_cand=n_cand, group_offsets=torch.from_numpy(np.asarray(offsets, np.uint32).view(np.int32)).to(dev),
        sat_count=torch.from_numpy(np.ascontiguousarray(sat).view(np.int32)).to(dev),
        latency=torch.from_numpy(np.ascontiguousarray(lat)).to(dev), keep=keep, n_kept=n_kept)
    torch.cuda.synchronize()
    return keep.cpu().numpy(), u32(n_kept)


@pytest.mark.parametrize("seed,sizes", [(1, [7, 0, 19, 1, 64]), (2, [256, 257, 3]), (3, [1000]),
                                        (4, [5] * 40), (5, [2047, 513])])
def test_batch_size_prune_matches_the_definition(seed, sizes):
    """Pareto pruning of batch sizes per parallelism configuration: groups of every size around the
    kernel's tile of 256 (ragged tails, empty groups), few distinct values so that ties abound,
    candidates that serve nobody - keep flags and per-group counts bit for bit."""
    rng = np.random.default_rng(300 + seed)
    offsets = np.concatenate([[0], np.cumsum(sizes)])
    n = int(offsets[-1])
    sat = (rng.integers(0, 12, n) * rng.integers(0, 2, n) * 7).astype(np.uint32)
    lat = (rng.integers(0, 16, n) / 16.0).astype(np.float32)
    ref_keep, ref_n = oracle.batch_size_prune(offsets, sat, lat)
    dw = binding.DeviceWorkload(W.config0())
    try:
        print(f"prune seed={seed} groups={len(sizes)} n={n}", flush=True)
        keep, n_kept = prune_on_gpu(dw.ctx, dw.prompt_len.device, offsets, sat, lat)
        assert binding.maaso_ctx_device_status(dw.ctx) == 0
        assert np.array_equal(keep, ref_keep)
        assert np.array_equal(n_kept, ref_n)
    finally:
        dw.close()


def test_batch_size_prune_edge_cases():
    rng = np.random.default_rng(9)
    sat = rng.integers(1, 9, 40).astype(np.uint32)
    lat = rng.random(40).astype(np.float32)
    dw = binding.DeviceWorkload(W.config0())
    try:
        dev = dw.prompt_len.device
        # a group that runs backwards and one that runs past the end: flagged and skipped, the
        # others served; candidates outside every group are not written
        offsets = [0, 10, 5, 12, 41]
        ref_keep, ref_n = oracle.batch_size_prune(offsets, sat, lat)
        keep, n_kept = prune_on_gpu(dw.ctx, dev, offsets, sat, lat)
        assert binding.maaso_ctx_device_status(dw.ctx) == 8
        assert np.array_equal(keep, ref_keep) and np.array_equal(n_kept, ref_n)
        assert (keep[12:] == 255).all() and n_kept.tolist() == [int(ref_n[0]), 0, int(ref_n[2]), 0]
        # NaN latency: compares false both ways, so the candidate stays and removes nobody
        lat2 = lat.copy()
        lat2[3] = np.nan
        ref_keep, ref_n = oracle.batch_size_prune([0, 40], sat, lat2)
        keep, n_kept = prune_on_gpu(dw.ctx, dev, [0, 40], sat, lat2)
        assert np.array_equal(keep, ref_keep) and keep[3] == 1 and np.array_equal(n_kept, ref_n)
        # no groups: nothing to do; missing arrays: refused
        binding.maaso_batch_size_prune(dw.ctx, n_cand=0, group_offsets=torch.zeros(1, dtype=torch.int32, device=dev),
                                       sat_count=None, latency=None, keep=None,
                                       n_kept=torch.zeros(1, dtype=torch.int32, device=dev))
        with pytest.raises(binding.MaasoError) as e:
            binding.maaso_batch_size_prune(dw.ctx, n_cand=4, group_offsets=torch.zeros(2, dtype=torch.int32, device=dev),
                                           sat_count=None, latency=None, keep=None,
                                           n_kept=torch.zeros(1, dtype=torch.int32, device=dev))
        assert e.value.status == -1
    finally:
        dw.close()


@pytest.mark.parametrize("window,rate", [(64, 300.0), (16, 900.0), (0, 300.0)])
def test_batch_size_prune_of_scored_configurations(window, rate):
    """The step as the placer uses it: every (strategy, batch size) pair as a single fresh instance,
    scored against the requests by maaso_placement_score, pruned per strategy on (admitted requests,
    Phi_L) - against the oracle's score followed by the oracle's pruning."""
    w = W.partition_case(n_req=3000, rate=rate, seed=61)
    batch_set = [1, 2, 4, 8, 16, 32, 64, 128]
    tp, b = W.all_configs(batch_set=batch_set)
    cw, _ = W.growth_chains(w, tp, b, 8, max_inst=1)          # one instance per configuration
    assert cw.n_cand == len(tp)
    offsets = np.arange(0, len(tp) + 1, len(batch_set))       # strategy-major: one group per strategy
    wts = SCORE_WEIGHTS[0]
    ref = oracle.placement_score(cw, *wts, window=window)
    ref_keep, ref_n = oracle.batch_size_prune(offsets, ref["sat_count"], ref["phi_l"])
    dw = binding.DeviceWorkload(cw)
    try:
        print(f"prune scored configurations window={window} rate={rate} C={cw.n_cand}", flush=True)
        dev = dw.prompt_len.device
        got = dw.score(*wts, window=window)
        keep = torch.full((cw.n_cand,), 255, dtype=torch.uint8, device=dev)
        n_kept = torch.zeros(len(offsets) - 1, dtype=torch.int32, device=dev)
        binding.maaso_batch_size_prune(
            dw.ctx, n_cand=cw.n_cand, group_offsets=torch.from_numpy(offsets.astype(np.int32)).to(dev),
            sat_count=got["sat_count"], latency=got["phi_l"], keep=keep, n_kept=n_kept)
        torch.cuda.synchronize()
        assert binding.maaso_ctx_device_status(dw.ctx) == 0
        assert np.array_equal(u32(got["sat_count"]), ref["sat_count"])
        assert np.array_equal(got["phi_l"].cpu().numpy(), ref["phi_l"])
        assert np.array_equal(keep.cpu().numpy(), ref_keep)
        assert np.array_equal(u32(n_kept), ref_n)
        assert 0 < int(ref_n.sum()) < cw.n_cand or window == 0   # something goes, something stays
    finally:
        dw.close()


def test_outer_algorithm_error_paths():
    w, cw, offs, tp, b = chain_case(200, 100.0, 8, seed=7)
    dw = binding.DeviceWorkload(cw)
    try:
        dev = dw.prompt_len.device
        score = torch.ones(cw.n_cand, dtype=torch.float32, device=dev)
        phi = torch.empty(4098, dtype=torch.float32, device=dev)
        cand = torch.empty(4098, dtype=torch.int32, device=dev)
        args = dict(n_cand=cw.n_cand, i_pad=cw.i_pad, n_inst=dw.n_inst, tp_idx=dw.tp_idx, score=score,
                    phi_star=phi, cand_star=cand)
        with pytest.raises(binding.MaasoError) as e:
            binding.maaso_ins_deploy_select(dw.ctx, n_gpus=4097, **args)
        assert e.value.status == -2
        # a chain list that runs backwards, and one that runs past the candidates: flagged, ignored
        bad = torch.tensor([0, 5, 3, cw.n_cand + 1], dtype=torch.int32, device=dev)
        binding.maaso_ins_deploy_select(dw.ctx, n_gpus=8, chain_offsets=bad, **args)
        torch.cuda.synchronize()
        assert binding.maaso_ctx_device_status(dw.ctx) == 8
        assert np.count_nonzero(cand[:9].cpu().numpy() >= 0) == 1     # only chain [0, 5) counted
        with pytest.raises(binding.MaasoError) as e:
            binding.maaso_resource_partition(dw.ctx, n_gpus=4, phi_t_star=phi, phi_l_star=phi,
                                             n_req_l=5, n_req=4, partition=cand, phi_opt=phi)
        assert e.value.status == -1
        # the one-call form refuses a work set without a required array, before launching anything
        work = dw.partition_work(8)
        del work["partition"]
        with pytest.raises(binding.MaasoError) as e:
            dw.resource_partition(offs, 0b1, 8, 4.0, 0.3, 512.0, 0.5, window=16, work=work)
        assert e.value.status == -1
        work = dw.partition_work(8)
        del work["phi_h_star"]      # score_h given, its list not
        with pytest.raises(binding.MaasoError) as e:
            dw.resource_partition(offs, 0b1, 8, 4.0, 0.3, 512.0, 0.5, window=16, work=work)
        assert e.value.status == -1
        # a profile loaded without GPU counts cannot drive Alg. 1's bookkeeping
        ctx = binding.maaso_profile_tables_load(cw.n_tp, cw.b_cap, cw.prefill_a, cw.prefill_p, cw.tbt,
                                                cw.d_ttft, cw.d_tbt, None, 0)
        try:
            with pytest.raises(binding.MaasoError) as e:
                binding.maaso_ins_deploy_select(ctx, n_gpus=8, **args)
            assert e.value.status == -1
        finally:
            ctx.close()
    finally:
        dw.close()


# ------------------------------------------------------------------------------------------------
# distributor, static
# ------------------------------------------------------------------------------------------------

def test_assign_config0_full():
    w = W.config0()
    check_assign(w)
    check_assign(W.stressed(w, seed=2))
    check_assign(w, tbt_mode=1)


@pytest.mark.parametrize("seed,i_pad,n_req,n_slo", [(21, 12, 5000, 3), (22, 1, 300, 1),
                                                    (23, 256, 1200, 16), (24, 64, 70000, 8),
                                                    (25, 33, 257, 2), (27, 8, 4003, 3),
                                                    (28, 5, 999, 4), (29, 9, 1000, 3)])
def test_assign_static_irregular(seed, i_pad, n_req, n_slo):
    w = W.random_small(seed, 3, i_pad, n_req, n_slo=n_slo, pen_kappa=0.5 if seed % 2 else 0.0)
    w = W.replace(w, n_inst=np.array([i_pad, max(1, i_pad // 2), 0], np.uint32))
    for cand in range(3):
        check_assign(w, cand=cand, window=0)
    check_assign(w, cand=0, window=0, latencies=False)


def test_assign_empty_and_identical_instances():
    w = W.random_small(31, 1, 6, 400)
    w = W.replace(w, n_inst=np.array([6], np.uint32))
    check_assign(w.with_requests(0, 0), window=0)
    for arr in (w.tp_idx, w.max_batch, w.occ, w.q_ticks):
        arr[0, 1:] = arr[0, 0]
    got = check_assign(w, window=0)
    assert (got["chosen"].cpu().numpy() == 0).all()            # lowest index among equal slacks


def test_assign_streaming_shape_sampled():
    """The bandwidth-bound shape (4 instances, long stream) at 2^22 requests."""
    w = W.streaming_shape(n_req=1 << 22)
    check_assign(w, window=0)


# ------------------------------------------------------------------------------------------------
# shortest-queue rule (policy 1) on every path that chooses an instance
# ------------------------------------------------------------------------------------------------
def shortest_queue(w, coarse_queues=True):
    """Policy 1 on `w`; with coarse_queues the queue lengths collide often (ties by index)."""
    occ = (w.occ // 3).astype(np.int32) if coarse_queues else w.occ
    return W.replace(w, policy=1, occ=occ)


@pytest.mark.parametrize("seed,i_pad,n_req,n_slo", [(121, 12, 5000, 3), (122, 1, 300, 1),
                                                    (123, 200, 2000, 8), (124, 256, 1027, 16),
                                                    (125, 7, 10001, 2), (126, 8, 4099, 3)])
def test_assign_static_shortest_queue(seed, i_pad, n_req, n_slo):
    w = W.random_small(seed, 1, i_pad, n_req, n_slo=n_slo, pen_kappa=0.5 if seed % 2 else 0.0)
    w = W.replace(w, n_inst=np.array([i_pad], np.uint32))
    differs = 0
    for v in (w, W.stressed(w, seed=seed), W.stressed(w, seed=seed, deadline_scale=0.05)):
        for coarse in (True, False):
            for lat in (True, False):
                got = check_assign(shortest_queue(v, coarse), window=0, latencies=lat)
            ref0 = oracle.score_assign(v, window=0)
            differs += int((got["chosen"].cpu().numpy() != ref0["chosen"]).sum())
    assert differs > 0 or i_pad == 1


def test_assign_static_shortest_queue_unaligned():
    w = shortest_queue(W.stressed(W.random_small(127, 1, 20, 3001, n_slo=3), seed=3))
    w = W.replace(w, n_inst=np.array([20], np.uint32))
    dw = binding.DeviceWorkload(w)
    try:
        dev = dw.prompt_len.device
        R = w.n_req - 1
        chosen = torch.empty(R + 1, dtype=torch.int32, device=dev)
        slack = torch.empty(R + 1, dtype=torch.float32, device=dev)
        n_sat = torch.empty(1, dtype=torch.int64, device=dev)
        binding.maaso_score_assign(
            dw.ctx, n_cand=1, i_pad=w.i_pad, n_inst=dw.n_inst, tp_idx=dw.tp_idx, max_batch=dw.max_batch,
            occ=dw.occ, q_ticks=dw.q_ticks, n_req=R, prompt_len=dw.prompt_len[1:],
            out_len=dw.out_len[1:], slo_class=dw.slo_class[1:], **dw.param_args(), chosen=chosen[1:],
            slack=slack[1:], n_satisfied=n_sat)
        torch.cuda.synchronize()
        ref = oracle.score_assign(w.with_requests(1, R + 1), window=0)
        assert np.array_equal(chosen[1:].cpu().numpy(), ref["chosen"])
        assert np.array_equal(slack[1:].cpu().numpy(), ref["slack"])
        assert int(n_sat.item()) == ref["n_satisfied"]
    finally:
        dw.close()


@pytest.mark.parametrize("seed,i_pad,n_inst,window,blocks", [
    (141, 8, 5, 64, 2), (142, 100, 77, 200, 32), (143, 256, 256, 128, 64), (144, 3, 3, 1000, 0),
    (145, 64, 64, 1, 1),
])
def test_assign_windowed_shortest_queue(seed, i_pad, n_inst, window, blocks):
    w = W.random_small(seed, 1, i_pad, 6000 if window > 1 else 300, n_slo=3, pen_kappa=0.25)
    w = W.replace(w, n_inst=np.array([n_inst], np.uint32), policy=1,
                  arrival_ticks=W.poisson_arrivals(W.rng_for(seed, 3), 800.0, w.n_req))
    check_assign(w, window=window, window_blocks=blocks)
    check_assign(W.stressed(w, seed=seed), window=window, window_blocks=blocks, latencies=False)


def test_assign_windowed_shortest_queue_config2_reduced():
    w = W.replace(W.config2(n_req=16384, window=512), policy=1)
    got = check_assign(w, window=512)
    ref0 = oracle.score_assign(W.replace(w, policy=0), window=512)
    assert (got["chosen"].cpu().numpy() != ref0["chosen"]).mean() > 0.05
    check_assign(W.replace(w, tbt_mode=1), window=512)      # with the worst-case estimate: the paper's rule


@pytest.mark.parametrize("seed,n_cand,i_pad,n_req,n_slo,window", [
    (161, 30, 16, 3000, 3, 256), (162, 9, 48, 2500, 5, 1000), (163, 4, 256, 900, 16, 333),
    (164, 20, 7, 300, 2, 1), (165, 12, 32, 2000, 3, 0),
])
def test_sweep_and_score_shortest_queue(seed, n_cand, i_pad, n_req, n_slo, window):
    w = W.random_small(seed, n_cand, i_pad, n_req, n_slo=n_slo, pen_kappa=0.5 if seed % 2 else 0.0)
    for v in (w, W.stressed(w, seed=seed, deadline_scale=0.25)):
        v = shortest_queue(v)
        if window:
            check_sweep_windowed(v, window)
        else:
            check_sweep(v)                      # static counts do not depend on the rule
        check_score(v, window, weights=SCORE_WEIGHTS[:2])


@pytest.mark.parametrize("window", [0, 300, 1])
def test_assign_on_a_row_selected_on_the_device(window):
    """Sweep, then distribute over the sweep's best candidate without the index leaving the GPU; and
    over every other row in turn; an out-of-range index is flagged and treated as an empty placement."""
    w = W.stressed(W.random_small(131, 9, 24, 2000, n_slo=3, pen_kappa=0.25), seed=5, deadline_scale=0.25)
    w = W.replace(w, arrival_ticks=W.poisson_arrivals(W.rng_for(131, 3), 700.0, 2000))
    dw = binding.DeviceWorkload(w)
    try:
        dev = dw.prompt_len.device
        cnt, _, best = dw.sweep()
        got = dw.assign_selected(best, window=window)
        torch.cuda.synchronize()
        b = int(best.item())
        assert b == oracle.placement_sweep(w)["best_cand"]
        rows = [(best, b, got)]
        for c in range(w.n_cand):
            sel = torch.tensor([c], dtype=torch.int32, device=dev)
            rows.append((sel, c, dw.assign_selected(sel, window=window)))
        torch.cuda.synchronize()
        assert binding.maaso_ctx_device_status(dw.ctx) == 0
        for sel, c, g in rows:
            ref = oracle.score_assign(w, cand=c, window=window)
            assert np.array_equal(g["chosen"].cpu().numpy(), ref["chosen"]), c
            assert np.array_equal(g["slack"].cpu().numpy(), ref["slack"])
            for k in ("ttft", "tbt", "e2e"):
                assert np.array_equal(g[k].cpu().numpy(), ref[k], equal_nan=True)
            assert int(g["n_satisfied"].item()) == ref["n_satisfied"]
            occ = g["occ"].cpu().numpy()
            assert np.array_equal(occ[c], ref["occ"])
            assert np.array_equal(np.delete(occ, c, axis=0), np.delete(w.occ, c, axis=0))   # other rows untouched
            assert np.array_equal(g["q_ticks"].cpu().numpy()[c].view(np.uint64), ref["q_ticks"])
        bad = torch.tensor([w.n_cand], dtype=torch.int32, device=dev)
        g = dw.assign_selected(bad, window=window)
        torch.cuda.synchronize()
        assert binding.maaso_ctx_device_status(dw.ctx) == 2
        assert (g["chosen"].cpu().numpy() == -1).all() and int(g["n_satisfied"].item()) == 0
    finally:
        dw.close()


def test_assign_static_unaligned_arrays_take_the_scalar_path():
    """Request and output arrays offset by one element are only 4-byte aligned."""
    w = W.stressed(W.random_small(26, 1, 20, 3001, n_slo=3), seed=3)
    w = W.replace(w, n_inst=np.array([20], np.uint32))
    dw = binding.DeviceWorkload(w)
    dev = dw.prompt_len.device
    R = w.n_req - 1
    chosen = torch.empty(R + 1, dtype=torch.int32, device=dev)
    slack = torch.empty(R + 1, dtype=torch.float32, device=dev)
    n_sat = torch.empty(1, dtype=torch.int64, device=dev)
    binding.maaso_score_assign(
        dw.ctx, n_cand=1, i_pad=w.i_pad, n_inst=dw.n_inst, tp_idx=dw.tp_idx, max_batch=dw.max_batch,
        occ=dw.occ, q_ticks=dw.q_ticks, n_req=R, prompt_len=dw.prompt_len[1:], out_len=dw.out_len[1:],
        slo_class=dw.slo_class[1:], **dw.param_args(), chosen=chosen[1:], slack=slack[1:],
        n_satisfied=n_sat)
    torch.cuda.synchronize()
    ref = oracle.score_assign(w.with_requests(1, R + 1), window=0)
    assert np.array_equal(chosen[1:].cpu().numpy(), ref["chosen"])
    assert np.array_equal(slack[1:].cpu().numpy(), ref["slack"])
    assert int(n_sat.item()) == ref["n_satisfied"]
    dw.close()


@pytest.mark.parametrize("seed,n_cand,i_pad,n_req,fresh_share", [
    (91, 40, 32, 5000, 0.5), (92, 25, 7, 3000, 0.3), (93, 12, 128, 2500, 0.8),
    (94, 6, 256, 1200, 0.1), (95, 60, 1, 900, 0.5), (96, 33, 48, 20000, 0.97),
])
def test_sweep_with_fresh_and_loaded_instances_mixed(seed, n_cand, i_pad, n_req, fresh_share):
    """Instances without a queue wait and instances with one inside the same candidates, in every
    proportion and with odd and even numbers of each."""
    base = W.stressed(W.random_small(seed, n_cand, i_pad, n_req, n_slo=3, pen_kappa=0.5), seed=seed,
                      deadline_scale=0.04)   # tight: a fresh instance serves short prompts only
    rng = np.random.default_rng(seed)
    fresh = rng.random((n_cand, i_pad)) < fresh_share
    w = W.replace(base, occ=np.where(fresh, 0, base.occ).astype(base.occ.dtype),
                  q_ticks=np.where(fresh, 0, base.q_ticks).astype(base.q_ticks.dtype))
    cnt = check_sweep(w, shapes=((0, 0, 0), (2, 1, 1), (16, 3, 2)), threshold=True)
    assert (cnt > 0).any() and (cnt < n_req).any()   # neither everything nor nothing is served
    dw = binding.DeviceWorkload(w)
    try:
        dw.sweep()
        pairs, nowait = binding.maaso_ctx_sweep_evaluated(dw.ctx, split=True)
        assert 0 < nowait < pairs
    finally:
        dw.close()


def test_sweep_reports_the_pairs_it_evaluated():
    """Pairs that reach the latency loop = sum over (candidate, class) of the instances whose
    between-token latency meets the class deadline, times the requests of that class; those of an
    instance without a queue wait are reported separately (the sweep skips their addition)."""
    w = W.stressed(W.config4(n_cand=40, n_req=5000), seed=2)
    # every third instance slot fresh (no queued prefill, nothing running): a mix of both kinds
    fresh = (np.arange(w.i_pad)[None, :] + np.arange(w.n_cand)[:, None]) % 3 == 0
    w = W.replace(w, occ=np.where(fresh, 0, w.occ).astype(w.occ.dtype),
                  q_ticks=np.where(fresh, 0, w.q_ticks).astype(w.q_ticks.dtype))
    dw = binding.DeviceWorkload(w)
    cnt, _, _ = dw.sweep()
    got, got_nowait = binding.maaso_ctx_sweep_evaluated(dw.ctx, split=True)
    per_class = np.bincount(w.slo_class, minlength=w.n_slo).astype(np.int64)
    want = want_nowait = 0
    for c in range(w.n_cand):
        st = oracle.stage(w, c)
        for k in range(w.n_slo):
            ok = st["tbt"] <= w.d_tbt[k]
            want += int(ok.sum()) * int(per_class[k])
            want_nowait += int((ok & (st["wait"] == 0)).sum()) * int(per_class[k])
    assert (got, got_nowait) == (want, want_nowait)
    assert 0 < got_nowait < got < w.valid_triples()
    assert np.array_equal(u32(cnt), oracle.placement_sweep(w)["sat_count"])
    dw.close()


# ------------------------------------------------------------------------------------------------
# distributor, windowed
# ------------------------------------------------------------------------------------------------

@pytest.mark.parametrize("n_req,window,blocks", [
    (8192, 512, 0), (8192, 512, 1), (8192, 512, 8), (8192, 512, 256),
    (5000, 384, 0),        # ragged last window
    (300, 1, 4),           # one request per window
    (3000, 4096, 0),       # a single window larger than the stream
    (6000, 3000, 16),      # exactly two windows
])
def test_assign_windowed_config2_reduced(n_req, window, blocks):
    w = W.config2(n_req=n_req, window=window)
    got = check_assign(w, window=window, window_blocks=blocks)
    assert (got["occ"].cpu().numpy() >= 0).all()


@pytest.mark.parametrize("seed,i_pad,n_inst,window,blocks", [
    (41, 8, 5, 64, 2), (42, 100, 77, 200, 32), (43, 256, 256, 128, 64), (44, 3, 3, 1000, 0),
    (45, 16, 0, 50, 4),
])
def test_assign_windowed_irregular(seed, i_pad, n_inst, window, blocks):
    w = W.random_small(seed, 1, i_pad, 4000, n_slo=4, pen_kappa=0.25)
    w = W.replace(w, n_inst=np.array([n_inst], np.uint32))
    check_assign(w, window=window, window_blocks=blocks)


@pytest.mark.parametrize("seed,i_pad,n_inst,n_req,window", [
    (141, 1, 1, 130, 1), (142, 64, 64, 1000, 1), (143, 65, 65, 63, 2), (144, 128, 100, 700, 3),
    (145, 200, 200, 64, 4), (146, 256, 256, 513, 1), (147, 20, 0, 70, 1), (148, 31, 31, 1, 1),
    (149, 8, 5, 4097, 4),
])
def test_assign_request_by_request(seed, i_pad, n_inst, n_req, window):
    """Windows of 1 to 4 requests - the online distributor taken literally - run on one wavefront with
    the instances in its lanes: every output and the final state against the oracle, with and without
    the latency outputs, at the state as generated and under load; the persistent kernel, asked for
    through its blocks knob, must give the same."""
    w = W.random_small(seed, 1, i_pad, n_req, n_slo=4, pen_kappa=0.25)
    w = W.replace(w, n_inst=np.array([n_inst], np.uint32),
                  arrival_ticks=W.poisson_arrivals(W.rng_for(seed, 3), 200.0, n_req))
    for v in (w, W.stressed(w, seed=seed, deadline_scale=0.25), W.replace(w, tbt_mode=1)):
        ref = oracle.score_assign(v, window=window)
        check_assign(v, window=window, ref=ref)
        check_assign(v, window=window, latencies=False, ref=ref)
        check_assign(v, window=window, window_blocks=2, ref=ref)


def test_assign_request_by_request_flags_out_of_range_elements():
    w = W.random_small(150, 1, 8, 300)
    w = W.replace(w, n_inst=np.array([8], np.uint32),
                  arrival_ticks=W.poisson_arrivals(W.rng_for(150, 3), 300.0, 300))
    rows = [3, 77, 299]
    bad_cls = w.slo_class.copy(); bad_cls[rows] = 9
    bad_tp = w.tp_idx.copy(); bad_tp[0, 2] = 200
    dw = binding.DeviceWorkload(W.replace(w, slo_class=bad_cls, tp_idx=bad_tp))
    try:
        got = dw.assign(window=1)
        torch.cuda.synchronize()
        assert binding.maaso_ctx_device_status(dw.ctx) == 3
        ch = got["chosen"].cpu().numpy()
        assert (ch[rows] == -1).all() and (ch != 2).all()
        assert np.isneginf(got["slack"].cpu().numpy()[rows]).all()
        assert np.isnan(got["ttft"].cpu().numpy()[rows]).all()
    finally:
        dw.close()
    hopeless = w.prompt_len.copy(); hopeless[rows] = 16777215
    unusable = w.q_ticks.copy(); unusable[0, 2] = 1 << 45
    ref = oracle.score_assign(W.replace(w, prompt_len=hopeless, q_ticks=unusable), window=1)
    keep = np.ones(300, bool); keep[rows] = False
    assert np.array_equal(ch[keep], ref["chosen"][keep])
    assert int(got["n_satisfied"].item()) == ref["n_satisfied"]


def test_windowed_with_one_window_matches_static_outputs():
    w = W.config2(n_req=4096, window=4096)
    a = check_assign(w, window=0)
    b = check_assign(w, window=4096)
    assert torch.equal(a["chosen"], b["chosen"]) and torch.equal(a["slack"], b["slack"])


def test_assign_windowed_config2_full():
    """The online-distributor configuration at full size (2^22 requests, 1024 windows of 4096)."""
    w = W.config2()
    ref = oracle.score_assign(w, latencies=False)
    for k in ("ttft", "tbt", "e2e"):
        ref.pop(k)
    check_assign(w, window=w.window, latencies=False, ref=ref)


# ------------------------------------------------------------------------------------------------
# argument and precondition handling
# ------------------------------------------------------------------------------------------------

# ------------------------------------------------------------------------------------------------
# seeded random combinations of shape, window, rule, estimate mode and penalty on every entry point
# ------------------------------------------------------------------------------------------------
@pytest.mark.parametrize("seed", range(40))
def test_random_combinations(seed):
    rng = np.random.default_rng(9000 + seed)
    n_cand = int(rng.integers(1, 25))
    i_pad = int(rng.choice([1, 2, 3, 5, 8, 9, 16, 31, 64, 100, 256]))
    n_req = int(rng.choice([0, 1, 63, 64, 65, 255, 257, 1000, 1024, 2500, 4099]))
    n_slo = int(rng.choice([1, 2, 3, 7, 16]))
    window = int(rng.choice([0, 1, 17, 64, 256, 300, 1024, 5000]))
    w = W.random_small(9000 + seed, n_cand, i_pad, max(n_req, 1), n_slo=n_slo,
                       pen_kappa=float(rng.choice([0.0, 0.25, 1.5]))).with_requests(0, n_req)
    if rng.random() < 0.5:
        w = W.stressed(w, seed=seed, deadline_scale=float(rng.choice([1.0, 0.25, 0.05])))
    w = W.replace(w, policy=int(rng.integers(0, 2)), tbt_mode=int(rng.integers(0, 2)),
                  arrival_ticks=W.poisson_arrivals(W.rng_for(seed, 3), float(rng.choice([50.0, 800.0, 20000.0])),
                                                   n_req))
    print(f"combo seed={seed} C={n_cand} I={i_pad} R={n_req} K={n_slo} window={window} policy={w.policy} "
          f"tbt_mode={w.tbt_mode} kappa={float(w.pen_kappa)}", flush=True)
    check_sweep(w)
    if window and n_req:
        check_sweep_windowed(w, window)
    check_score(w, window if n_req else 0, weights=SCORE_WEIGHTS[:1])
    c = int(rng.integers(0, n_cand))
    one = w.with_candidates(c, c + 1)
    check_assign(one, window=window, window_blocks=int(rng.choice([0, 1, 3, 16, 64])))


def largest_tables(n_tp, b_cap, seed):
    """A profile that fills the table limit (n_tp * (b_cap + 1) = 2048 cells), eight instances per
    candidate drawn over all rows and batch sizes, Poisson arrivals."""
    rng = np.random.default_rng(seed)
    t = np.arange(n_tp, dtype=np.float64)[:, None]
    b = np.arange(b_cap + 1, dtype=np.float64)[None, :]
    a = np.broadcast_to(0.02 / (1 + t) ** 0.3, (n_tp, b_cap + 1)) * rng.uniform(0.9, 1.1, (n_tp, b_cap + 1))
    p = np.broadcast_to(4e-5 / (1 + t) ** 0.3, (n_tp, b_cap + 1)) * rng.uniform(0.9, 1.1, (n_tp, b_cap + 1))
    tb = 0.012 / (1 + t) ** 0.2 * (1 + 0.002 * b) * rng.uniform(0.9, 1.1, (n_tp, b_cap + 1))
    tabs = []
    for m in (a, p, tb):
        m32 = m.astype(np.float32)
        m32[:, 0] = np.nan
        tabs.append(np.ascontiguousarray(m32))
    n_cand, i_pad, n_req = 12, 8, 3000
    w = W.random_small(seed, n_cand, i_pad, n_req, n_slo=3)
    max_batch = rng.integers(1, b_cap + 1, size=(n_cand, i_pad)).astype(np.uint16)
    return W.replace(
        w, name=f"largest_tables_{n_tp}x{b_cap}", tp_degree=np.ones(n_tp, np.uint32), b_cap=b_cap,
        prefill_a=tabs[0], prefill_p=tabs[1], tbt=tabs[2],
        tp_idx=rng.integers(0, n_tp, size=(n_cand, i_pad)).astype(np.uint16).astype(np.uint8)
        if n_tp <= 256 else (rng.integers(0, 256, size=(n_cand, i_pad))).astype(np.uint8),
        max_batch=max_batch, occ=(rng.random((n_cand, i_pad)) * max_batch * 1.5).astype(np.int32),
        arrival_ticks=W.poisson_arrivals(W.rng_for(seed, 3), 500.0, n_req))


@pytest.mark.parametrize("n_tp,b_cap", [(1, 2047), (1024, 1), (8, 255)])
def test_tables_at_the_size_limit(n_tp, b_cap):
    w = largest_tables(n_tp, b_cap, seed=300 + n_tp)
    check_sweep(w, threshold=True)
    check_sweep_windowed(w, 256)
    check_score(w, 500, weights=SCORE_WEIGHTS[:1])
    one = W.replace(w.with_candidates(3, 4), n_inst=np.array([8], np.uint32))
    check_assign(one, window=0)
    check_assign(one, window=200)
    with pytest.raises(binding.MaasoError) as e:        # one more cell is refused at load
        binding.maaso_profile_tables_load(1, 2048, np.ones((1, 2049), np.float32), np.ones((1, 2049), np.float32),
                                          np.ones((1, 2049), np.float32), w.d_ttft, w.d_tbt, None, 0)
    assert e.value.status == -2


def test_host_side_argument_errors():
    w = W.random_small(51, 2, 8, 100)
    dw = binding.DeviceWorkload(w)
    dev = dw.prompt_len.device
    cnt = torch.empty(2, dtype=torch.int32, device=dev)
    base = dict(n_cand=2, i_pad=8, n_inst=dw.n_inst, tp_idx=dw.tp_idx, max_batch=dw.max_batch,
                occ=dw.occ, q_ticks=dw.q_ticks, **dw.request_args(), **dw.param_args())

    def status(fn, **kw):
        with pytest.raises(binding.MaasoError) as e:
            fn(dw.ctx, **{**base, **kw})
        return e.value.status

    sweep, assign = binding.maaso_placement_sweep, binding.maaso_score_assign
    assert status(sweep, sat_count=None) == -1
    assert status(sweep, sat_count=cnt, window=4) == -1                 # windowed without arrivals
    assert status(sweep, sat_count=cnt, i_pad=257) == -2
    assert status(sweep, sat_count=cnt, i_pad=0) == -2
    assert status(sweep, sat_count=cnt, s_bar=0.0) == -1
    assert status(sweep, sat_count=cnt, pen_kappa=-1.0) == -1
    assert status(sweep, sat_count=cnt, tbt_mode=2) == -1
    assert status(sweep, sat_count=cnt, n_inst=None) == -1
    assert status(sweep, sat_count=cnt, prompt_len=None) == -1
    n_sat = torch.empty(1, dtype=torch.int64, device=dev)
    assert status(assign, n_satisfied=n_sat) == -1                      # n_cand must be 1
    assert status(assign, n_cand=1) == -1                               # no output at all
    assert status(assign, n_cand=1, n_satisfied=n_sat, window=16) == -1  # windowed without arrivals
    dw.close()


def test_out_of_range_elements_are_flagged_not_followed():
    w = W.random_small(52, 4, 8, 500)
    w = W.replace(w, n_inst=np.full(4, 8, np.uint32))
    bad_cls = w.slo_class.copy(); bad_cls[[3, 77, 400]] = 9
    bad_tp = w.tp_idx.copy(); bad_tp[1, 2] = 200
    bad_b = w.max_batch.copy(); bad_b[2, 0] = 0; bad_b[2, 5] = 60000
    wb = W.replace(w, slo_class=bad_cls, tp_idx=bad_tp, max_batch=bad_b)
    dw = binding.DeviceWorkload(wb)
    cnt, _, _ = dw.sweep()
    torch.cuda.synchronize()
    assert binding.maaso_ctx_device_status(dw.ctx) == 3
    assert binding.maaso_ctx_device_status(dw.ctx) == 0                    # cleared by the read
    # the flagged elements count as absent: same result as removing them
    keep = np.ones(500, bool); keep[[3, 77, 400]] = False
    ref_w = W.replace(w, prompt_len=w.prompt_len[keep].copy(), out_len=w.out_len[keep].copy(),
                      slo_class=w.slo_class[keep].copy(), arrival_ticks=None)
    ref = oracle.placement_sweep(ref_w)["sat_count"]
    got = u32(cnt)
    assert got[0] == ref[0] and got[3] == ref[3]
    got_a = dw.assign(cand=1, window=0)
    torch.cuda.synchronize()
    assert binding.maaso_ctx_device_status(dw.ctx) == 3
    ch = got_a["chosen"].cpu().numpy()
    assert (ch[[3, 77, 400]] == -1).all() and (ch != 2).all()
    dw.close()


def test_inter_window_wait_gives_up_cleanly():
    """A spin limit of zero makes the first block to reach a window boundary give up: the kernel
    must end by itself and the status must say so."""
    w = W.config2(n_req=8192, window=256)
    dw = binding.DeviceWorkload(w)
    binding.maaso_ctx_set_launch_shape(dw.ctx, 0, 0, 0, 64)
    binding.maaso_ctx_set_wait_limit(dw.ctx, 0)
    occ0, q0 = dw.occ.clone(), dw.q_ticks.clone()
    gave_up = dw.assign(window=256)
    with pytest.raises(binding.MaasoError) as e:
        binding.maaso_ctx_device_status(dw.ctx)
    assert e.value.status == -6
    # what such a call leaves behind is defined: the count is marked incomplete, the state is as given
    assert int(gave_up["n_satisfied"].item()) & (1 << 63) or int(gave_up["n_satisfied"].item()) < 0
    assert torch.equal(gave_up["occ"], occ0[0:1]) and torch.equal(gave_up["q_ticks"], q0[0:1])
    binding.maaso_ctx_set_wait_limit(dw.ctx, 1 << 22)
    got = dw.assign(window=256)                      # the context is usable again
    torch.cuda.synchronize()
    assert binding.maaso_ctx_device_status(dw.ctx) == 0
    ref = oracle.score_assign(w, window=256)
    assert np.array_equal(got["chosen"].cpu().numpy(), ref["chosen"])
    dw.close()


# ------------------------------------------------------------------------------------------------
# random shapes, every path
# ------------------------------------------------------------------------------------------------

@pytest.mark.parametrize("seed", [11, 12, 13])
def test_random_shapes_every_path(seed):
    """Forty random small workloads per seed - slot counts around the lane and tile sizes, request
    counts around the block sizes (zero included), 1 to 16 classes, windows from one request to more
    than there are requests - through the static sweep (both entry points), the capacity-aware sweep,
    the composite score and the distributor (static and windowed, both selection rules): counts, best
    candidates, choices, slacks and final states bit for bit."""
    from dataclasses import replace
    rng = np.random.default_rng(seed)
    for case in range(40):
        s = int(rng.integers(1, 1 << 30))
        i_pad = int(rng.choice([1, 2, 3, 7, 8, 9, 16, 31, 32, 33, 64, 65, 128, 200, 256]))
        n_cand = int(rng.integers(1, 60))
        n_req = int(rng.choice([0, 1, 5, 63, 64, 65, 255, 256, 257, 1000, 2049, 4100]))
        n_slo = int(rng.choice([1, 2, 3, 5, 16]))
        window = int(rng.choice([1, 2, 3, 4, 16, 17, 64, 256, 300, 1024, 5000]))
        w = W.random_small(s, n_cand, i_pad, n_req, n_slo=n_slo, b_cap=int(rng.choice([8, 32, 128])),
                           over_cap=bool(rng.integers(0, 2)), queued=bool(rng.integers(0, 2)),
                           pen_kappa=float(rng.choice([0.0, 0.5])))
        what = f"case {case}: seed={s} C={n_cand} I={i_pad} R={n_req} K={n_slo} window={window}"
        print(what, flush=True)
        dw = binding.DeviceWorkload(w)
        try:
            ref = oracle.placement_sweep(w)
            cnt, _, best = dw.sweep()
            torch.cuda.synchronize()
            assert np.array_equal(u32(cnt), ref["sat_count"]) and int(best.item()) == int(ref["best_cand"]), what
            cnt, _, best = dw.sweep(noalloc=True)
            torch.cuda.synchronize()
            assert np.array_equal(u32(cnt), ref["sat_count"]) and int(best.item()) == int(ref["best_cand"]), what
            if n_req == 0:
                continue
            refw = oracle.placement_sweep_windowed(w, window=window)
            cnt, _, best = dw.sweep(window=window)
            torch.cuda.synchronize()
            assert np.array_equal(u32(cnt), refw["sat_count"]) and int(best.item()) == int(refw["best_cand"]), what
            refs = oracle.placement_score(w, *SCORE_WEIGHTS[0], window=window)
            sc = dw.score(*SCORE_WEIGHTS[0], window=window)
            torch.cuda.synchronize()
            assert np.array_equal(sc["score"].cpu().numpy(), refs["score"]), what
            assert np.array_equal(u32(sc["sat_count"]), refs["sat_count"]), what
            c = int(rng.integers(0, n_cand))
            for win in (0, window):
                for policy in (0, 1):
                    w2 = w if policy == 0 else replace(w, policy=1)
                    dwx = dw if policy == 0 else binding.DeviceWorkload(w2)
                    try:
                        r = oracle.score_assign(w2, cand=c, window=win)
                        got = dwx.assign(cand=c, window=win)
                        torch.cuda.synchronize()
                        assert np.array_equal(got["chosen"].cpu().numpy(), r["chosen"]), (what, win, policy)
                        assert np.array_equal(got["slack"].cpu().numpy(), r["slack"], equal_nan=True), (what, win, policy)
                        assert int(got["n_satisfied"].item()) == r["n_satisfied"], (what, win, policy)
                        if win:
                            assert np.array_equal(got["occ"].cpu().numpy()[0], r["occ"]), (what, win, policy)
                            assert np.array_equal(got["q_ticks"].cpu().numpy()[0].view(np.uint64), r["q_ticks"])
                    finally:
                        if dwx is not dw:
                            dwx.close()
        finally:
            dw.close()


# ------------------------------------------------------------------------------------------------
# the boundary's promises: no allocation in compute calls, order between streams, one call at a time
# ------------------------------------------------------------------------------------------------

def _all_compute_calls(dw, w, window):
    """Every compute entry point once on the resident workload; returns the static sweep's counts."""
    cnt = dw.sweep()[0].clone()
    dw.sweep(window=window)
    dw.sweep(noalloc=True)
    dw.score(4.0, 0.3, 512.0, 0.5, window=window)
    dw.score_sets([(0, w.n_req // 2), (w.n_req // 2, w.n_req)], 4.0, 0.3, 512.0, 0.5, window=window)
    dw.assign(cand=0, window=0)
    dw.assign(cand=0, window=window)
    dw.assign(cand=0, window=1)
    best = torch.zeros(1, dtype=torch.int32, device=cnt.device)
    dw.assign_selected(best, window=0)
    dw.resource_partition(np.array([0, w.n_cand], np.uint32), 0b1, 64, 4.0, 0.3, 512.0, 0.5, window=window)
    torch.cuda.synchronize()
    return u32(cnt)


def test_compute_calls_never_allocate():
    """After maaso_profile_tables_load (and one maaso_ctx_reserve for shapes beyond the default
    workspace) no compute entry point changes the context's workspace, at growing shapes; a shape
    beyond what is held is refused before anything runs."""
    shapes = [(5, 8, 300), (60, 32, 5000), (300, 128, 20000), (20, 256, 70000)]
    ws = [W.random_small(700 + i, c, ip, r, n_slo=3) for i, (c, ip, r) in enumerate(shapes)]
    ws = [W.replace(w, arrival_ticks=W.poisson_arrivals(W.rng_for(700 + i, 3), 900.0, w.n_req))
          for i, w in enumerate(ws)]
    ctx0 = None
    for w in ws:
        dw = binding.DeviceWorkload(w)
        try:
            before = binding.maaso_ctx_workspace(dw.ctx)
            assert before == (64 << 20, 1)
            cnt = _all_compute_calls(dw, w, window=250)
            assert binding.maaso_ctx_workspace(dw.ctx) == before
            assert np.array_equal(cnt, oracle.placement_sweep(w)["sat_count"])
            assert binding.maaso_ctx_device_status(dw.ctx) == 0
        finally:
            dw.close()
    # beyond the default: 150,000 candidates of 32 slots need 77 MB of records
    big = W.config1(n_cand=150000, n_req=512)
    dw = binding.DeviceWorkload(big)
    try:
        with pytest.raises(binding.MaasoError) as e:
            dw.sweep()
        assert e.value.status == -7 and "maaso_ctx_reserve" in str(e.value)
        assert binding.maaso_ctx_workspace(dw.ctx) == (64 << 20, 1)
        binding.maaso_ctx_reserve(dw.ctx, big.n_cand, big.i_pad, big.n_req)
        held = binding.maaso_ctx_workspace(dw.ctx)
        assert held[1] == 2 and held[0] >= 16 * 150000 * 32
        for shape in ((0, 0, 0), (2, 1, 0), (16, 64, 0)):
            binding.maaso_ctx_set_launch_shape(dw.ctx, shape[0], shape[1], shape[2], 0)
            cnt = dw.sweep()[0]
            torch.cuda.synchronize()
            assert binding.maaso_ctx_workspace(dw.ctx) == held
        binding.maaso_ctx_reserve(dw.ctx, 10, 8, 100)                 # never shrinks, nothing to do
        assert binding.maaso_ctx_workspace(dw.ctx) == held
        sample = [0, 77777, 149999]
        for c in sample:
            assert u32(cnt)[c] == oracle.placement_sweep(big, c, c + 1)["sat_count"][c]
    finally:
        dw.close()


def test_calls_on_different_streams_are_ordered_by_the_library():
    """One context, calls alternating between two streams without any wait in between: each call
    works in the same workspace, so it must run behind the one before it."""
    w = W.stressed(W.config1(n_cand=500, n_req=9000), seed=71)
    ref = oracle.placement_sweep(w)
    dw = binding.DeviceWorkload(w)
    try:
        streams = [torch.cuda.Stream(), torch.cuda.Stream(), None]
        outs = []
        for i in range(12):
            st = streams[i % 3]
            outs.append(dw.sweep(stream=st if st is not None else torch.cuda.default_stream()))
        torch.cuda.synchronize()
        for cnt, ratio, best in outs:
            assert np.array_equal(u32(cnt), ref["sat_count"])
            assert int(u32(best)[0]) == ref["best_cand"]
        assert binding.maaso_ctx_device_status(dw.ctx) == 0
    finally:
        dw.close()


def test_a_second_thread_is_turned_away_not_mixed_in():
    """Two host threads on one context: a call either runs (and is right) or is refused as busy."""
    import threading
    w = W.stressed(W.config1(n_cand=200, n_req=4000), seed=72)
    ref = oracle.placement_sweep(w)["sat_count"]
    dw = binding.DeviceWorkload(w)
    results, busy, errors = [], [0], []

    def worker():
        torch.cuda.set_device(0)
        for _ in range(60):
            try:
                results.append(dw.sweep()[0])
            except binding.MaasoError as e:
                if e.status == -8:
                    busy[0] += 1
                else:
                    errors.append(e)
    try:
        ts = [threading.Thread(target=worker) for _ in range(2)]
        for t in ts:
            t.start()
        for t in ts:
            t.join()
        torch.cuda.synchronize()
        assert not errors
        assert len(results) + busy[0] == 120 and len(results) >= 2
        for cnt in results:
            assert np.array_equal(u32(cnt), ref)
        print(f"  {len(results)} calls ran, {busy[0]} were refused as busy", flush=True)
    finally:
        dw.close()


def test_valu_probe_reports_a_plausible_rate():
    """The instrumentation kernel that measures what the chip sustains for the sweep's instruction mix:
    a rate between a tenth of and the whole nominal peak (256 CUs x 4 SIMDs x 32 lanes x 2.4 GHz),
    the scalar-operand and compare patterns clearly below the all-register ones; bad arguments refused."""
    rates = [binding.maaso_probe_valu(p, 2048) for p in range(5)]
    peak = 256 * 4 * 32 * 2.4e9
    for (rate, n), expect in zip(rates, (24, 40, 96, 16, 8)):
        assert n == expect and 0.1 * peak < rate < 1.05 * peak
    assert rates[4][0] < 0.85 * rates[2][0] and rates[3][0] < 0.85 * rates[2][0]
    with pytest.raises(binding.MaasoError) as e:
        binding.maaso_probe_valu(5, 16)
    assert e.value.status == -1
    with pytest.raises(binding.MaasoError) as e:
        binding.maaso_probe_valu(0, 0)
    assert e.value.status == -1


def test_batch_size_prune_of_overlapping_groups():
    """Offsets that run backwards: a candidate of several groups goes by the last, however the blocks end.  The first
    group is the longest to prune, so it ends last."""
    rng = np.random.default_rng(19)
    n = 900
    sat = rng.integers(0, 9, n).astype(np.uint32)
    lat = rng.random(n).astype(np.float32)
    offsets = [0, n, 3, 300, 100, 700]
    ref_keep, ref_n = oracle.batch_size_prune(offsets, sat, lat)
    dw = binding.DeviceWorkload(W.config0())
    try:
        keep, n_kept = prune_on_gpu(dw.ctx, dw.prompt_len.device, offsets, sat, lat)
        assert np.array_equal(keep, ref_keep) and np.array_equal(n_kept, ref_n)
    finally:
        dw.close()


def test_batch_size_prune_of_many_groups():
    """More groups than a block each, and than every block looks through: in order, and with steps backwards, one at each end and
    in between; small ones, and large ones among them."""
    rng = np.random.default_rng(23)
    dw = binding.DeviceWorkload(W.config0())
    try:
        for groups, large in ((1024, 0), (1025, 40), (2048, 0), (2049, 0), (2051, 300), (2200, 128), (5000, 65), (8192, 129), (8195, 64)):
            n = 3 * groups
            sat = rng.integers(0, 5, n).astype(np.uint32)
            lat = rng.integers(0, 6, n).astype(np.float32)
            valid = np.sort(rng.integers(0, n + 1, groups + 1))
            if large:  # groups of that many among the others
                at = int(valid[groups // 3])
                valid[groups // 3 + 1:] = np.maximum(valid[groups // 3 + 1:], min(at + large, n))
            backwards = valid.copy()
            for at in (1, groups // 2, groups):
                backwards[at] = max(0, int(backwards[at]) - 40)
            for offsets in (valid, backwards):
                print(f"prune of {groups} groups, backwards {bool((np.diff(offsets) < 0).any())}", flush=True)
                ref_keep, ref_n = oracle.batch_size_prune(offsets, sat, lat)
                keep, n_kept = prune_on_gpu(dw.ctx, dw.prompt_len.device, offsets, sat, lat)
                assert np.array_equal(keep, ref_keep) and np.array_equal(n_kept, ref_n)
                status = binding.maaso_ctx_device_status(dw.ctx)
                assert status == (8 if (np.diff(offsets) < 0).any() else 0)
    finally:
        dw.close()


def test_batch_size_prune_grows_with_the_number_of_groups():
    """Four times the groups take some four times as long: not every block may look through all of them."""
    dw = binding.DeviceWorkload(W.config0())
    dev = dw.prompt_len.device
    best = {}
    try:
        for groups in (65_536, 262_144):
            offsets = (torch.arange(groups + 1, device=dev) * 2).to(torch.int32)
            sat = torch.ones(2 * groups, dtype=torch.int32, device=dev)
            lat = torch.rand(2 * groups, device=dev)
            keep = torch.empty(2 * groups, dtype=torch.uint8, device=dev)
            n_kept = torch.empty(groups, dtype=torch.int32, device=dev)
            for _ in range(6):
                t0, t1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
                t0.record()
                binding.maaso_batch_size_prune(dw.ctx, n_cand=2 * groups, group_offsets=offsets, sat_count=sat, latency=lat,
                                               keep=keep, n_kept=n_kept)
                t1.record()
                torch.cuda.synchronize()
                best[groups] = min(best.get(groups, 1e9), t0.elapsed_time(t1))
            assert int(n_kept.sum()) == int(keep.sum()) >= groups
    finally:
        dw.close()
    print(f"prune: {best}", flush=True)
    assert best[262_144] < 8.0 * best[65_536]
