"""The static sweep against the triple oracle at the edges of its grouping and of its thresholds: around
4096 requests (grouped by every block or by launches of their own, or compared with every threshold), around the 1024 requests a grouping
block takes, all lengths alike, empty prompts, lengths no binary32 holds exactly, one class and
sixteen, rows of slots that do and do not fill 16 lanes, and profiles whose quotient is far off."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

import oracle  # noqa: E402
from paper_2509_06362_amd import binding, workloads as W  # noqa: E402


def check(w):
    dw = binding.DeviceWorkload(w)
    try:
        ref = oracle.placement_sweep(w)
        per_class = np.bincount(w.slo_class, minlength=w.n_slo).astype(np.int64)
        pairs = sum(int((oracle.stage(w, c)["tbt"][:, None] <= w.d_tbt[None]).astype(np.int64).sum(0) @ per_class)
                    for c in range(w.n_cand))
        for noalloc in (False, True, False):   # the accumulators are left as they were found
            cnt, ratio, best = dw.sweep(noalloc=noalloc)
            torch.cuda.synchronize()
            assert np.array_equal(cnt.cpu().numpy().view(np.uint32), ref["sat_count"])
            assert np.array_equal(ratio.cpu().numpy(), ref["sat_ratio"])
            assert int(best.cpu().numpy().view(np.uint32)[0]) == ref["best_cand"]
            assert binding.maaso_ctx_sweep_evaluated(dw.ctx) == pairs
        assert binding.maaso_ctx_device_status(dw.ctx) == 0
        return ref["sat_count"]
    finally:
        dw.close()


@pytest.mark.parametrize("n_cand,i_pad,n_req,n_slo", [
    (1, 1, 1, 1), (3, 16, 4096, 1), (70, 7, 4097, 3), (1100, 3, 1025, 2), (5, 255, 5120, 16),
    (9, 256, 5121, 3), (1, 64, 9000, 16), (40, 33, 4095, 8), (2100, 32, 4100, 3),
    # compared with every threshold (up to 128 candidates of 512 slots together), or grouped
    (128, 4, 5000, 16), (129, 3, 5000, 16), (2, 256, 4097, 5), (3, 171, 4097, 5), (37, 13, 20481, 1),
    # thresholds beside the grouping or behind it: either side of 512 candidates and of 65,536 requests, rows of slots
    # that fill 16 lanes and not, several groups of candidates a block, more blocks than deliver at once, and (the last)
    # thresholds that the no-allocation scratch has no room for
    (511, 20, 4100, 16), (512, 20, 4100, 16), (512, 16, 4097, 2), (140, 48, 65535, 2), (140, 48, 65536, 2), (129, 5, 70001, 3),
    (5000, 1, 4097, 16), (1900, 255, 4099, 1), (140_000, 1, 4200, 16),
])
def test_static_sweep_edges(n_cand, i_pad, n_req, n_slo):
    w = W.random_small(n_cand + 3 * i_pad + n_req, n_cand, i_pad, n_req, n_slo=n_slo, b_cap=64, pen_kappa=0.5)
    w = W.stressed(w, seed=n_req)
    print(f"static sweep C={n_cand} I={i_pad} R={n_req} K={n_slo}", flush=True)
    check(w)


@pytest.mark.parametrize("lengths", ["alike", "empty", "steps", "long", "beyond"])
@pytest.mark.parametrize("n_req,i_pad", [(1500, 20), (6000, 20), (6000, 8)])
def test_static_sweep_lengths(lengths, n_req, i_pad):
    w = W.stressed(W.random_small(n_req + len(lengths), 60, i_pad, n_req, n_slo=3, b_cap=32), seed=5)
    rng = np.random.default_rng(n_req)
    if lengths == "alike":
        L = np.full(n_req, 1777)
    elif lengths == "empty":
        L = np.where(rng.random(n_req) < 0.5, 0, rng.integers(0, 3, n_req))
    elif lengths == "steps":    # around the bins' edges
        L = (1 << rng.integers(0, 14, n_req)) * rng.integers(8, 17, n_req) // 8 + rng.integers(-1, 2, n_req)
        L = np.maximum(L, 0)
    elif lengths == "long":
        L = rng.integers(0, 1 << 24, n_req)
    else:                       # more than binary32 holds exactly
        L = rng.integers(1 << 24, (1 << 32) - 1, n_req)
        L[:3] = (1 << 32) - 1, (1 << 24) + 1, 1 << 31
    w = W.replace(w, prompt_len=L.astype(np.uint32))
    if lengths in ("long", "beyond"):  # deadlines such lengths can meet
        w = W.replace(w, d_ttft=(w.d_ttft * np.float32(400.0 if lengths == "long" else 2e5)))
    cnt = check(w)
    if lengths != "empty":
        assert len(np.unique(cnt)) > 1


@pytest.mark.parametrize("a_scale,p_scale,d_scale", [
    (1.0, 1e-9, 1.0), (1.0, 1e6, 1.0), (1e-6, 1e-7, 1e-3), (40.0, 1e-4, 1.0), (1.0, 1.0, 4000.0), (1e-30, 1e-30, 1.0),
])
@pytest.mark.parametrize("n_cand", [50, 20])
def test_static_sweep_extreme_profiles(a_scale, p_scale, d_scale, n_cand):
    w = W.random_small(17, n_cand, 24, 5000, n_slo=3, b_cap=32)
    rng = np.random.default_rng(3)
    w = W.replace(w, prefill_a=(w.prefill_a * np.float32(a_scale)), prefill_p=(w.prefill_p * np.float32(p_scale)),
                  d_ttft=(w.d_ttft * np.float32(d_scale)),
                  prompt_len=np.floor(np.exp(rng.uniform(0, np.log(2.0 ** 24), 5000))).astype(np.uint32))
    print(f"static sweep a*{a_scale} p*{p_scale} D*{d_scale}", flush=True)
    check(w)


@pytest.mark.parametrize("n_cand,i_pad,n_req,n_slo", [
    # every number of bins a class can have: 128 (two classes) down to 16 (sixteen), in one launch and in three
    (40, 12, 900, 2), (30, 9, 2000, 3), (25, 7, 3000, 7), (20, 20, 4096, 16), (150, 5, 5000, 2), (60, 33, 7000, 5),
    (140, 12, 9000, 16), (70, 40, 30000, 9), (200, 3, 50000, 16),
    # and all 256 where the look-ups would get too many
    (2100, 6, 70000, 2),
    # compared with every threshold: as many candidates as can be and one more; five trips of slots and six, which
    # are grouped; one trip of sixteen classes' thresholds and two
    (128, 4, 16384, 1), (129, 4, 16384, 1), (5, 256, 20000, 1), (6, 256, 20000, 1), (40, 40, 500000, 3), (8, 32, 6000, 16),
    (9, 32, 6000, 16),
])
def test_static_sweep_groups(n_cand, i_pad, n_req, n_slo):
    w = W.random_small(2 * n_cand + i_pad + n_req, n_cand, i_pad, n_req, n_slo=n_slo, b_cap=64, pen_kappa=0.5)
    print(f"static sweep groups C={n_cand} I={i_pad} R={n_req} K={n_slo}", flush=True)
    check(W.stressed(w, seed=n_slo))
