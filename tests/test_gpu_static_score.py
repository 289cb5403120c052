"""The static composite score (window 0: one window over all requests, no arrivals at hand) of few requests,
around the longest windows in which a candidate's lanes are its instances: alone, over request sets, and
inside Alg. 2, against the CPU oracle."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

import oracle  # noqa: E402
from paper_2509_06362_amd import binding, workloads as W  # noqa: E402

WEIGHTS = (4.0, 0.3, 2048.0, 1.0)
KEYS = ("sat_count", "phi_s", "phi_t", "phi_l", "score")


def same(out, ref):
    for k in KEYS:
        got = out[k].cpu().numpy()
        assert np.array_equal(got.view(np.uint32) if k == "sat_count" else got, ref[k]), k
    assert int(out["best_cand"].item()) == ref["best_cand"]


@pytest.mark.parametrize("policy", [0, 1])
@pytest.mark.parametrize("i_pad", [32, 33, 64, 128, 256])
@pytest.mark.parametrize("n_req", [1, 2, 8, 9, 16, 17])
def test_static_score_without_arrivals(n_req, i_pad, policy):
    w = W.random_small(n_req * 31 + i_pad, 7, i_pad, n_req, n_slo=3, b_cap=64, pen_kappa=0.5)
    w = W.replace(w, arrival_ticks=None, policy=policy)
    print(f"static score C=7 I={i_pad} R={n_req} policy={policy}", flush=True)
    dw = binding.DeviceWorkload(w)
    try:
        assert dw.arrival_ticks is None
        out = dw.score(*WEIGHTS, window=0)
        half = n_req // 2
        ranges = [(0, n_req), (0, half), (half, n_req)]
        outs = dw.score_sets(ranges, *WEIGHTS, window=0)
        torch.cuda.synchronize()
        same(out, oracle.placement_score(w, *WEIGHTS, window=0))
        for (lo, hi), o in zip(ranges, outs):
            same(o, oracle.placement_score(w.with_requests(lo, hi), *WEIGHTS, window=0))
        assert binding.maaso_ctx_device_status(dw.ctx) == 0
    finally:
        dw.close()


@pytest.mark.parametrize("n_req,n_gpus", [(2, 8), (8, 24), (9, 24), (16, 64), (17, 64)])
def test_static_partition_without_arrivals(n_req, n_gpus):
    w = W.partition_case(n_req=n_req, rate=300.0, seed=61, tight_share=0.5)
    tp, b = W.all_configs(batch_set=[4, 16])
    cw, offs = W.growth_chains(w, tp, b, n_gpus)
    cw = W.replace(cw, arrival_ticks=None)
    print(f"static partition R={n_req} G={n_gpus} C={cw.n_cand} I={cw.i_pad}", flush=True)
    r_t, r_l = oracle.split_by_slo(w, 0b1)
    ref = {tag: oracle.placement_score(W.replace(cw, prompt_len=ws.prompt_len, out_len=ws.out_len,
                                                 slo_class=ws.slo_class), *WEIGHTS, window=0)["score"]
           for tag, ws in (("t", r_t), ("l", r_l), ("h", w))}
    dw = binding.DeviceWorkload(cw)
    try:
        got = dw.resource_partition(offs, 0b1, n_gpus, *WEIGHTS, window=0)
        torch.cuda.synchronize()
        assert int(got["n_tight"].item()) == r_t.n_req
        for tag in ("t", "l", "h"):
            assert np.array_equal(got[f"score_{tag}"].cpu().numpy(), ref[tag]), tag
        assert binding.maaso_ctx_device_status(dw.ctx) == 0
    finally:
        dw.close()
