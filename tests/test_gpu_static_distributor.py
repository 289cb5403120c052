"""The static distributor against the CPU oracle where a request is compared with lists of instances:
lists that end inside and at a trip of four records, placements whose instances are all alike or all
listed, requests nothing can serve (their list is another one, or the same where nearly all are listed), both selection rules, block counts on
both sides of one accumulator line each, aligned arrays and not."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

import oracle  # noqa: E402
from paper_2509_06362_amd import binding, workloads as W  # noqa: E402


@pytest.mark.parametrize("i_pad,n_req,variant", [
    (9, 1000, "mixed"), (64, 32768, "mixed"), (64, 32769, "mixed"), (256, 33000, "different"),
    (65, 40001, "alike"), (128, 2051, "different"), (200, 36000, "blocked"), (33, 5, "blocked"),
    (16, 70000, "bad"), (256, 3000, "different blocked"), (70, 3001, "different blocked"),
    # listed with one, two and four slots per lane; and few slots with a second group of requests for a part of the
    # threads, where nothing is listed, next to one group, two, and one slot more
    (63, 700, "different"), (65, 700, "different blocked"), (128, 900, "mixed"), (129, 900, "different"), (12, 300, "blocked"),
    (9, 2_097_152, "different"), (9, 2_097_160, "blocked"), (16, 2_100_003, "different blocked"), (17, 2_100_000, "different"),
    (10, 4_194_309, "mixed"),
])
def test_static_distributor_lists(i_pad, n_req, variant):
    few = min(n_req, 100_003)   # (the generator's arrivals end at 2^32 ticks: more requests repeat these)
    w = W.random_small(i_pad + n_req, 1, i_pad, few, n_slo=3, b_cap=64, pen_kappa=0.5)
    if n_req != few:
        w = W.replace(w, arrival_ticks=None, **{k: np.resize(getattr(w, k), n_req) for k in ("prompt_len", "out_len", "slo_class")})
    w = W.replace(w, n_inst=np.full(1, i_pad, np.uint32))
    if variant == "alike":
        w = W.replace(w, tp_idx=np.full_like(w.tp_idx, 2), max_batch=np.full_like(w.max_batch, 8),
                      occ=np.zeros_like(w.occ), q_ticks=np.zeros_like(w.q_ticks))
    elif variant.startswith("different"):   # nobody dominates: the stronger the instance, the longer its queue
        order = np.argsort(w.tp_idx[0], kind="stable")
        q = np.empty(i_pad, np.uint64)
        q[order] = np.arange(i_pad, dtype=np.uint64) * np.uint64(1500)
        w = W.replace(w, q_ticks=q[None], occ=np.zeros_like(w.occ),
                      max_batch=(1 + np.argsort(np.argsort(-q.astype(np.int64))) % 64).astype(np.uint16)[None])
    if variant.endswith("blocked"):     # most requests cannot be served by anyone
        w = W.replace(w, d_ttft=w.d_ttft * np.float32(0.02), d_tbt=w.d_tbt * np.float32(0.3))
    elif variant == "bad":
        w = W.replace(w, tp_idx=np.where(np.arange(i_pad) % 3 == 0, 9, w.tp_idx).astype(np.uint8))
    for policy in (0, 1):
        wp = W.replace(w, policy=policy)
        ref = None
        if variant != "bad":
            ref = oracle.score_assign(wp, window=0)
        else:                      # absent slots: as good as instances that can never win
            q = np.where(np.arange(i_pad) % 3 == 0, np.uint64(1 << 62), w.q_ticks).astype(np.uint64)
            tp = np.where(np.arange(i_pad) % 3 == 0, 0, w.tp_idx).astype(np.uint8)
            ref = oracle.score_assign(W.replace(wp, q_ticks=q, tp_idx=tp), window=0)
        for latencies in (False, True):
            print(f"static distributor I={i_pad} R={n_req} {variant} policy={policy} latencies={latencies}", flush=True)
            dw = binding.DeviceWorkload(wp)
            try:
                for _ in range(2):   # the accumulators are left as they were found
                    got = dw.assign(window=0, latencies=latencies)
                    torch.cuda.synchronize()
                    assert np.array_equal(got["chosen"].cpu().numpy(), ref["chosen"])
                    assert np.array_equal(got["slack"].cpu().numpy(), ref["slack"])
                    assert int(got["n_satisfied"].item()) == ref["n_satisfied"]
                    if latencies:
                        for k in ("ttft", "tbt", "e2e"):
                            assert np.array_equal(got[k].cpu().numpy(), ref[k], equal_nan=True), k
                assert binding.maaso_ctx_device_status(dw.ctx) == (2 if variant == "bad" else 0)
            finally:
                dw.close()
