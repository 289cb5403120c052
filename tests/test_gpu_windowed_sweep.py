"""The windowed sweep and score against the CPU oracle at the edges of its shapes: a candidate per
wavefront and per block, 64 / 128 / 256 instance slots, windows around the 64-, 256- and
1024-request batches, placements whose instances are all alike, all different, or out of the tables,
deadlines beyond what the 32-bit tick sums take, and both sides of the longest short window."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

import oracle  # noqa: E402
from paper_2509_06362_amd import binding, workloads as W  # noqa: E402

WEIGHTS = (4.0, 0.3, 2048.0, 1.0)


@pytest.mark.parametrize("n_cand,i_pad,window,n_req,variant", [
    (1030, 3, 255, 600, "mixed"), (1030, 65, 256, 520, "mixed"), (1025, 129, 257, 300, "mixed"),
    (1027, 64, 64, 130, "alike"), (1, 64, 63, 400, "mixed"), (3, 65, 1023, 2500, "different"),
    (2, 256, 1024, 3000, "different"), (5, 128, 1025, 2100, "alike"), (4, 200, 300, 1000, "long"),
    (1024, 20, 256, 513, "long"), (6, 33, 40, 500, "bad"), (1031, 9, 100, 350, "bad"),
    (4100, 2, 5000, 300, "mixed"),
    # the longest windows in which a candidate's lanes are its instances, and one request more
    (33, 32, 8, 210, "mixed"), (33, 32, 9, 210, "different"), (30, 33, 16, 210, "different"),
    (30, 33, 17, 210, "mixed"), (9, 256, 16, 150, "long"), (9, 256, 17, 150, "mixed"),
])
def test_windowed_sweep_edges(n_cand, i_pad, window, n_req, variant):
    w = W.random_small(n_cand * 7 + i_pad, n_cand, i_pad, n_req, n_slo=3, b_cap=64, pen_kappa=0.5)
    if variant == "alike":
        one = lambda x: np.ascontiguousarray(np.broadcast_to(x[:, :1], x.shape))
        w = W.replace(w, tp_idx=one(w.tp_idx), max_batch=one(w.max_batch), occ=np.zeros_like(w.occ),
                      q_ticks=np.zeros_like(w.q_ticks), n_inst=np.full_like(w.n_inst, i_pad))
    elif variant == "different":  # longer queues on the stronger instances: few are dominated
        q = (w.tp_idx.astype(np.uint64) * np.uint64(1 << 19) + w.max_batch.astype(np.uint64) * np.uint64(4099))
        w = W.replace(w, q_ticks=q, occ=np.zeros_like(w.occ), n_inst=np.full_like(w.n_inst, i_pad))
    elif variant == "long":
        w = W.replace(w, d_ttft=w.d_ttft * np.float32(1000.0),
                      q_ticks=w.q_ticks * np.uint64(300), prompt_len=w.prompt_len * np.uint32(700))
    ref_w = w
    if variant == "bad":
        # slots outside the tables are absent: as good as instances nobody can ever be admitted to
        tp, B, q = w.tp_idx.copy(), w.max_batch.copy(), w.q_ticks.copy()
        q[:, [0, i_pad // 2]] = np.uint64(1 << 50)
        ref_w = W.replace(w, q_ticks=q)
        tp[:, 0] = 9
        B[:, i_pad // 2] = 65
        w = W.replace(w, tp_idx=tp, max_batch=B)
    for policy in (0, 1):
        wp = W.replace(w, policy=policy)
        print(f"windowed sweep C={n_cand} I={i_pad} window={window} R={n_req} {variant} policy={policy}", flush=True)
        dw = binding.DeviceWorkload(wp)
        try:
            cnt, _, best = dw.sweep(window=window)
            sc = dw.score(*WEIGHTS, window=window)
            torch.cuda.synchronize()
            ref = oracle.placement_score(W.replace(ref_w, policy=policy), *WEIGHTS, window=window)
            assert np.array_equal(cnt.cpu().numpy().view(np.uint32), ref["sat_count"])
            assert int(best.item()) == int(np.argmax(ref["sat_count"]))
            for k in ("sat_count", "phi_s", "phi_t", "phi_l", "score"):
                got = sc[k].cpu().numpy()
                assert np.array_equal(got.view(np.uint32) if k == "sat_count" else got, ref[k]), k
            assert binding.maaso_ctx_device_status(dw.ctx) == (2 if variant == "bad" else 0)
        finally:
            dw.close()


@pytest.mark.parametrize("i_pad,window,n_windows,variant", [
    (9, 300, 60, "alike"), (64, 257, 48, "mixed"), (128, 500, 48, "different"), (256, 700, 40, "different"),
    (33, 1024, 30, "alike"), (100, 1025, 24, "different"), (256, 1500, 24, "mixed"),
])
def test_wavefronts_that_share_a_candidate_stay_alike(i_pad, window, n_windows, variant):
    """Few candidates and windows of more than 256 requests: four wavefronts per candidate, one request a lane
    below 1024 and four from there on.  Dozens of windows in bursts: over all slots windows with one to several
    instances to choose among, over two slots windows in which nobody can be admitted next to others."""
    n_req = window * n_windows - window // 3
    w = W.random_small(i_pad + n_windows, 3, i_pad, n_req, n_slo=3, b_cap=64, pen_kappa=0.5)
    n_inst = np.array([i_pad, 2, i_pad // 2 + 1], np.uint32)
    burst = np.arange(n_req) // (6 * window)
    # within a burst 64 ticks from one request to the next; then half a minute in which the queues empty
    ticks = np.arange(n_req, dtype=np.uint64) * 64 + burst.astype(np.uint64) * (30 << 20)
    w = W.replace(w, n_inst=n_inst, arrival_ticks=ticks.astype(np.uint32), occ=np.zeros_like(w.occ))
    if variant == "alike":
        w = W.replace(w, tp_idx=np.full_like(w.tp_idx, 1), max_batch=np.full_like(w.max_batch, 16),
                      q_ticks=np.zeros_like(w.q_ticks))
    elif variant == "different":  # longer queues on the stronger instances: few are dominated
        q = w.tp_idx.astype(np.uint64) * np.uint64(1 << 19) + w.max_batch.astype(np.uint64) * np.uint64(4099)
        w = W.replace(w, q_ticks=q)
    if variant != "alike":
        w = W.replace(w, d_ttft=w.d_ttft * np.float32(0.1))
    chosen = [0, 0]  # windows by the instances that are chosen: two or more of all slots, none of two slots
    for c in (0, 1):
        run = oracle.score_assign(w, cand=c, window=window)
        for lo in range(0, n_req, window):
            of = run["chosen"][lo:lo + window][run["slack"][lo:lo + window] >= 0]
            chosen[c] += len(np.unique(of)) >= 2 if c == 0 else len(of) == 0
    assert (variant == "alike" or chosen[0] >= 3) and 2 <= chosen[1] <= n_windows - 2, chosen
    for policy in (0, 1):
        check_against_oracle(W.replace(w, policy=policy), window, f"shared candidate windows={n_windows} {variant}")


def check_against_oracle(w, window, what, status=0, ref_w=None):
    print(f"{what} C={w.n_cand} I={w.i_pad} R={w.n_req} window={window} policy={w.policy}", flush=True)
    dw = binding.DeviceWorkload(w)
    try:
        cnt, _, best = dw.sweep(window=window)
        sc = dw.score(*WEIGHTS, window=window)
        torch.cuda.synchronize()
        ref = oracle.placement_score(w if ref_w is None else ref_w, *WEIGHTS, window=window)
        assert np.array_equal(cnt.cpu().numpy().view(np.uint32), ref["sat_count"])
        assert int(best.item()) == int(np.argmax(ref["sat_count"]))
        for k in ("sat_count", "phi_s", "phi_t", "phi_l", "score"):
            got = sc[k].cpu().numpy()
            assert np.array_equal(got.view(np.uint32) if k == "sat_count" else got, ref[k]), k
        assert binding.maaso_ctx_device_status(dw.ctx) == status
    finally:
        dw.close()


@pytest.mark.parametrize("n_cand,i_pad,window,n_req,policy,variant", [
    # one lane a request and several, passes that end inside and at a window, instances that do not fill a trip
    (3, 1, 5, 61, 0, "mixed"), (4, 2, 6, 90, 0, "mixed"), (2, 17, 9, 200, 0, "mixed"), (3, 16, 16, 160, 0, "bad"),
    (2, 64, 17, 300, 0, "mixed"), (2, 255, 64, 700, 0, "mixed"), (3, 256, 65, 800, 0, "mixed"), (5, 33, 128, 1000, 0, "bad"),
    (2, 128, 129, 900, 0, "long"), (4, 5, 255, 1100, 0, "long"), (3, 70, 256, 1300, 0, "mixed"), (3, 70, 257, 1300, 0, "mixed"),
    (6, 40, 9000, 200, 0, "mixed"), (2, 64, 4, 210, 0, "mixed"),
    # the largest numbers of candidates and slots that are taken this way at windows of 256, 128, 64 and 32, and one more
    (768, 4, 512, 600, 0, "mixed"), (768, 4, 513, 600, 0, "mixed"), (8, 9, 256, 600, 0, "mixed"), (8, 9, 257, 600, 0, "mixed"),
    (769, 4, 70, 150, 0, "mixed"), (4, 65, 128, 300, 0, "mixed"),
    (4, 65, 129, 300, 0, "mixed"), (1024, 13, 128, 150, 0, "mixed"), (1024, 12, 65, 150, 0, "mixed"), (1025, 13, 64, 140, 0, "mixed"),
    (1536, 3, 7, 40, 0, "mixed"), (1536, 3, 6, 40, 0, "mixed"), (1537, 13, 32, 70, 0, "mixed"), (1537, 12, 32, 70, 0, "mixed"),
    (2560, 13, 9, 40, 0, "mixed"), (2561, 13, 9, 40, 0, "mixed"),
    # shortest queue
    (3, 1, 1, 40, 1, "mixed"), (2, 20, 3, 150, 1, "mixed"), (2, 8, 256, 530, 1, "bad"), (2, 9, 129, 530, 1, "mixed"),
    (2, 32, 128, 330, 1, "mixed"), (2, 33, 64, 330, 1, "bad"), (2, 33, 65, 330, 1, "mixed"), (3, 256, 7, 200, 1, "long"),
    (769, 5, 32, 70, 1, "mixed"), (769, 5, 33, 70, 1, "mixed"), (1280, 3, 16, 70, 1, "mixed"), (1281, 3, 16, 70, 1, "mixed"),
])
def test_block_per_candidate_edges(n_cand, i_pad, window, n_req, policy, variant):
    w = W.random_small(n_cand * 5 + i_pad + window, n_cand, i_pad, n_req, n_slo=3, b_cap=64, pen_kappa=0.5)
    w = W.replace(w, policy=policy)
    ref_w, status = w, 0
    if variant == "long":     # ticks beyond 32 bits
        w = ref_w = W.replace(w, d_ttft=w.d_ttft * np.float32(1000.0), q_ticks=w.q_ticks * np.uint64(300),
                              prompt_len=w.prompt_len * np.uint32(700))
    elif variant == "bad":    # absent slots: as good as instances nobody can ever be admitted to
        tp, q = w.tp_idx.copy(), w.q_ticks.copy()
        w = W.replace(w, n_inst=np.full_like(w.n_inst, i_pad))
        tp[:, i_pad // 2] = 9
        q[:, i_pad // 2] = np.uint64(1 << 50)
        ref_w, w, status = W.replace(w, q_ticks=q), W.replace(w, tp_idx=tp), 2
    check_against_oracle(w, window, f"block per candidate {variant}", status, ref_w)


@pytest.mark.parametrize("n_cand,i_pad,window,n_req", [
    (1540, 20, 40, 200), (1540, 70, 100, 450), (1540, 128, 150, 400), (1540, 256, 200, 450), (5, 256, 1100, 4000),
])
def test_windows_that_load_many_instances(n_cand, i_pad, window, n_req):
    """Instances of which none is better than another in everything, and tight deadlines: more than a few stay in a
    window and take requests, with a wavefront and with a block per candidate."""
    w = W.random_small(n_cand + i_pad, n_cand, i_pad, n_req, n_slo=3, b_cap=64, pen_kappa=0.5)
    order = np.argsort(np.argsort(w.tp_idx, axis=1, kind="stable"), axis=1).astype(np.uint64)
    w = W.replace(w, tbt_mode=1, n_inst=np.full_like(w.n_inst, i_pad), occ=np.zeros_like(w.occ), q_ticks=order * np.uint64(2000),
                  max_batch=(64 - (order * np.uint64(60)) // np.uint64(i_pad)).astype(np.uint16),
                  d_ttft=w.d_ttft * np.float32(0.1))
    run = oracle.score_assign(w, cand=0, window=window)
    first = run["chosen"][:window][run["slack"][:window] >= 0]
    assert len(np.unique(first)) > 4
    for policy in (0, 1):
        check_against_oracle(W.replace(w, policy=policy), window, "many instances")


@pytest.mark.parametrize("n_cand,i_pad,window,variant", [
    (2600, 129, 24, "mixed"), (2600, 129, 25, "mixed"), (2565, 128, 17, "different"), (2565, 9, 8, "mixed"),
])
def test_longest_short_windows_of_many_candidates(n_cand, i_pad, window, variant):
    w = W.random_small(n_cand + i_pad, n_cand, i_pad, 3 * window + 5, n_slo=3, b_cap=64, pen_kappa=0.5)
    if variant == "different":
        q = w.tp_idx.astype(np.uint64) * np.uint64(1 << 19) + w.max_batch.astype(np.uint64) * np.uint64(4099)
        w = W.replace(w, q_ticks=q, occ=np.zeros_like(w.occ), n_inst=np.full_like(w.n_inst, i_pad))
    check_against_oracle(w, window, f"short windows {variant}")


@pytest.mark.parametrize("n_cand,i_pad,window,n_req", [
    (1024, 12, 512, 600), (1024, 12, 513, 600), (769, 66, 288, 350), (769, 66, 289, 350), (1449, 5, 1025, 1100),
    (1448, 5, 1025, 1100), (4095, 3, 8190, 8300), (4096, 3, 8300, 8300),
])
def test_one_wavefront_per_candidate_or_four(n_cand, i_pad, window, n_req):
    """Both sides of the line between the two, which runs with the square of the number of candidates.  A first-token deadline of ten
    minutes keeps the requests from being laid out, whatever the shape."""
    w = W.random_small(n_cand + i_pad, n_cand, i_pad, n_req, n_slo=3, b_cap=64, pen_kappa=0.5)
    w = W.replace(w, d_ttft=np.where(w.d_ttft == w.d_ttft.max(), 600.0, w.d_ttft).astype(np.float32))
    check_against_oracle(w, window, "one wavefront or four")
