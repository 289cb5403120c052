"""Windows laid out by class and prompt length, against the CPU oracle: sizes around the batches (16 and 64
requests), the groups of 256 and the segments of 4096 requests, empty and single classes, ties on the between-token margin, and prefills
beyond eight seconds."""
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


# candidates enough for the laid-out form (1000 and more; fewer with windows of 2048 and 4096)
@pytest.mark.parametrize("n_cand,i_pad,n_slo,window,n_req,variant", [
    (1001, 3, 3, 257, 600, "mixed"), (1000, 2, 1, 300, 901, "alike"), (1003, 5, 16, 320, 700, "mixed"),
    (1000, 4, 8, 384, 800, "alike"), (1000, 4, 8, 385, 800, "mixed"),           # 32 batches of 16, and one group more
    (1002, 3, 3, 464, 930, "long"), (1002, 3, 3, 465, 940, "one class"), (1000, 3, 2, 512, 1024, "zeros"),
    (1000, 70, 3, 500, 700, "mixed"), (1000, 130, 3, 300, 400, "alike"),        # two and four slots a lane
    (400, 3, 3, 2048, 4100, "one length"), (64, 5, 5, 4095, 8190, "mixed"), (64, 4, 3, 4096, 8193, "long"),
    (65, 4, 16, 4097, 9000, "zeros"), (64, 140, 3, 8200, 8300, "alike"), (4100, 2, 3, 256, 300, "mixed"),
    (1000, 3, 3, 5000, 300, "mixed"),                                           # one window, shorter than its size
])
def test_sweep_and_score(n_cand, i_pad, n_slo, window, n_req, variant):
    w = variant_of(W.random_small(n_cand + 31 * i_pad + window, n_cand, i_pad, n_req, n_slo=n_slo, b_cap=64, pen_kappa=0.5,
                                  jitter=variant != "alike"), variant)
    for policy in (0, 1):
        wp = W.replace(w, policy=policy)
        print(f"laid out C={n_cand} I={i_pad} K={n_slo} window={window} R={n_req} {variant} policy={policy}", flush=True)
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


def test_captured_sweep_keeps_off_the_workspace():
    """A windowed sweep captured in a graph replays beside other calls of the context, which use its workspace."""
    w = W.random_small(33, 1200, 6, 1200, b_cap=32)
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
