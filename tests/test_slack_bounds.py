"""The bounds by which a batch of requests is settled from its shortest and longest prompt (ordered_windows.hpp), in
binary32 as the kernels compute them: no request's slack is above min(s1, s2) at the shortest prompt or below
min(s1 - c, s2) at the longest, c = 2^-20 De / Dt of the longest output."""
import numpy as np
import pytest

F = np.float32


def fma(a, b, c):
    """binary32 fma; the product is exact in binary64 and so, to one rounding in 2^29, is the result."""
    return (a.astype(np.float64) * b.astype(np.float64) + c.astype(np.float64)).astype(F)


@pytest.mark.parametrize("seed", range(6))
def test_slack_stays_within_the_batch_bounds(seed):
    rng = np.random.default_rng(seed)
    n, m = 20_000, 16
    u = lambda lo, hi: np.exp(rng.uniform(np.log(lo), np.log(hi), size=(n, 1))).astype(F)
    Dt, Db = u(0.05, 400.0), u(0.002, 0.5)
    iDt, iDb = (1.0 / Dt.astype(np.float64)).astype(F), (1.0 / Db.astype(np.float64)).astype(F)
    a, p = u(1e-4, 0.1), u(1e-7, 1e-3)
    L = np.floor(np.exp(rng.uniform(0.0, 9.0, size=(n, m)))).astype(F)
    S = np.floor(np.exp(rng.uniform(-1.0, 10.5, size=(n, m)))).astype(F)
    lo, hi, most = L.min(1, keepdims=True), L.max(1, keepdims=True), S.max(1, keepdims=True)
    # margins of all sizes, and many batches where the two are equal but for a few units in the last place
    tbt = (Db * (F(1) - (rng.random((n, 1)) ** 3).astype(F))).astype(F)
    near = (Dt.astype(np.float64) * tbt / Db - a - p.astype(np.float64) * rng.choice([0.0, 1.0, 0.5], size=(n, 1)) * hi)
    wait = np.where(rng.random((n, 1)) < 0.5, near * (1.0 + rng.integers(-4, 5, size=(n, 1)) * 2.0 ** -23),
                    Dt * rng.random((n, 1))).astype(F)
    wait = np.maximum(wait, F(0))

    def margins(x):
        ttft = wait + fma(p, x, a)
        return ttft, (Dt - ttft) * iDt, (Db - tbt) * iDb

    ttft, s1, s2 = margins(L)
    De = fma(S, Db, Dt)
    s3 = (De - fma(S, tbt, ttft)) * (F(1) / De)
    slack = np.minimum(np.minimum(s1, s2), s3)
    _, s1_hi, s2_hi = margins(hi)
    _, s1_lo, _ = margins(lo)
    clear = F(2.0 ** -20) * (fma(most, Db, Dt) * iDt)
    up, low = np.minimum(s1_lo, s2_hi), np.minimum(s1_hi - clear, s2_hi)
    assert (slack <= up).all()
    used = (low >= 0)[:, 0]  # a batch is settled by this bound only where it is not negative
    assert used.sum() > n // 8
    assert (slack >= low)[used].all()
    # exact on the between-token margin
    on = used & (low == s2_hi)[:, 0] & (up == s2_hi)[:, 0]
    assert on.sum() > n // 50 and (slack[on] == s2_hi[on]).all()
