"""The rule by which the windowed sweep leaves instances out of a window (live_slots.hpp,
find_admissible), restated in numpy binary32 and compared with scoring every instance: every request
that any instance can serve is given the same instance, under both selection rules, over records that
differ by nothing, by a few units in the last place, around the rule's margins, and freely."""
import numpy as np
import pytest

F = np.float32


def fma(a, b, c):
    """binary32 fma: the product of two binary32 numbers is exact in binary64, and the sum is rounded
    to odd there before the last rounding, so that the result is rounded once."""
    p = a.astype(np.float64) * b.astype(np.float64)
    c = c.astype(np.float64)
    s = p + c
    bb = s - p
    err = (p - (s - bb)) + (c - bb)
    bits = s.view(np.int64)
    odd = (bits & 1) == 0
    away = np.where((err > 0) == (s > 0), 1, -1)
    s = np.where((err != 0) & odd & np.isfinite(s), (bits + np.where(away > 0, 1, -1)).view(np.float64), s)
    return s.astype(F)


def slacks(a, p, tbt, wait, L, S, Dt, Db):
    L, S, Dt, Db = (x[:, None] for x in (L, S, Dt, Db))
    n = a.shape[0]
    up = lambda x: np.broadcast_to(x, (L.shape[0], n))
    iDt, iDb = (1.0 / Dt.astype(np.float64)).astype(F), (1.0 / Db.astype(np.float64)).astype(F)
    De = fma(S, Db, Dt)
    iDe = F(1.0) / De
    ttft = up(wait) + fma(up(p), up(L), up(a))
    e2e = fma(up(S), up(tbt), ttft)
    return np.fmin(np.fmin((Dt - ttft) * iDt, up((Db - tbt[None]) * iDb)), (De - e2e) * iDe)


def admissible(a, p, tbt, wait, occ, d_ttft, d_tbt, shortest_queue):
    n = a.shape[0]
    e_t, e_b = d_ttft.max() * F(2.0 ** -20), d_tbt.max() * F(2.0 ** -20)
    keep = (tbt <= d_tbt.max()) & ~(wait + a > d_ttft.max())
    j = np.arange(n)
    steps = 0
    for k in range(n):
        if not keep[k] or steps == 16:
            continue
        steps += 1
        ap = (a[k] <= a) & (p[k] <= p)
        le = ap & (tbt[k] <= tbt) & (wait[k] <= wait)
        if shortest_queue:
            gone = le & ((occ[k] < occ) | ((occ[k] == occ) & (j > k)))
        else:
            gone = (le & (j > k)) | (ap & (tbt[k] + e_b <= tbt) & (wait[k] + e_t <= wait))
        keep &= ~gone
    return keep


def pick(sl, occ, shortest_queue, among):
    order = np.lexsort((np.arange(len(occ)), occ))
    rank = np.empty(len(occ), np.float64)
    rank[order] = 512.0 - np.arange(len(occ))
    val = sl.astype(np.float64)
    if shortest_queue:
        val = np.where(sl >= 0, rank[None], val)
    val = np.where(among[None], val, -np.inf)
    return val.argmax(axis=1), val.max(axis=1) >= 0


@pytest.mark.parametrize("spread", ["equal", "ulps", "margins", "free", "long"])
@pytest.mark.parametrize("shortest_queue", [False, True])
def test_the_set_holds_every_admitted_requests_instance(spread, shortest_queue):
    rng = np.random.default_rng(sum(map(ord, spread)) + shortest_queue)
    dropped = total = served = 0
    for _ in range(150):
        n, R = int(rng.integers(1, 40)), 400
        k = int(rng.integers(1, 5))
        d_ttft = np.sort(rng.uniform(0.05, 60.0, k)).astype(F)
        d_tbt = np.sort(rng.uniform(0.02, 0.3, k)).astype(F)
        strat = rng.integers(0, 3, n)
        a, p = np.array([.02, .011, .006], F)[strat], np.array([4e-5, 2.2e-5, 1.2e-5], F)[strat]
        base_t, base_w = F(rng.uniform(0.2, 0.9)) * d_tbt[-1], F(rng.uniform(0, 0.8)) * d_ttft[-1]
        if spread == "equal":
            tbt, wait = np.full(n, base_t), np.full(n, base_w)
        elif spread == "ulps":
            tbt = (np.full(n, base_t).view(np.int32) + rng.integers(-3, 4, n).astype(np.int32)).view(F)
            wait = (np.full(n, base_w).view(np.int32) + rng.integers(-3, 4, n).astype(np.int32)).view(F)
        elif spread == "margins":  # multiples of about half the rule's margins
            tbt = (base_t + rng.integers(0, 6, n) * (d_tbt.max() * 2.0 ** -21)).astype(F)
            wait = (base_w + rng.integers(0, 6, n) * (d_ttft.max() * 2.0 ** -21)).astype(F)
        else:
            tbt = (rng.uniform(0.1, 1.2, n) * d_tbt[-1]).astype(F)
            wait = np.where(rng.random(n) < 0.2, 0, rng.uniform(0, 1.2, n) * d_ttft[-1]).astype(F)
            wait[rng.random(n) < 0.05] = np.inf
        occ = rng.integers(0, 4, n).astype(np.int32)
        hi = 2.0 ** 24 if spread == "long" else 16384.0
        L, S = (np.floor(np.exp(rng.uniform(0, np.log(hi), R))).astype(F) for _ in range(2))
        c = rng.integers(0, k, R)
        with np.errstate(invalid="ignore"):
            sl = slacks(a, p, tbt, wait, L, S, d_ttft[c], d_tbt[c])
        keep = admissible(a, p, tbt, wait, occ, d_ttft, d_tbt, shortest_queue)
        all_j, all_adm = pick(sl, occ, shortest_queue, np.ones(n, bool))
        set_j, set_adm = pick(sl, occ, shortest_queue, keep)
        assert np.array_equal(all_adm, set_adm)
        assert np.array_equal(all_j[all_adm], set_j[all_adm])
        dropped += int((~keep).sum())
        total += n
        served += int(all_adm.sum())
    assert served > 1000
    assert dropped > total // 4   # the rule does take instances out
