"""Top-k selection on both sides of the row length at which one workgroup per
row stops searching alone (8192 tiles of 256), over key distributions that
take each branch: a Gaussian row, entries piled up in a narrow range of keys
(the second digit of the band, many candidates in one bin), heavy ties and
zero rows (the full-row search, with and without its index digits), more than
k large entries that no sampled run meets (the keys above the band are k or
more: the search hands the row over), and a dense band that overflows a wave's
staging.  Two iterations, so that the histograms and counters that must be
zero between iterations are; everything against the oracle."""
import numpy as np
import pytest

from gpu_common import GpuState, compare_step, inputs
from synth.configs import custom

pytestmark = pytest.mark.gpu

SHORT, LONG = 8192 * 256, 8192 * 256 + 1024
SIZES = {"d511": 511, "d513": 513, "d66000": 66000, "short_edge": SHORT - 3, "long_edge": LONG - 1021,
         "long": 2_300_007}
KINDS = ["gauss", "piled", "ties", "zeros", "cluster", "band", "equal"]


RUN = 64  # elements of a sampled run


def _sample_stride(w):
    """Elements from one sampled run of a row to the next: 512 runs at most in
    the short rows, 4096 in longer ones."""
    short = w.ld // 256 <= 8192
    most = 512 if short else 4096
    return max(512 if short else 2048, (-(-w.d // most) + RUN - 1) // RUN * RUN)


def _band_misses(w, x):
    """Whether k or more keys of a row lie above the band that its sample gives."""
    at = np.arange(w.d) % _sample_stride(w) < RUN
    ns, f = int(at.sum()), w.k / w.d
    upper = int(np.floor(f * ns - 8.0 * (np.sqrt(ns * f * (1.0 - f)) + 1.0)))  # + 1: the rank of the upper end
    if upper < 1:
        return False  # the band is open
    hi = np.sort(np.abs(x[at]))[::-1][upper]
    return int((np.abs(x) > hi * np.float32(1.0 + 2.0 ** -17)).sum()) >= w.k


def _gradients(kind, w):
    rng = np.random.default_rng(len(kind) + w.d % 1000)
    n = (w.M, w.d)
    x = rng.standard_normal(n, dtype=np.float32)
    if kind == "piled":          # 3 % of the entries within 1e-4 of one value, k of them above all others
        at = rng.random(n) < 0.03
        x = np.where(at, (8.0 + 1e-4 * x).astype(np.float32), 0.1 * x)
    if kind == "ties":
        x = rng.choice(np.array([0.5, -0.5, 1.0, -0.25], np.float32), size=n)
    if kind == "zeros":
        x[0] = 0.0
        x[1, :: 7] = 0.0
        x[1, w.k // 2:] = 0.0    # fewer than k entries that are not zero
    if kind == "cluster":        # more than k large entries, all between the sampled runs
        away = np.flatnonzero(np.arange(w.d) % _sample_stride(w) >= RUN)
        x[:, rng.choice(away, min(len(away), w.k + w.k // 4 + 1), replace=False)] *= 1000.0
    if kind == "band":           # a run of entries just around the k-th largest
        a, b = w.d // 4, w.d // 4 + max(1, w.k // 2)
        x *= 1e-3
        big = rng.permutation(w.d)[: max(1, int(0.75 * w.k))]
        x[:, big] = 10.0 + 0.1 * rng.standard_normal((w.M, len(big)), dtype=np.float32)
        x[:, a:b] = 1.0 + 1e-4 * rng.standard_normal((w.M, b - a), dtype=np.float32)
    if kind == "equal":
        x[:] = np.where(rng.random(n) < 0.5, np.float32(-2.0), np.float32(2.0))
    return x


@pytest.mark.parametrize("kind", KINDS)
@pytest.mark.parametrize("size", sorted(SIZES))
def test_topk_rows(size, kind):
    from oracle import oracle as orc
    d = SIZES[size]
    w = custom(d=d, M=2, kind="topk", k=max(1, d // 50), eta=1.0, seed=3)
    print("case", size, kind, "k", w.k, flush=True)
    G, E, W = inputs(w)
    G[:, :d] = _gradients(kind, w)
    E[:] = 0.0
    if kind == "cluster" and d > 1000:  # (the shortest rows' bands are open)
        assert all(_band_misses(w, G[m, :d]) for m in range(w.M))
    s = GpuState(w, G, E, W)
    E_r, W_r = E.copy(), W.copy()
    for t in (1, 2):
        s.fused(t)
        ref = orc.step(w.as_dict(), np.float32(w.eta), t, G, E_r, W_r)
        compare_step(w, s.host(), ref)
        E_r, W_r = ref["E"], ref["W"]
    s.close()


@pytest.mark.parametrize("d", [66_000, 300_003, LONG - 1021])
def test_rows_that_fall_back_together(d):
    """One search over rows that fall back and rows that do not, decided by
    different digits (ties need the index digits, a zero row has no key above
    the k-th), in units of one to several tiles per wave."""
    from oracle import oracle as orc
    kinds = ["gauss", "ties", "zero", "equal", "sparse", "ties", "gauss"]
    w = custom(d=d, M=len(kinds), kind="topk", k=d // 50, eta=1.0, seed=5)
    print("case", d, "k", w.k, flush=True)
    G, E, W = inputs(w)
    rng = np.random.default_rng(d)
    for m, kind in enumerate(kinds):
        x = rng.standard_normal(d, dtype=np.float32)
        if kind == "ties":
            x = rng.choice(np.array([0.5, -0.5, 1.0, -0.25], np.float32), size=d)
        if kind == "zero":
            x[:] = 0.0
        if kind == "equal":
            x[:] = np.where(rng.random(d) < 0.5, np.float32(-2.0), np.float32(2.0))
        if kind == "sparse":
            x[rng.random(d) > 0.004] = 0.0
        G[m, :d] = x
    E[:] = 0.0
    s = GpuState(w, G, E, W)
    E_r, W_r = E.copy(), W.copy()
    for t in (1, 2):
        s.fused(t)
        ref = orc.step(w.as_dict(), np.float32(w.eta), t, G, E_r, W_r)
        compare_step(w, s.host(), ref)
        E_r, W_r = ref["E"], ref["W"]
    s.close()
