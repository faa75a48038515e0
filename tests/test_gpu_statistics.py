"""The statistics pass and the worker's encoder over pieces that start off a
quad, segments of one, a few and more pieces than the pass combines by itself,
and worker counts on both sides of the encoder's row batches: three iterations
on one plan against the oracle, as one fused call, without a plan and as the
worker's own call."""
import numpy as np
import pytest

from gpu_common import GpuState, assert_same, compare_step, inputs, to_dev
from synth.configs import custom

pytestmark = pytest.mark.gpu

P = 16380  # elements of a piece in a small workload
LAYOUTS = {
    "one piece": [0, 1, 3001, 5126],
    "off a quad": [0, 3, 3 + P, 6 + 3 * P, 7 + 3 * P, 70001],
    "sixteen pieces": [0, 5, 5 + 16 * P],
    "seventeen pieces": [0, 5, 5 + 16 * P + 1],
    "two waves of pieces": [0, 66 * P],
}
KINDS = {"sign": dict(kind="sign"), "qsgd15": dict(kind="qsgd", levels=15),
         "mbit8": dict(kind="mbit", levels=8, norm="linf")}


@pytest.mark.parametrize("M", [1, 3, 4, 5])
@pytest.mark.parametrize("kind", sorted(KINDS))
@pytest.mark.parametrize("layout", sorted(LAYOUTS))
def test_statistics_and_encoder(layout, kind, M):
    import torch
    from oracle import oracle as orc
    from paper_2010_13359_amd import dqgan
    offs = LAYOUTS[layout]
    w = custom(d=offs[-1], M=M, eta=1e-2, seed=M, seg_offsets=offs, **KINDS[kind])
    G, E, W = inputs(w, t=1)
    s, n, c = (GpuState(w, G, E, W) for _ in range(3))
    print("case", layout, kind, "M", M, flush=True)
    for t in (1, 2, 3):
        s.fused(t)
        dqgan.step_fused_noalloc(n.plan, w.eta, t, n.G, n.E, n.W, n.WX, n.wire, n.Q)
        dqgan.compress_ef(c.plan, w.eta, t, c.G, c.E, None, c.wire)
        torch.cuda.synchronize()
        gpu, noalloc, worker = s.host(), n.host(), c.host()
        own = orc.step(w.as_dict(), np.float32(w.eta), t, G, E.copy(), W.copy())
        # binary64 sums in another order, rounded once: at most the neighbouring binary32 value
        np.testing.assert_allclose(gpu["scale"], own["scale"], rtol=2.0 ** -23, atol=0)
        ref = orc.step(w.as_dict(), np.float32(w.eta), t, G, E.copy(), W.copy(), scales_in=gpu["scale"])
        compare_step(w, gpu, ref)
        compare_step(w, noalloc, ref)
        for plane in ("scale", "sign", "level", "E"):
            if plane in gpu:
                assert_same(plane + " of the worker", worker[plane], gpu[plane])
        E, W = gpu["E"], gpu["W"]
    for x in (s, n, c):
        x.close()
