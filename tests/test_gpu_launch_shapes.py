"""The fused step over worker counts at the edges of its launch shapes (one
wave per R rows, only the waves that own a row are launched) and segment
boundaries inside, at and between the 256-column workgroups, against the
oracle with the library's own scales."""
import numpy as np
import pytest

from gpu_common import GpuState, compare_step, inputs
from synth.configs import custom

pytestmark = pytest.mark.gpu

SEGS = [0, 255, 257, 768, 1024, 1500]
KINDS = {"sign": dict(kind="sign", seg_offsets=SEGS), "qsgd15": dict(kind="qsgd", levels=15, seg_offsets=SEGS),
         "mbit8": dict(kind="mbit", levels=8, norm="linf", seg_offsets=SEGS), "topk": dict(kind="topk", k=37),
         "identity": dict(kind="identity")}


@pytest.mark.parametrize("kind", sorted(KINDS))
@pytest.mark.parametrize("M", [1, 2, 3, 5, 7, 9, 15, 17, 29, 33, 63, 65, 127, 129, 193, 256, 257])
def test_fused_step_worker_counts(kind, M):
    from oracle import oracle as orc
    w = custom(d=1500, M=M, eta=1e-2, seed=M, **KINDS[kind])
    G, E, W = inputs(w, t=2)
    print("case", kind, "M", M, flush=True)
    s = GpuState(w, G, E, W)
    s.fused(2)
    gpu = s.host()
    s.close()
    scales = gpu.get("scale")
    if scales is not None:
        own = orc.step(w.as_dict(), np.float32(w.eta), 2, G, E.copy(), W.copy())
        np.testing.assert_allclose(scales, own["scale"], rtol=1e-5, atol=0)
    ref = orc.step(w.as_dict(), np.float32(w.eta), 2, G, E.copy(), W.copy(), scales_in=scales)
    compare_step(w, gpu, ref)
