"""dqgan_pack, dqgan_unpack and dqgan_aggregate over worker counts at the edges
of their row batches and layers that put one, a few or many segments in a
1024-column tile, against the message's definition in numpy binary32."""
import numpy as np
import pytest

from gpu_common import assert_same, to_dev

pytestmark = pytest.mark.gpu

LAYOUTS = {"one": [0, 3001], "few": [0, 5, 1020, 1024, 1030, 2900, 3001],
           "many": [0] + list(range(1, 400, 7)) + list(range(1024, 1300, 3)) + [3001],
           "exact": [0, 1024, 2048]}
KINDS = [("sign", "l1", 0), ("qsgd", "l2", 15), ("qsgd", "l2", 255), ("mbit", "linf", 8), ("mbit", "linf", 4)]


def _expect(kind, levels, codes, scales, offs):
    """[M][d] decoded values in binary32, one rounding per operation."""
    f32 = np.float32
    counts = np.diff(offs)
    sc = np.repeat(scales, counts, axis=1)
    neg = (codes >> 15) != 0
    if kind == "sign":
        mag = sc
    else:
        top = f32((1 << (levels - 1)) - 1 if kind == "mbit" else levels)
        tiny = sc < f32(2.0 ** -64)
        b = (sc * np.where(tiny, f32(2.0 ** 64), f32(1))) / top
        mag = ((codes & 0x7FFF).astype(f32) * b) * np.where(tiny, f32(2.0 ** -64), f32(1))
    return np.where(neg, -mag, mag).astype(f32)


@pytest.mark.parametrize("layout", sorted(LAYOUTS))
@pytest.mark.parametrize("kind,norm,levels", KINDS)
@pytest.mark.parametrize("M", [1, 3, 4, 7, 9, 65])
def test_messages(kind, norm, levels, layout, M):
    import torch
    from paper_2010_13359_amd import dqgan
    offs = LAYOUTS[layout]
    d = offs[-1]
    print("case", kind, levels, layout, "M", M, flush=True)
    rng = np.random.default_rng(M)
    top = (1 << (levels - 1)) - 1 if kind == "mbit" else levels
    ld = (d + 1023) // 1024 * 1024
    codes = (rng.integers(0, top + 1, (M, ld)) | (rng.integers(0, 2, (M, ld)) << 15)).astype(np.uint16)
    scales = rng.lognormal(-5.0, 1.0, (M, len(offs) - 1)).astype(np.float32)
    scales[0, 0] = 0.0
    scales[-1, -1] = 1e-25          # below 2^-64: the scaled constants
    plan = dqgan.Plan(d, M, kind, seg_offsets=offs, norm=norm, levels=levels, seed=1)
    wire = plan.new_wire("cuda")
    P = torch.full((M, ld), float("nan"), device="cuda")
    Q = torch.full((ld,), float("nan"), device="cuda")
    dqgan.pack(plan, to_dev(codes.view(np.int16)), to_dev(scales), wire)
    dqgan.unpack(plan, wire, P)
    dqgan.aggregate(plan, wire, Q)
    torch.cuda.synchronize()
    exp = _expect(kind, levels, codes[:, :d], scales, offs)
    assert_same("scale", wire.scale.cpu().numpy(), scales.ravel())
    got = P.cpu().numpy()
    assert np.array_equal(got[:, :d].view(np.uint32), exp.view(np.uint32)) and np.all(got[:, d:] == 0)
    total = exp[0].copy()
    for m in range(1, M):
        total = total + exp[m]
    mean = (total.astype(np.float64) / M).astype(np.float32)
    got = Q.cpu().numpy()
    assert np.array_equal(got[:d].view(np.uint32), mean.view(np.uint32)) and np.all(got[d:] == 0)
    plan.close()


@pytest.mark.parametrize("kind,norm,levels", KINDS)
@pytest.mark.parametrize("M", [4, 6, 16])
def test_average_by_segments_per_tile(kind, norm, levels, M):
    """The server average on both sides of the segments per tile up to which
    each segment is summed in a pass of its own (4 to 12, by messages and
    workers), next to a tile of one segment."""
    import torch
    from paper_2010_13359_amd import dqgan
    rng = np.random.default_rng(M)
    top = (1 << (levels - 1)) - 1 if kind == "mbit" else levels
    d, ld = 2047, 2048
    for n in range(3, 15):
        print("case", kind, levels, "M", M, "segments", n, flush=True)
        offs = [1024 * j // n for j in range(n)] + [1024, d]
        codes = (rng.integers(0, top + 1, (M, ld)) | (rng.integers(0, 2, (M, ld)) << 15)).astype(np.uint16)
        scales = rng.lognormal(-5.0, 1.0, (M, len(offs) - 1)).astype(np.float32)
        scales[0, 1] = 0.0
        scales[-1, 2] = 1e-25       # below 2^-64: the scaled constants
        plan = dqgan.Plan(d, M, kind, seg_offsets=offs, norm=norm, levels=levels, seed=1)
        wire = plan.new_wire("cuda")
        Q = torch.full((ld,), float("nan"), device="cuda")
        dqgan.pack(plan, to_dev(codes.view(np.int16)), to_dev(scales), wire)
        dqgan.aggregate(plan, wire, Q)
        torch.cuda.synchronize()
        exp = _expect(kind, levels, codes[:, :d], scales, offs)
        total = exp[0].copy()
        for m in range(1, M):
            total = total + exp[m]
        mean = (total.astype(np.float64) / M).astype(np.float32)
        got = Q.cpu().numpy()
        assert np.array_equal(got[:d].view(np.uint32), mean.view(np.uint32)) and np.all(got[d:] == 0)
        plan.close()
