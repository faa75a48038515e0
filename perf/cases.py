"""Performance cases of the library: the calls a user's program makes in every
iteration of Algorithm 2, over the range of sizes, worker counts, compressors
and roles the library serves.

A case names a role (`op`):
  step     one whole iteration for all M workers on one GPU (step_fused);
  noalloc  the same from a descriptor, without a plan's scratch
           (step_fused_noalloc: graph capture, serving loops);
  worker   what one worker process runs in an iteration around the network
           exchange: compress_ef, then omd_step with the server's average;
  server   what the server process runs: the average of the M messages;
  codec    a message built from a caller's own codes and decoded again:
           pack (quantizers), then unpack.
and the compressor (`kind`, `levels`, `norm`, `k`), the parameters per worker
d, the workers M and the layers (segments) of the model.

Inputs are gradient-shaped: every layer has its own scale, drawn log-uniformly
over three decades, and the error residuals have the size of one step's
gradients.
"""
import math
import random

import numpy as np
import torch

from paper_2010_13359_amd import dqgan

ETA = 2e-4
T = 7                    # iteration number (a counter word of the rounding generator)
QUANT_SEED = 3 | (2 << 32)

# parameter counts per layer: the 2-512-512-512-1 MLP of generator and of
# discriminator, and DCGAN 64x64 (deconvolutions / convolutions and batch norm)
MLP = [1536, 262656, 262656, 513] * 2
DCGAN = [820224, 2097664, 524544, 131200, 3072, 3072, 131328, 524800, 2098176, 8192]
D_MLP, D_DCGAN, D_RESNET, D_LARGE = sum(MLP), sum(DCGAN), 33_554_432, 100_000_000


def listed():
    return [
        # the smallest model, sign compressor: launches and host work count
        dict(name="tiny_sign_step", op="step", kind="sign", norm="l1", levels=0, k=0, d=65536, M=4, layers=1),
        # an MLP GAN on eight workers, one scale per network: data stays in the caches
        dict(name="mlp_sign_step", op="step", kind="sign", norm="l1", levels=0, k=0, d=D_MLP, M=8, layers=2),
        # the same model with the sparse compressor at 1 %
        dict(name="mlp_topk_step", op="step", kind="topk", norm="none", levels=0, k=D_MLP // 100, d=D_MLP, M=8,
             layers=8),
        # the paper's experiment: DCGAN, 8-bit codes with the max-norm scale
        dict(name="dcgan_mbit8_step", op="step", kind="mbit", norm="linf", levels=8, k=0, d=D_DCGAN, M=16, layers=10),
        # the largest dense workload of the benchmark: ResNet WGAN-GP, 32 workers, 4-bit levels
        dict(name="resnet_qsgd15_step", op="step", kind="qsgd", norm="l2", levels=15, k=0, d=D_RESNET, M=32,
             layers=64),
        # a large generator, 1 % of 10^8 entries per worker
        dict(name="large_topk_step", op="step", kind="topk", norm="none", levels=0, k=D_LARGE // 100, d=D_LARGE, M=16,
             layers=256),
        # many workers (above the counts the paper ran): the MLP on 256
        dict(name="many_workers_step", op="step", kind="qsgd", norm="l2", levels=255, k=0, d=D_MLP, M=256, layers=8),
        # a ragged size from a loop that must not allocate
        dict(name="ragged_noalloc_step", op="noalloc", kind="qsgd", norm="linf", levels=255, k=0, d=1_000_003, M=5,
             layers=3),
        # one worker process of a ResNet run
        dict(name="worker_qsgd255", op="worker", kind="qsgd", norm="l2", levels=255, k=0, d=D_RESNET, M=1, layers=64),
        # the server process of a ResNet run with 32 workers
        dict(name="server_qsgd15", op="server", kind="qsgd", norm="l2", levels=15, k=0, d=D_RESNET, M=32, layers=64),
        # the server process of the large sparse run
        dict(name="server_topk", op="server", kind="topk", norm="none", levels=0, k=D_LARGE // 100, d=D_LARGE, M=16,
             layers=256),
        # a caller's own 8-bit codes to messages and back, odd length
        dict(name="codec_mbit8", op="codec", kind="mbit", norm="linf", levels=8, k=0, d=D_DCGAN + 1, M=16, layers=10),
    ]


KINDS = [("sign", "l1", 0), ("qsgd", "l2", 255), ("qsgd", "l2", 15), ("qsgd", "linf", 255), ("qsgd", "linf", 15),
         ("mbit", "linf", 8), ("mbit", "linf", 4), ("mbit", "l2", 8), ("topk", "none", 0), ("topk", "none", 0),
         ("identity", "none", 0)]


def draw(rng):
    op = rng.choice(["step", "step", "step", "step", "noalloc", "worker", "server", "codec"])
    kind, norm, levels = rng.choice(KINDS)
    if op == "noalloc" and kind == "topk":
        op = "step"
    d = int(math.exp(rng.uniform(math.log(5e4), math.log(6e7)))) | rng.choice([0, 1])
    # workers: mostly the counts of the paper's study, now and then many
    most = max(1, min(32 if rng.random() < 0.8 else 512, 800_000_000 // d))
    M = 1 if op == "worker" else int(round(math.exp(rng.uniform(0.0, math.log(most)))))
    layers = rng.randint(1, 64)
    if op == "noalloc":  # the fixed scratch: 12 bytes per (worker, piece of 16384)
        M = max(1, min(M, int(6e6 / (12.0 * (d / 16384 + layers)))))
    k = max(1, int(d * math.exp(rng.uniform(math.log(1e-3), math.log(5e-2))))) if kind == "topk" else 0
    return dict(op=op, kind=kind, norm=norm, levels=levels, k=k, d=d, M=M, layers=layers)


# ---------------------------------------------------------------------------
# inputs


def _ld(case):
    return (case["d"] + 1023) // 1024 * 1024


def _offsets(case):
    """Layer boundaries: the named models' own, else log-uniform sizes (ratio
    up to 1000) that depend on the case alone."""
    d, n = case["d"], case["layers"]
    if n == 2 and d == D_MLP:
        return [0, D_MLP // 2, D_MLP]
    if n == len(MLP) and d == D_MLP:
        sizes = MLP
    elif n == len(DCGAN) and abs(d - D_DCGAN) <= 1:
        sizes = DCGAN[:-1] + [DCGAN[-1] + d - D_DCGAN]
    else:
        r = random.Random(1000 * n + d)
        w = [math.exp(r.uniform(0.0, math.log(1000.0))) for _ in range(n)]
        cuts = [int(d * x) for x in np.cumsum(w) / sum(w)]
        return sorted({0, d} | {c for c in cuts if 0 < c < d})
    return [int(x) for x in np.cumsum([0] + sizes)]


def _gen(seed, salt):
    g = torch.Generator(device="cuda")
    g.manual_seed(1_000_003 * seed + salt)
    return g


def _layer_scale(case):
    """Per-element gradient scale, one value per layer."""
    off = _offsets(case)
    r = random.Random(77 + case["layers"])
    s = torch.tensor([math.exp(r.uniform(math.log(1e-4), math.log(1e-1))) for _ in off[1:]], device="cuda")
    n = torch.tensor([b - a for a, b in zip(off, off[1:])], device="cuda")
    return torch.repeat_interleave(s, n)


def _rows(case, seed, salt, mult):
    """[M][ld] normal rows times the layer scales and `mult`, zero padding."""
    d = case["d"]
    x = torch.zeros((case["M"], _ld(case)), dtype=torch.float32, device="cuda")
    sv = _layer_scale(case) * mult
    g = _gen(seed, salt)
    for m in range(case["M"]):
        x[m, :d].normal_(generator=g).mul_(sv)
    return x


def _vector(case, seed, salt, std):
    v = torch.zeros(_ld(case), dtype=torch.float32, device="cuda")
    v[:case["d"]].normal_(0.0, std, generator=_gen(seed, salt))
    return v


def _top(case):
    """The quantizer's largest level."""
    return (1 << (case["levels"] - 1)) - 1 if case["kind"] == "mbit" else case["levels"]


def _codes(case, seed):
    """[M][ld] uint16 codes (bit 15 the sign, the level below it), most levels
    small as those of gradients are, and the scales per (worker, layer)."""
    M, d, s = case["M"], case["d"], _top(case)
    codes = torch.zeros((M, _ld(case)), dtype=torch.int16, device="cuda")
    g = _gen(seed, 11)
    for m in range(M):
        u = torch.rand(d, generator=g, device="cuda")
        lev = (u.pow_(4).mul_(s + 1)).to(torch.int16).clamp_(max=s) if case["kind"] != "sign" else 0
        neg = torch.rand(d, generator=g, device="cuda") < 0.5
        codes[m, :d] = torch.where(neg, torch.tensor(-32768, dtype=torch.int16, device="cuda"), 0) + lev
    n_seg = len(_offsets(case)) - 1
    scales = torch.empty((M, n_seg), device="cuda").log_normal_(-5.0, 1.0, generator=g)
    return codes, scales


def _index_lists(case, seed):
    """[M][k] ascending distinct indices and their values: each worker's k
    entries, spread over the layers by their gradient scales (a layer with
    larger gradients keeps more of its entries, at most nine tenths)."""
    M, d, k = case["M"], case["d"], case["k"]
    off = _offsets(case)
    r = random.Random(77 + case["layers"])
    s = [math.exp(r.uniform(math.log(1e-4), math.log(1e-1))) for _ in off[1:]]
    n = [b - a for a, b in zip(off, off[1:])]
    lo, hi = 0.0, 10.0   # the common threshold: sum of n * erfc(t / (s sqrt 2)) = k
    for _ in range(60):
        mid = 0.5 * (lo + hi)
        lo, hi = (mid, hi) if sum(c * math.erfc(mid / (x * 1.4142135)) for c, x in zip(n, s)) > k else (lo, mid)
    want = [min(c, int(0.9 * c), int(c * math.erfc(hi / (x * 1.4142135)))) for c, x in zip(n, s)]
    for j in sorted(range(len(n)), key=lambda j: -s[j]):   # what rounding left over
        more = min(k - sum(want), n[j] - want[j])
        want[j] += max(0, more)
    # entry q of a layer that keeps c of its n: one index in [q n / c, (q + 1) n / c)
    parts = [(torch.arange(c, device="cuda", dtype=torch.float64) * (w / c) + a, w / c)
             for a, w, c in zip(off, n, want) if c]
    base = torch.cat([p for p, _ in parts])
    width = torch.cat([torch.full_like(p, x) for p, x in parts])
    sv = _layer_scale(case)
    idx = torch.empty((M, k), dtype=torch.int32, device="cuda")
    val = torch.empty((M, k), dtype=torch.float32, device="cuda")
    g = _gen(seed, 12)
    for m in range(M):
        u = torch.rand(k, generator=g, device="cuda", dtype=torch.float64)
        # ceil keeps below the stratum's end, so indices stay distinct
        i = torch.ceil(base + 0.999999 * u * (width - 1.0)).to(torch.int64)
        idx[m] = i.to(torch.int32)
        val[m].normal_(generator=g).mul_(sv[i]).mul_(ETA)
    return idx, val


def _inputs(case, seed):
    """The tensors a program holds before the call, from the seed alone."""
    op, x = case["op"], {}
    if op in ("step", "noalloc", "worker"):
        x["G"] = _rows(case, seed, 1, 1.0)
        x["E"] = _rows(case, seed, 2, ETA)
        x["W"] = _vector(case, seed, 3, 0.02)
    if op == "worker":
        x["Q"] = _vector(case, seed, 4, 1e-5)
    if op in ("server", "codec"):
        if case["kind"] == "topk":
            x["idx"], x["val"] = _index_lists(case, seed)
        elif case["kind"] == "identity":
            x["val"] = _rows(case, seed, 5, ETA)
        else:
            x["codes"], x["scales"] = _codes(case, seed)
    return x


def prepare(case, seed):
    s = _inputs(case, seed)
    M, ld = case["M"], _ld(case)
    plan = dqgan.Plan(case["d"], M, case["kind"], seg_offsets=_offsets(case) if case["kind"] not in ("topk", "identity")
                      else None, norm=case["norm"], levels=case["levels"], k=case["k"], seed=QUANT_SEED)
    s.update(op=case["op"], kind=case["kind"], plan=plan, wire=plan.new_wire("cuda"))
    if case["op"] in ("step", "noalloc", "worker"):
        s["WX"] = torch.zeros((M, ld), dtype=torch.float32, device="cuda")
    if case["op"] in ("server", "codec"):
        if case["kind"] in ("topk", "identity"):
            s["wire"].val, s["wire"].idx = s["val"].view(-1), s["idx"].view(-1) if "idx" in s else None
        elif case["op"] == "server":
            dqgan.pack(plan, s["codes"], s["scales"], s["wire"])
            del s["codes"]
        s["out"] = torch.zeros((M, ld) if case["op"] == "codec" else ld, dtype=torch.float32, device="cuda")
    return s


def _message(wire):
    planes = {"sign": wire.sign, "level": wire.level, "scale": wire.scale, "val": wire.val, "idx": wire.idx}
    return {k: v for k, v in planes.items() if v is not None}


def run(s):
    op, plan, wire = s["op"], s["plan"], s["wire"]
    if op == "step":
        dqgan.step_fused(plan, ETA, T, s["G"], s["E"], s["W"], s["WX"], wire)
        return {"E": s["E"], "W": s["W"], "WX": s["WX"], **_message(wire)}
    if op == "noalloc":
        dqgan.step_fused_noalloc(plan, ETA, T, s["G"], s["E"], s["W"], s["WX"], wire)
        return {"E": s["E"], "W": s["W"], "WX": s["WX"], **_message(wire)}
    if op == "worker":
        dqgan.compress_ef(plan, ETA, T, s["G"], s["E"], None, wire)
        dqgan.omd_step(plan, ETA, s["Q"], s["W"], s["G"], s["E"], s["WX"])
        return {"E": s["E"], "W": s["W"], "WX": s["WX"], **_message(wire)}
    if op == "server":
        dqgan.aggregate(plan, wire, s["out"])
        return {"out": s["out"]}
    if s["kind"] in ("topk", "identity"):
        dqgan.unpack(plan, wire, s["out"])
        return {"out": s["out"]}
    dqgan.pack(plan, s["codes"], s["scales"], wire)
    dqgan.unpack(plan, wire, s["out"])
    return {"out": s["out"], **_message(wire)}


# ---------------------------------------------------------------------------
# what a pass cannot do without


def _message_bytes(case):
    """Bytes of one worker's message."""
    bits = {"sign": 1, "qsgd": 1 + (8 if case["levels"] == 255 else 4), "mbit": case["levels"], "identity": 32}
    if case["kind"] == "topk":
        return 8 * case["k"]
    return case["d"] * bits[case["kind"]] / 8 + 4 * (len(_offsets(case)) - 1)


def work(case):
    d, M, op = case["d"], case["M"], case["op"]
    msg = M * _message_bytes(case)
    if op in ("step", "noalloc"):      # g, e read; e, evaluation points written; w read and written
        return {"bytes": 16.0 * M * d + msg + 8.0 * d, "flops": 9.0 * M * d + 2.0 * d}
    if op == "worker":                 # ... and g, e read again after the exchange, with w and the average
        return {"bytes": 24.0 * M * d + msg + 12.0 * d, "flops": 11.0 * M * d + d}
    if op == "server":
        return {"bytes": msg + 4.0 * d, "flops": 2.0 * M * (case["k"] if case["kind"] == "topk" else d) + d}
    if case["kind"] in ("topk", "identity"):
        return {"bytes": msg + 4.0 * M * d, "flops": 0.0}
    return {"bytes": 2.0 * M * d + 2.0 * msg + 4.0 * M * d, "flops": 1.0 * M * d}


def tolerance(case):
    """Every operation has its rounding and every sum its order in the
    library's contract, so outputs are the same; only the layers' mean and
    Euclidean norms are sums of 64 bits in an order left open, which may round
    to the neighbouring 32-bit scale."""
    if case["op"] in ("step", "noalloc", "worker") and case["norm"] in ("l1", "l2"):
        return {"rel": 1e-5, "differ": 1e-6}
    return "exact"


# ---------------------------------------------------------------------------
# The same in 64 bits.  Decisions (which level, which entries) are those of
# the 32-bit definition; every value around them is computed in 64 bits.


def _philox(blocks, m, t):
    """The four words of Philox4x32-10 (Salmon et al. 2011) for each counter
    (lo32(block), m, t, hi32(block)), as 64-bit integers."""
    mask = 0xFFFFFFFF
    c = [blocks & mask, torch.full_like(blocks, m), torch.full_like(blocks, t), blocks >> 32]
    k0, k1 = QUANT_SEED & mask, QUANT_SEED >> 32
    for _ in range(10):
        a, b = c[0] * 0xD2511F53, c[2] * 0xCD9E8D57
        c = [((b >> 32) & mask) ^ c[1] ^ k0, b & mask, ((a >> 32) & mask) ^ c[3] ^ k1, a & mask]
        k0, k1 = (k0 + 0x9E3779B9) & mask, (k1 + 0xBB67AE85) & mask
    return c


def _encode(case, m, p32, p, off, counts):
    """p-hat of one row and the row's scales in 64 bits; p32 is p as the
    32-bit definition rounds it, which decides signs and levels."""
    kind, d = case["kind"], case["d"]
    if kind == "identity":
        return p, None
    seg = [p[a:b] for a, b in zip(off, off[1:])]
    if kind == "sign":
        sc = torch.stack([x.abs().mean() for x in seg])
        return torch.where(p32.signbit(), -1.0, 1.0) * torch.repeat_interleave(sc, counts), sc
    s = _top(case)
    norm = (lambda x: x.norm()) if case["norm"] == "l2" else (lambda x: x.abs().max())
    sc = torch.stack([norm(x) for x in seg])
    sc32 = torch.stack([norm(x) for x in p32.double().split(counts.tolist())]).float()
    ratio = torch.repeat_interleave((s / sc32.double()).float(), counts)
    words = _philox(torch.arange((d + 3) // 4, device="cuda"), m, T)
    u = (torch.stack(words, 1).view(-1)[:d] >> 8).float() * 2.0 ** -24
    r = p32.abs() * ratio
    low = r.floor().clamp_(max=float(s))
    level = (low + (u < torch.where(low == s, 0.0, r - low))).clamp_(max=float(s)).double()
    return torch.copysign(level * torch.repeat_interleave(sc / s, counts), p32.double()), sc


def _exact_rows(case, seed):
    x = _inputs(case, seed)
    M, d, off = case["M"], case["d"], _offsets(case)
    counts = torch.tensor([b - a for a, b in zip(off, off[1:])], device="cuda")
    G, E = x["G"], x["E"].double()
    total = torch.zeros(d, dtype=torch.float64, device="cuda")
    scale, val = [], []
    for m in range(M):
        p32 = G[m, :d] * np.float32(ETA).item() + E[m, :d].float()      # two roundings, as the definition has
        p = G[m, :d].double() * np.float32(ETA).item() + E[m, :d]
        if case["kind"] == "topk":
            key = p32.abs()
            least = torch.topk(key, case["k"], sorted=True).values[-1]
            pick = key > least
            ties = (key == least).nonzero().view(-1)[: case["k"] - int(pick.sum())]
            pick[ties] = True
            hat, sc = torch.where(pick, p, 0.0), None
            val.append(p[pick])
        else:
            hat, sc = _encode(case, m, p32, p, off, counts)
        if sc is not None:
            scale.append(sc)
        if case["kind"] == "identity":
            val.append(torch.nn.functional.pad(p, (0, _ld(case) - d)))
        total += hat
        E[m, :d] = p - hat
    W = x["W"].double()
    W[:d] -= x["Q"][:d].double() if case["op"] == "worker" else total / M
    WX = torch.zeros_like(E)
    for m in range(M):
        WX[m, :d] = W[:d] - (G[m, :d].double() * np.float32(ETA).item() + E[m, :d])
    return {"E": E, "W": W, "WX": WX, "scale": torch.stack(scale).view(-1) if scale else None,
            "val": torch.cat(val) if val else None}


def _exact_messages(case, seed):
    x = _inputs(case, seed)
    M, d, ld, off = case["M"], case["d"], _ld(case), _offsets(case)
    out = torch.zeros((M, ld) if case["op"] == "codec" else ld, dtype=torch.float64, device="cuda")
    counts = torch.tensor([b - a for a, b in zip(off, off[1:])], device="cuda")
    for m in range(M):
        if case["kind"] == "topk":
            hat = torch.zeros(d, dtype=torch.float64, device="cuda")
            hat[x["idx"][m].long()] = x["val"][m].double()
        elif case["kind"] == "identity":
            hat = x["val"][m, :d].double()
        else:
            c = x["codes"][m, :d].long() & 0xFFFF
            mag = torch.repeat_interleave(x["scales"][m].double(), counts)
            if case["kind"] != "sign":
                mag = mag * (c & 0x7FFF).double() / _top(case)
            hat = torch.where(c >= 0x8000, -mag, mag)
        if case["op"] == "codec":
            out[m, :d] = hat
        else:
            out[:d] += hat / M
    return {"out": out, "scale": x["scales"].double().view(-1) if case["op"] == "codec" and "scales" in x else None}


def exact(case, seed):
    if case["op"] in ("server", "codec"):
        return _exact_messages(case, seed)
    return _exact_rows(case, seed)
