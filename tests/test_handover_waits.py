"""The hand-overs between workgroups of the top-k kernels, in the assembly that
the compiler makes of them (no GPU needed).

A workgroup publishes its results by one thread's release fence and an atomic
arrival, after a barrier.  The fence's own wait covers the operations of the
wave that executes it; the other waves' stores and atomics are covered only if
each of them waits for its own (s_waitcnt vmcnt(0)) before it enters that
barrier.  Checked by data flow: on no path through a kernel may a wave enter a
barrier that a release fence follows with a store or atomic that it has not
waited for.
"""
import re
import subprocess

import pytest

from paper_2010_13359_amd import build

# kernels that hand over inside one launch, and how many of their instances
KERNELS = {"k_topk_sample": 1, "k_topk_band": 1, "k_topk_fallback": 2}
WRITE = re.compile(r"(global|flat|buffer)_(store|atomic)")
WAIT = re.compile(r"s_waitcnt\b.*vmcnt\(0\)")


def functions(asm):
    """{name: [line, ...]} of a listing, labels and instructions only."""
    out, name = {}, None
    for line in asm.splitlines():
        code = line.split(";")[0].strip()
        m = re.fullmatch(r"(_Z\w+):", code)
        if m:
            name = m.group(1)
            out[name] = []
        elif code.startswith(".Lfunc_end"):
            name = None
        elif name and code and (not code.startswith(".") or re.fullmatch(r"\.LBB\w+:", code)):
            out[name].append(code)
    return out


def uncovered_handovers(code):
    """(releases, barriers that a wave can enter with writes it has not waited
    for and that a release fence follows without another barrier between)."""
    at = {c[:-1]: i for i, c in enumerate(code) if c.endswith(":")}
    after = []
    for i, c in enumerate(code):
        op = c.split()[0]
        to = [i + 1] if op not in ("s_branch", "s_endpgm") and i + 1 < len(code) else []
        if op == "s_branch" or op.startswith("s_cbranch"):
            to.append(at[c.split()[1]])
        after.append(to)
    # forward: may the wave have writes on the way before instruction i
    seen, dirty = [False] * len(code), [False] * len(code)
    seen[0], work = True, [0]
    while work:
        i = work.pop()
        out = bool(WRITE.match(code[i])) or (dirty[i] and not WAIT.match(code[i]))
        for j in after[i]:
            if not seen[j] or (out and not dirty[j]):
                seen[j], dirty[j] = True, dirty[j] or out
                work.append(j)
    bad = []
    for b in [i for i, c in enumerate(code) if c.startswith("s_barrier") and dirty[i]]:
        met, work = set(), list(after[b])
        while work:
            i = work.pop()
            if i in met or code[i].startswith("s_barrier"):
                continue
            met.add(i)
            if code[i].startswith("buffer_wbl2"):
                bad.append(b)
                break
            work += after[i]
    return sum(c.startswith("buffer_wbl2") for c in code), bad


@pytest.mark.parametrize("drained", [False, True])
def test_checker_on_a_listing(drained):
    listing = ["s_cbranch_execz .LBB0_1", "global_atomic_add v[0:1], v2, off", ".LBB0_1:",
               "s_waitcnt %s" % ("vmcnt(0)" if drained else "lgkmcnt(0)"), "s_barrier", "s_cbranch_execz .LBB0_2",
               "buffer_wbl2 sc1", "s_waitcnt vmcnt(0)", "global_atomic_add v0, v[0:1], v2, off sc0", ".LBB0_2:",
               "s_waitcnt vmcnt(0)", "s_barrier", "global_store_dword v[0:1], v2, off", "s_endpgm"]
    assert uncovered_handovers(listing) == (1, [] if drained else [4])


def test_every_wave_waits_before_a_hand_over():
    flags = [f for f in build.FLAGS if f not in ("-shared", "-fPIC")]
    src = [s for s in build.sources() if s.endswith("topk.hip")]
    asm = subprocess.run([build.HIPCC] + flags + ["-I", build.ROOT + "/include", "-S", "--cuda-device-only", "-o", "-"]
                         + src, stdout=subprocess.PIPE, stderr=subprocess.DEVNULL, text=True, check=True).stdout
    handing_over = {}
    for name, code in functions(asm).items():
        releases, bad = uncovered_handovers(code)
        if releases:
            kernel = [k for k in KERNELS if k in name]
            assert len(kernel) == 1, "%s hands over and is not listed here" % name
            handing_over[kernel[0]] = handing_over.get(kernel[0], 0) + 1
            assert not bad, "%s: barriers entered with writes on the way: instructions %s" % (name, bad)
    assert handing_over == KERNELS
