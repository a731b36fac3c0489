"""Static check of the scans' partial memory waits (CPU only: compiles to
gfx950 assembly, runs nothing).

At the end of every chunk the scans publish the next chunk's LDS-DMA data
with `s_waitcnt vmcnt(N)` followed by a barrier, N > 0 leaving that many of
the wave's newest vector-memory operations in flight.  Vector memory
operations complete in issue order, so this is correct only if those N
newest operations were all issued after the last LDS-DMA (they are register
prefetches and stores, whose own uses the compiler waits for).  This test
compiles both scan kernels and checks, for every such wait in every template
instance, that at least N vector-memory instructions lie between the last
LDS-DMA instruction and the wait.

The side waves of the wave-specialised scans leave newer LDS-DMA in flight as
well, so for them every path through their part of the assembly is followed for
sequences of 1 to 4 chunks: the groups of memory operations, and the places
where a group's copies must have landed, are named by comments in the assembly
(RLA_NOTE), a wait for all but N operations completes every operation with N or
more newer ones, and no path may reach the place where a copy is awaited before
a wait has completed it.
"""
import functools
import os
import re
import subprocess
import tempfile

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2509_25223_amd", "csrc")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


@functools.lru_cache(None)
def _asm(src: str) -> str:
    from paper_2509_25223_amd import build as B
    with tempfile.TemporaryDirectory() as d:
        out = os.path.join(d, "k.s")
        cmd = [HIPCC] + [f for f in B.FLAGS if f not in ("-fPIC",)] + [
            "-x", "hip", "--cuda-device-only", "-S", os.path.join(CSRC, src), "-o", out]
        r = subprocess.run(cmd, capture_output=True, text=True)
        assert r.returncode == 0, r.stderr[-2000:]
        return open(out).read()


def _publishing_waits(body):
    """(N, ops after the last LDS-DMA, index) for each vmcnt(N > 0) wait
    that reaches a barrier before any other vector-memory op or vmcnt wait."""
    out = []
    for k, line in enumerate(body):
        m = re.match(r"s_waitcnt vmcnt\((\d+)\)", line)
        if not m or int(m.group(1)) == 0:
            continue
        publishes = False
        for x in body[k + 1:]:
            op = x.split()[0]
            if op == "s_barrier":
                publishes = True
                break
            if op.startswith(("global_", "buffer_")) or "vmcnt" in x:
                break
        if not publishes:
            continue
        after = 0
        for x in reversed(body[:k]):
            op = x.split()[0]
            if op.startswith(("global_", "buffer_")):
                if "_lds" in op:
                    break
                after += 1
        out.append((int(m.group(1)), after, k))
    return out


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="hipcc not available")
@pytest.mark.parametrize("src,kernel", [("fwd_scan.hip", "fwd_scan_kernel"),
                                        ("bwd_scan.hip", "bwd_scan_kernel")])
def test_partial_waits_leave_no_dma_in_flight(src, kernel):
    s = _asm(src)
    names = re.findall(r"^(_Z\w*%s\w*):" % kernel, s, re.M)
    assert names, "no %s instances found" % kernel
    checked = 0
    for name in names:
        i = s.index(name + ":")
        j = s.index(".Lfunc_end", i)
        body = [l.strip() for l in s[i:j].split("\n")
                if l.strip() and not l.strip().startswith((";", "."))
                and not l.strip().endswith(":")]
        for n, after, _ in _publishing_waits(body):
            assert after >= n, (name, n, after)
            checked += 1
    assert checked > 0


# ---- wave-specialised scans: every path of a side wave ----
VMEM = ("global_", "buffer_", "scratch_", "flat_")


def fwd_notes(rdn, ckpt, nch, w0):
    """The notes a side wave (w0: the one that moves the gates) passes over nch chunks."""
    yield from ["copy gates"] * w0 + ["copy V", "copy S matrices"] + ["copy R matrices"] * rdn
    yield from ["await gates"] * w0 + ["copy gates"] * (w0 and nch > 1)
    for c in range(nch):
        more = c + 1 < nch
        yield from ["copy V"] * more + ["store o, r"] * (c > 0) + ["await S matrices"]
        yield from ["store U^R"] * (ckpt and rdn and c > 0) + ["await R matrices"] * rdn
        if more and w0:
            yield from ["first chunk"] * (c == 0) + ["await gates"] + ["copy gates"] * (c + 2 < nch)
        yield from ["copy S matrices"] * more + ["store R, U"] * ckpt
        yield from ["copy R matrices"] * (more and rdn) + ["await V"] * more
    yield "end"


def bwd_notes(nch, w0):
    yield from ["copy gates"] * w0 + ["copy dO", "copy mask", "copy matrices", "copy MG"]
    for c in reversed(range(nch)):
        later, more = c + 1 < nch, c > 0
        yield from ["await gates"] * w0 + ["store dR"] * later
        yield from ["copy gates"] * (w0 and more) + ["store dX, dYR"] * later + ["await matrices, mask"]
        yield from ["copy dO", "load Q"] * more + ["store dY"] * later + ["await MG"]
        yield from ["await dO", "copy matrices"] * more
        yield from ["copy mask", "copy MG"] * more + ["store dv, dS"]
    yield "end"


class SideWave:
    def __init__(self, name, asm):
        i = asm.index("\n" + name + ":")
        text = [l.strip() for l in asm[i:asm.index(".Lfunc_end", i)].split("\n")]
        self.name, self.code, label = name, [], {}
        for l in text:
            m = re.match(r"(\.LBB\w+):", l)
            if m:
                label[m.group(1)] = len(self.code)
            elif l.startswith("; rla: "):
                self.code.append(("note", l[7:]))
            elif l and l[0] not in ";.#" and not l.endswith(":"):
                op = l.split()[0]
                if op.startswith(VMEM):
                    self.code.append(("copy" if "_lds_" in op else "vmem", None))
                elif op == "s_waitcnt" and "vmcnt" in l:
                    self.code.append(("wait", int(re.search(r"vmcnt\((\d+)\)", l).group(1))))
                elif op.startswith(("s_cbranch", "s_branch")):
                    self.code.append((op, l.split()[1]))
                elif op in ("s_endpgm", "s_setpc_b64"):
                    self.code.append(("stop", None))
        self.code = [(k, label[a] if k.startswith("s_") else a) for k, a in self.code]

    def follow(self, notes):
        """Follows every path whose notes are these, from the note "side waves".  A
        state: instruction, notes passed, the group that copies belong to, whether a
        store's rows may all be missing, and for each group with copies in flight the
        operations issued since its last one.  Returns the awaits passed."""
        start = [k for k, (op, a) in enumerate(self.code) if op == "note" and a == "side waves"]
        assert len(start) == 1, self.name
        todo, seen, awaits, complete = [(start[0] + 1, 0, None, False, ())], set(), 0, False
        while todo:
            state = todo.pop()
            if state in seen:
                continue
            seen.add(state)
            k, pos, group, maybe, flight = state
            op, a = self.code[k]
            if op == "note":
                if a != notes[pos]:
                    continue   # not a path of this sequence
                if a == "end":
                    complete = True
                    continue
                pos += 1
                if a.startswith("await "):
                    awaits += 1
                    late = [g for g, _ in flight if g in a[6:].split(", ")]
                    assert not late, "%s: %s in flight at note %d of %s" % (self.name, late, pos, notes)
                else:
                    group = a[5:] if a.startswith("copy ") else None
                    maybe = a == "store dv, dS"
            elif op in ("copy", "vmem"):
                flight = {g: min(n + 1, 63) for g, n in flight}
                if op == "copy":
                    assert group, "%s: a copy outside a named group, note %d of %s" % (self.name, pos, notes)
                    flight[group] = 0
                flight = tuple(sorted(flight.items()))
            elif op == "wait":
                flight = tuple((g, n) for g, n in flight if n < a)
            elif op == "stop":
                continue
            nxt = [k + 1]
            if op == "s_branch":
                nxt = [a]
            elif op in ("s_cbranch_execz", "s_cbranch_execnz"):
                # some lane is active but where a group may have no row to store
                skip, go = (a, k + 1) if op.endswith("execz") else (k + 1, a)
                nxt = [go, skip] if maybe else [go]
            elif op.startswith("s_cbranch"):
                nxt = [k + 1, a]
            todo += [(n, pos, group, maybe, flight) for n in nxt]
        assert complete, "%s: no path with the notes %s" % (self.name, notes)
        return awaits


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="hipcc not available")
@pytest.mark.parametrize("src,kernel", [("fwd_scan.hip", "fwd_scan_ws_kernel"), ("bwd_scan.hip", "bwd_scan_ws_kernel")])
def test_side_waves_await_their_copies(src, kernel):
    asm = _asm(src)
    names = re.findall(r"^(_Z\w*%s\w*):" % kernel, asm, re.M)
    assert len(names) >= 8
    for name in names:
        args = re.search(kernel + r"It((?:L[ib]\d+E)+)", name).group(1)   # template arguments after the type
        args = [int(x) for x in re.findall(r"L[ib](\d+)E", args)]
        wave = SideWave(name, asm)
        for nch in range(1, 5):
            for w0 in (True, False):
                notes = list(fwd_notes(bool(args[2]), bool(args[4]), nch, w0) if src[0] == "f" else bwd_notes(nch, w0))
                assert wave.follow(notes) > 0
