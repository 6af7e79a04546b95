"""Ordering rules of the tile kernels that no result shows reliably, checked on
the gfx950 assembly that the compiler makes of them.

Tiles reach LDS by loads that the compiler does not order against LDS reads
(inline assembly), so the kernels order them with barriers: before a barrier
that lets other waves refill a tile, this wave's reads of it are complete.  Nor
does the compiler's hazard pass look inside inline assembly: the loads keep the
wait state between writing M0 and reading it themselves."""

import os
import re
import subprocess

import pytest

from paper_2512_04752_amd import build


def assembly(src, tmp):
    out = os.path.join(tmp, src + ".s")
    r = subprocess.run([build.HIPCC, *build.FLAGS, *build.EXTRA.get(src, []), "--offload-device-only",
                        "-S", os.path.join(build.CSRC, src), "-o", out], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    return open(out).read()


def kernels(text):
    """{mangled name: instructions and labels, in order} of every kernel."""
    found, body = {}, None
    for line in text.splitlines():
        line = line.split(";")[0].strip()
        m = re.match(r"(_ZN\w+):$", line)
        if m:
            body = found.setdefault(m.group(1), [])
        elif line.startswith(".Lfunc_end"):
            body = None
        elif body is not None and line and (line.startswith(".LBB") or not line.startswith(".")):
            body.append(line)
    return {k: v for k, v in found.items() if any(i.startswith("s_endpgm") for i in v)}


def reads_at_barriers(body):
    """Most LDS reads that can be outstanding at each barrier, over all paths."""
    at = {line[:-1]: n for n, line in enumerate(body) if line.endswith(":")}
    most, barriers, todo = {}, {}, [(0, 0)]
    while todo:
        n, out = todo.pop()
        while n < len(body) and most.get(n, -1) < out:
            most[n] = out
            ins = body[n].split()
            wait = re.search(r"lgkmcnt\((\d+)\)", body[n]) if ins[0] == "s_waitcnt" else None
            if ins[0].startswith("ds_read"):
                out = min(out + 1, 63)
            elif wait:
                out = min(out, int(wait.group(1)))
            elif ins[0] == "s_barrier":
                barriers[n] = max(barriers.get(n, 0), out)
            elif ins[0] == "s_endpgm":
                break
            elif ins[0] == "s_branch":
                n = at[ins[1]]
                continue
            elif ins[0].startswith("s_cbranch"):
                todo.append((at[ins[1]], out))
            n += 1
    return [barriers[n] for n in sorted(barriers)]


@pytest.fixture(scope="module")
def gemm(tmp_path_factory):
    return kernels(assembly("gemm.hip", str(tmp_path_factory.mktemp("asm"))))


def of(found, name):
    picked = {k: v for k, v in found.items() if name in k}
    assert picked, name
    return picked


def test_reads_at_barriers_follows_branches():
    body = ["ds_read_b128 a", "s_cbranch_scc1 .LBB0_1", "s_waitcnt vmcnt(0) lgkmcnt(0)", ".LBB0_1:",
            "s_barrier", "ds_read_b128 b", "s_waitcnt lgkmcnt(1)", "s_cbranch_scc0 .LBB0_1", "s_barrier",
            "s_endpgm"]
    assert reads_at_barriers(body) == [1, 1]


def test_opposite_phases_leave_one_half_unread(gemm):
    """256 x 256: a half (8 reads of A, 4 of B) may be in flight at the barrier after its reads,
    as its rows are refilled behind the barrier after that one; two halves may not: the older
    one is refilled behind this barrier."""
    for name, body in of(gemm, "gemm_256x256_kernel").items():
        at = reads_at_barriers(body)
        assert len(at) > 8 and max(at) <= 8, (name, at)


@pytest.mark.parametrize("name", ["gemm_256x128_kernel", "gemm_ring_kernel"])
def test_reads_complete_at_every_barrier(gemm, name):
    """A stage is refilled right behind the barrier that follows its last reads."""
    for kernel, body in of(gemm, name).items():
        at = reads_at_barriers(body)
        assert at and max(at) == 0, (kernel, at)


@pytest.mark.parametrize("src", ["gemm.hip", "attention.hip"])
def test_wait_state_between_m0_and_lds_load(src, tmp_path):
    """gfx9: an LDS-direct load needs one wait state after a scalar write of M0, which holds its
    LDS address (the compiler puts an s_nop there for its own loads)."""
    loads = 0
    for name, body in kernels(assembly(src, str(tmp_path))).items():
        for before, ins in zip(body, body[1:]):
            if "load_lds" in ins:
                loads += 1
                assert not re.match(r"s_\w+ m0,", before), (name, before, ins)
    assert loads > 0
