"""Kernels that refill LDS with direct loads: no wavefront says at a barrier that a stage may be refilled while its own reads
of it are outstanding.  Read from the assembly of this repository's kernels, since which side of a bare barrier a wait for
a read falls on is the compiler's choice."""
import os
import re
import subprocess

import pytest

from paper_2505_03983_amd import build


DIRECT_LOAD = re.compile(r"global_load_lds_|buffer_load_\S+ .*\blds\b")     # from memory into LDS


def kernels(asm):
    """{name: [instruction or label, ...]} of the kernels that use direct loads."""
    out, name, body = {}, None, []
    for line in asm.splitlines():
        s = line.split(";")[0].strip()
        m = re.match(r"(_ZN\S+):$", s)
        if m:
            name, body = m.group(1), []
        elif s.startswith(".Lfunc_end"):
            if name and any(DIRECT_LOAD.match(x) for x in body):
                out[name] = body
            name = None
        elif name and s and (s.startswith(".LBB") or not s.startswith(".")):
            body.append(s)
    return out


def reads_at_barriers(body):
    """For every barrier the largest number of LDS reads that may be outstanding, over all paths to it."""
    at = {s[:-1]: i for i, s in enumerate(body) if s.endswith(":")}
    seen, work, barriers = {}, [(0, 0)], {}
    while work:
        i, n = work.pop()
        while i < len(body) and seen.get(i, -1) < n:
            seen[i] = n
            s = body[i]
            op = s.split()[0]
            if op.startswith("ds_read"):
                n = min(n + 1, 16)
            elif op == "s_waitcnt":
                m = re.search(r"lgkmcnt\((\d+)\)", s)
                n = min(n, int(m.group(1))) if m else n
            elif op == "s_barrier":
                barriers[i] = max(barriers.get(i, 0), n)
            elif op == "s_branch":
                i = at[s.split()[1]]
                continue
            elif op.startswith("s_cbranch"):
                work.append((at[s.split()[1]], n))
            elif op == "s_endpgm":
                break
            i += 1
    return list(barriers.values())


def test_reads_at_barriers_follows_branches():
    loop = ["s_branch .LBB0_2", ".LBB0_1:", "ds_read_b128 v[0:3], v4", "s_cbranch_scc1 .LBB0_3", "s_waitcnt lgkmcnt(0)",
            ".LBB0_2:", "s_barrier", "s_cbranch_scc0 .LBB0_1", ".LBB0_3:", "s_waitcnt vmcnt(0) lgkmcnt(1)", "s_barrier", "s_endpgm"]
    assert reads_at_barriers(loop) == [0, 1]


def assembly(source, tmp_path):
    out = tmp_path / "k.s"
    flags = [f for f in build.FLAGS if f != "-shared"]
    r = subprocess.run([os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")] + flags +
                       ["--cuda-device-only", "-S", os.path.join(build.CSRC, source), "-o", str(out)],
                       stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    assert r.returncode == 0, r.stdout
    return out.read_text()


@pytest.mark.parametrize("source, least", [("mlp.hip", 96), ("gmm.hip", 1)])
def test_no_lds_read_is_outstanding_at_a_barrier(source, least, tmp_path):
    ks = kernels(assembly(source, tmp_path))
    print(source, len(ks))
    assert len(ks) >= least
    bad = {k: b for k, b in ((k, reads_at_barriers(v)) for k, v in ks.items()) if any(b)}
    assert not bad, bad


def test_kernels_of_few_rows_do_not_wait_for_every_read(tmp_path):
    """Their direct loads do not make the compiler wait for every read of LDS at once: waits in their loops leave some
    outstanding."""
    ks = {k: v for k, v in kernels(assembly("mlp.hip", tmp_path)).items() if "gemm_bf16_few" in k}
    assert len(ks) >= 16
    for k, body in ks.items():
        waits = [int(m.group(1)) for m in (re.search(r"lgkmcnt\((\d+)\)", x) for x in body if x.startswith("s_waitcnt")) if m]
        assert sum(n >= 2 for n in waits) >= 6, (k, waits)
