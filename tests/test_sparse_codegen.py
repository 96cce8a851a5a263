"""attn_sparse_kernel holds 251 of 256 registers.  A register spilled inside its loop would be reloaded behind vmcnt(0) and so wait for
the tiles on their way: its loops over tiles must not touch scratch memory, nor read spilled scalars back.  CPU only (hipcc cross-compiles)."""
import os
import re
import subprocess

import pytest

from paper_2604_12798_amd import build

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="hipcc not installed")
def test_sparse_loops_hold_their_registers(tmp_path):
    out = tmp_path / "vfa_fwd.s"
    flags = [f for f in build.HIPCC_FLAGS if f not in ("-shared", "-fPIC")]
    subprocess.run([HIPCC] + flags + ["-S", "--cuda-device-only", "-o", str(out), os.path.join(build.CSRC, "vfa_fwd.hip")],
                   check=True, capture_output=True)
    m = re.search(r"^(_Z\S*attn_sparse_kernel\S*):[^\n]*\n(.*?)\.Lfunc_end", out.read_text(), re.S | re.M)
    assert m and "scratch_" not in m.group(2)
    body = m.group(2).split("\n")
    labels = {x.group(1): n for n, l in enumerate(body) if (x := re.match(r"^(\.LBB\d+_\d+):", l))}
    loops = {}  # first line -> last line
    for n, l in enumerate(body):
        x = re.search(r"s_c?branch\w* (\.LBB\d+_\d+)", l)
        if x and labels.get(x.group(1), n) < n:
            loops[labels[x.group(1)]] = n
    # the loop over unmasked tiles: two steps, their P.V and Q.K^T with and without softmax; the loop over the tiles that may need a mask: one
    for n in (2, 1):
        steps = [body[a:b] for a, b in loops.items() if sum("v_mfma" in x for x in body[a:b]) == n * 48]
        assert len(steps) == 1, [sum("v_mfma" in x for x in body[a:b]) for a, b in loops.items()]
        assert not any("v_readlane" in x for x in steps[0]), n
