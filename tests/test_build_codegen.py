"""The VSA ping-pong kernel sits at the register limit: a spill inside one of its steady loops costs a factor, because
a scratch reload waits for vmcnt(0) and so drains the tile prefetches.  This test compiles vsa_pp.hip to assembly with
the flags build.py uses and checks that the fast loops hold no scratch access.  CPU only (hipcc cross-compiles)."""
import os
import re
import subprocess

import pytest

from paper_2604_12798_amd import build

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="hipcc not installed")
def test_vsa_fast_loops_have_no_scratch_access(tmp_path):
    out = tmp_path / "vsa_pp.s"
    flags = [f for f in build.HIPCC_FLAGS if f not in ("-shared", "-fPIC")] + build.EXTRA_FLAGS["vsa_pp.hip"]
    subprocess.run([HIPCC] + flags + ["-S", "--cuda-device-only", "-o", str(out), os.path.join(build.CSRC, "vsa_pp.hip")],
                   check=True, capture_output=True)
    text = out.read_text()
    start = text.index("attn_vsa_pp_kernel")
    start = text.index(":\n", start)
    body = text[start:text.index(".Lfunc_end", start)].split("\n")
    labels = {m.group(1): n for n, l in enumerate(body) if (m := re.match(r"^(\.LBB\d+_\d+):", l))}
    # innermost loops = backward branches; a step pair of the pipeline holds 64 MFMAs
    loops = {}
    for n, l in enumerate(body):
        m = re.search(r"s_c?branch\w* (\.LBB\d+_\d+)", l)
        if m and m.group(1) in labels and labels[m.group(1)] < n:
            a = labels[m.group(1)]
            seg = body[a:n]
            if sum("v_mfma" in x for x in seg) == 64:
                loops[a] = min(loops.get(a, (1 << 30, 0)), (n - a, sum("scratch_" in x for x in seg)))
    assert len(loops) >= 4, "expected a fast and a general loop per group"
    # the fast loops are the two shortest ones (no masked / exact-max / ragged variants inside)
    fast = sorted(loops.values())[:2]
    assert all(length < 1300 for length, _ in fast), fast
    assert all(scratch == 0 for _, scratch in fast), f"scratch accesses in the VSA fast loops: {fast}"


@pytest.fixture(scope="module")
def other_kernels(tmp_path_factory):
    """The AMD assembly of vfa_fwd.hip."""
    out = tmp_path_factory.mktemp("codegen") / "vfa_fwd.s"
    flags = [f for f in build.HIPCC_FLAGS if f not in ("-shared", "-fPIC")]
    subprocess.run([HIPCC] + flags + ["-S", "--cuda-device-only", "-o", str(out), os.path.join(build.CSRC, "vfa_fwd.hip")],
                   check=True, capture_output=True)
    return out.read_text()


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="hipcc not installed")
def test_inner_loops_have_no_scratch_access(other_kernels):
    """The other kernels: several (the ping-pong baselines, the 8-bit and 4-bit forms with folded scales) have spilled registers, all
    of them outside the loops over tiles.  Left out: the generic kernel with ablation switches at d = 128, block_m = 128."""
    seen = []
    for m in re.finditer(r"^(_Z\S*):[^\n]*\n(.*?)\.Lfunc_end", other_kernels, re.S | re.M):
        kernel = re.search(r"(attn_\w+?_kernel|decode_split_kernel)I(\w+?)EEv", m.group(1))
        if not kernel or re.fullmatch(r"Li128ELi4ELi[12]ELb0E", kernel.group(2)):
            continue
        body = m.group(2).split("\n")
        labels = {x.group(1): n for n, l in enumerate(body) if (x := re.match(r"^(\.LBB\d+_\d+):", l))}
        loops = {}  # first line -> last line
        for n, l in enumerate(body):
            x = re.search(r"s_c?branch\w* (\.LBB\d+_\d+)", l)
            if x and labels.get(x.group(1), n) < n:
                loops[labels[x.group(1)]] = n
        inner = [body[a:b] for a, b in loops.items() if not any(a < c and d <= b for c, d in loops.items())]
        tiles = [seg for seg in inner if any("v_mfma" in x for x in seg)]
        assert tiles, m.group(1)
        for seg in tiles:
            assert not any("scratch_" in x for x in seg), m.group(1)
        seen.append(kernel.group(1))
    assert {"attn_fwd_pp_kernel", "attn_fwd_frozen_kernel", "attn_fwd_short_kernel", "attn_fwd_kernel", "attn_fp8_kernel",
            "attn_mx4_kernel", "decode_split_kernel"} <= set(seen), seen


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="hipcc not installed")
def test_decode_needs_no_function_attribute(other_kernels):
    """A decode step may be the first call of a process and be captured: its kernels' LDS is of fixed size, so nothing has to raise a
    limit for what a launch adds to it, also where four or eight waves take 128 KiB."""
    lds = {m.group(1): int(m.group(2)) for m in
           re.finditer(r"\.amdhsa_kernel (\S*decode_split_kernel\S*)\n\s*\.amdhsa_group_segment_fixed_size (\d+)", other_kernels)}
    assert len(lds) >= 19, sorted(lds)
    for name, size in lds.items():
        d, waves = (int(x) for x in re.search(r"ILi(\d+)ELi(\d)E", name).groups())
        assert size == waves * 2 * 64 * 2 * d, (name, size)  # a tile of K and one of V for each wave


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="hipcc not installed")
def test_only_requests_use_m0(other_kernels):
    """request4_at and request2_at leave M0 as they set it, so the compiler must have no use of its own for it in the kernels that call them."""
    seen = set()
    for m in re.finditer(r"^(_Z\S*):[^\n]*\n(.*?)\.Lfunc_end", other_kernels, re.S | re.M):
        kernel = re.search(r"attn_fwd_short_kernel|attn_sparse_kernel", m.group(1))
        if not kernel:
            continue
        assert re.search(r"#ASMSTART\n\s*s_mov_b32 m0, ", m.group(2)), m.group(1)
        assert not re.search(r"\bm0\b", re.sub(r"#ASMSTART.*?#ASMEND", "", m.group(2), flags=re.S)), m.group(1)
        seen.add(kernel.group(0))
    assert len(seen) == 2, seen
