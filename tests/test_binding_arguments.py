"""Arguments outside the range of their C type: the native module takes them as ctypes does (the low bits), so that the C entry
points judge what is in range, with the codes that vfa.h names.  CPU only: nothing below gets as far as a launch."""
import ctypes

import pytest

from paper_2604_12798_amd import build


@pytest.fixture(scope="module")
def pkg():
    import os
    import paper_2604_12798_amd as p
    if not os.path.exists(p.LIB_PATH) or not os.path.exists(build.BINDING):
        build.build_lib()
    return p


class Index:
    def __index__(self):
        return 65


@pytest.mark.parametrize("n", [2 ** 31, -2 ** 31 - 1, 2 ** 32 + 65, 2 ** 63, 2 ** 64 + 65, 10 ** 30, True, Index()])
def test_whole_numbers(pkg, n):
    L, N = pkg.lib(), pkg._n()
    i = ctypes.c_int
    assert N.vfa_workspace_bytes(1, 1, n, 64, 64) == L.vfa_workspace_bytes(i(1), i(1), i(n if not isinstance(n, Index) else 65), i(64), i(64))
    # a size, a count and pointers, in calls that are refused or have nothing to do
    p = 0x1000
    assert N.vfa_attn_fwd(p, p, p, p, None, 1, 4, 2, 256, 128, 128, 64, 1, n, 1, 1, float("nan"), p, n, None) == -1
    ptr = p if isinstance(n, Index) else n
    assert N.vfa_fp8_quantize(ptr, ptr, 0, 1.0, ptr) == 0 and N.vfa_fp8_quantize(p, p, n, -1.0, None) == -1


def test_wrong_types(pkg):
    N = pkg._n()
    for bad in (1.0, "1", None, [1]):
        with pytest.raises(TypeError):
            N.vfa_workspace_bytes(1, 1, bad, 64, 64)
    with pytest.raises(TypeError):
        N.vfa_workspace_bytes(1, 1, 64, 64)
    with pytest.raises(TypeError):
        N.vfa_fp8_quantize(None, None, 0, "1", None)
    with pytest.raises(TypeError):
        N.vfa_fp8_quantize(1.5, None, 0, 1.0, None)


def test_out_of_range_is_an_error_code(pkg):
    """The wrappers raise VfaError, which callers catch, and not OverflowError."""
    L = pkg._n()
    assert pkg.workspace_bytes(1, 1, 2 ** 31, 64, 64) == 0
    assert L.vfa_kblock_summary_append(0x1000, 0x1000, 1, 1, 64, 0, 2 ** 31, 128, 64, None) == -1
