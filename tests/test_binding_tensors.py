"""What the native module looks up on tensors for the wrappers: the same attributes as Python code would, for whatever has them, with the
same refusals.  CPU only: objects that only look like tensors, and calls that are refused before anything is launched."""
import itertools
import os
import sys

import pytest

from paper_2604_12798_amd import build


@pytest.fixture(scope="module")
def pkg():
    import paper_2604_12798_amd as p
    if not os.path.exists(p.LIB_PATH) or not os.path.exists(build.BINDING):
        build.build_lib()
    p._n()
    return p


class Fake:
    def __init__(self, shape, dtype, is_cuda=True, contiguous=True, ptr=0x1000):
        self.shape, self.dtype, self.is_cuda, self.c, self.ptr = shape, dtype, is_cuda, contiguous, ptr

    def is_contiguous(self):
        return self.c

    def dim(self):
        return len(self.shape)

    def data_ptr(self):
        if isinstance(self.ptr, Exception):
            raise self.ptr
        return self.ptr


def rule(Q, K, V, dtype):
    for t in (Q, K, V):
        if not (t.is_cuda and t.dtype == dtype and t.is_contiguous() and t.dim() == 4):
            return None
    B, Hq, N, d = Q.shape
    if K.shape != V.shape or K.shape[0] != B or K.shape[2] != N or K.shape[3] != d:
        return None
    return B, Hq, K.shape[1], N, d


def test_check_qkv(pkg):
    import torch
    bf, shapes = torch.bfloat16, [(2, 4, 70, 64), (2, 2, 70, 64), (2, 4, 71, 64), (1, 4, 70, 64), (2, 4, 70, 128), (4, 70, 64), [2, 2, 70, 64], torch.Size((2, 2, 70, 64))]
    kinds = [dict(), dict(is_cuda=False), dict(contiguous=False), dict(dtype=torch.float16)]
    seen = 0
    for s, kind, which in itertools.product(itertools.product(shapes, repeat=3), kinds, range(3)):
        t = [Fake(x, **{"dtype": bf, **(kind if i == which else {})}) for i, x in enumerate(s)]
        want = rule(*t, bf)
        if want is None:
            with pytest.raises(ValueError):
                pkg._n().check_qkv(*t, bf)
        else:
            assert pkg._n().check_qkv(*t, bf) == want
            seen += 1
    assert seen > 10


def test_check_cache(pkg):
    import torch
    n, bf = pkg._n(), torch.bfloat16
    q, K = Fake((3, 8, 64), bf), Fake((3, 2, 500, 64), bf)
    assert n.check_cache(q, K, K, bf) == (3, 8, 64, 2, 500)
    for bad in (dict(is_cuda=False), dict(contiguous=False), dict(dtype=torch.float16)):
        for which in range(3):
            t = [q, K, K]
            t[which] = Fake(t[which].shape, **{"dtype": bf, **bad})
            with pytest.raises(ValueError):
                n.check_cache(*t, bf)
            assert n.check_cache(*t, None) == (3, 8, 64, 2, 500)
    with pytest.raises(ValueError):
        n.check_cache(Fake((3, 8, 1, 64), bf), K, K, bf)
    with pytest.raises(ValueError):
        n.check_cache(q, Fake((3, 2), bf), K, None)


def test_missing_attributes_and_errors_pass_through(pkg):
    import torch
    n, bf = pkg._n(), torch.bfloat16
    K = Fake((3, 2, 500, 64), bf)
    for call in (lambda: n.check_qkv(1, K, K, bf), lambda: n.check_cache(1, K, K, bf), lambda: n.bytes_of(1)):
        with pytest.raises(AttributeError):
            call()
    with pytest.raises(TypeError):
        n.check_qkv(K, K, K)

    class Bad(Fake):
        def is_contiguous(self):
            raise KeyError("mine")
    with pytest.raises(KeyError):
        n.check_qkv(K, Bad((3, 2, 500, 64), bf), K, bf)


def test_pointers_of_tensors(pkg):
    """An integer stands for no tensor, whatever data_ptr() raises comes through, and None is the null pointer."""
    n = pkg._n()
    x = Fake((8,), None)
    assert n.vfa_fp8_quantize_t(x, x, 0, 1.0, 0) == 0 and n.vfa_fp8_quantize_t(None, x, 8, 1.0, None) == -1
    assert n.vfa_fp8_quantize_t(Fake((8,), None, ptr=0x1008), x, 8, 1.0, None) == -1  # (misaligned)
    for bad in (0x1000, "x", 1.5, [x]):
        with pytest.raises(AttributeError):
            n.vfa_fp8_quantize_t(bad, x, 0, 1.0, 0)
    with pytest.raises(ZeroDivisionError):
        n.vfa_fp8_quantize_t(Fake((8,), None, ptr=ZeroDivisionError()), x, 0, 1.0, 0)
    with pytest.raises(TypeError):
        n.vfa_fp8_quantize_t(Fake((8,), None, ptr=None), x, 0, 1.0, "stream")
    with pytest.raises(TypeError):
        n.vfa_fp8_quantize_t(Fake((8,), None, ptr="0x1000"), x, 0, 1.0, 0)
    import torch
    t = torch.empty((3, 5), dtype=torch.float32)
    assert n.bytes_of(t) == 60 and n.vfa_fp8_quantize_t(t, t, 0, 1.0, 0) == 0


def test_nothing_is_kept(pkg):
    """References are given back, on the way out with an error too."""
    import torch
    n, bf = pkg._n(), torch.bfloat16
    shape = (3, 2, 500, 64)
    good, bad = Fake(shape, bf), Fake(shape, bf, contiguous=False)
    before = [sys.getrefcount(x) for x in (good, bad, shape, bf)]
    for _ in range(100):
        n.check_qkv(good, good, good, bf)
        n.vfa_fp8_quantize_t(good, good, 0, 1.0, 0)
        for t in ((good, bad, good), (good, good, 1)):
            with pytest.raises((ValueError, AttributeError)):
                n.check_qkv(*t, bf)
    after = [sys.getrefcount(x) for x in (good, bad, shape, bf)]
    assert all(abs(a - b) <= 2 for a, b in zip(after, before)), (before, after)
