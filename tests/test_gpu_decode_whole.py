"""Decode steps whose cache is not cut into ranges although the caller asks for several: one workgroup for each KV head, its waves
sharing the keys, on both sides of the lines (a chip of 256 units); and the merge of ranges at the numbers where it changes its rounds.
Against exact attention in 64 bits; bars as in the other parity tests."""
import numpy as np
import pytest

from gpu_util import LSE_ABS, O_MAX_ABS, O_MEAN_ABS

pytestmark = pytest.mark.gpu


def _exact(q, K, V, lens):
    import torch
    O, L = [], []
    for b, n in enumerate(lens):
        g = q.shape[1] // K.shape[1]
        k, v = (x[b, :, :n].double().repeat_interleave(g, 0) for x in (K, V))
        s = (k * q[b].double()[:, None]).sum(-1) * q.shape[-1] ** -0.5
        L.append(torch.logsumexp(s, 1))
        O.append(((s - L[-1][:, None]).exp()[..., None] * v).sum(1))
    return torch.stack(O), torch.stack(L)


# few tiles: fewer, as many and more than the workgroup's waves (four at d = 128, eight at d = 64), the last in the list behind the line
FEW = [(1, 8, 2, 128, n) for n in (1, 64, 65, 192, 256, 257, 320, 321)] + [(1, 8, 2, 64, n) for n in (1, 65, 511, 513, 769, 1024, 1025)]
# as many KV heads as nearly fill the units, fewer; more than units (two workgroups to each), nearly all of the halves, more
MANY = [(24, 8, 8, 128, 700), (16, 8, 8, 128, 700), (24, 24, 8, 64, 1100), (33, 16, 8, 128, 130), (33, 16, 8, 64, 1100), (50, 8, 8, 128, 1100),
        (64, 8, 8, 64, 1100), (65, 8, 8, 128, 130), (48, 8, 8, 128, 1100), (49, 8, 8, 64, 1100)]


@pytest.mark.parametrize("B,Hq,Hkv,d,n", FEW + MANY)
@pytest.mark.parametrize("ragged", [False, True])
def test_whole_cache(B, Hq, Hkv, d, n, ragged):
    import torch
    import paper_2604_12798_amd as vfa
    gen = torch.Generator(device="cuda").manual_seed(B + n)
    q, K, V = (torch.randn(s, generator=gen, device="cuda").bfloat16() for s in ((B, Hq, d), (B, Hkv, n + 7, d), (B, Hkv, n + 7, d)))
    q *= 2
    K[:, :, n:], V[:, :, n:] = float("nan"), float("nan")  # rows beyond the keys are not read
    lens = [n] + [int(x) for x in np.random.default_rng(n).integers(1, n + 1, B - 1)] if ragged else [n] * B
    if ragged:
        K, V = K[:, :, :n].contiguous(), V[:, :, :n].contiguous()  # the longest entry fills the capacity
        O, L = vfa.decode_varlen_fwd(q, K, V, torch.tensor(lens, dtype=torch.int32, device="cuda"), use_minit=False, n_splits=3)
    else:
        O, L = vfa.decode_fwd(q, K, V, n, use_minit=False, n_splits=3)
    eO, eL = _exact(q, K, V, lens)
    err = (O.double() - eO).abs()
    assert err.max() <= O_MAX_ABS and err.mean() <= O_MEAN_ABS and (L.double() - eL).abs().max() <= LSE_ABS


# ranges: one round of the merge (8 at d = 128, 16 at d = 64), two, four and more than four; ranges without keys among them
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("n_splits", [2, 7, 8, 9, 15, 16, 17, 31, 32, 33, 63, 64, 65, 130])
@pytest.mark.parametrize("ragged", [False, True])
def test_ranges(d, n_splits, ragged):
    import torch
    import paper_2604_12798_amd as vfa
    B, Hq, Hkv, n = 3, 6, 2, 64 * 40 + 11
    gen = torch.Generator(device="cuda").manual_seed(n_splits)
    q, K, V = (torch.randn(s, generator=gen, device="cuda").bfloat16() for s in ((B, Hq, d), (B, Hkv, n, d), (B, Hkv, n, d)))
    q *= 2
    lens = [n, 1300, 70] if ragged else [n] * B
    kw = dict(use_minit=False, n_splits=n_splits)
    O, L = vfa.decode_varlen_fwd(q, K, V, torch.tensor(lens, dtype=torch.int32, device="cuda"), **kw) if ragged else vfa.decode_fwd(q, K, V, n, **kw)
    eO, eL = _exact(q, K, V, lens)
    err = (O.double() - eO).abs()
    assert err.max() <= O_MAX_ABS and err.mean() <= O_MEAN_ABS and (L.double() - eL).abs().max() <= LSE_ABS


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("n", [1, 2, 17, 63, 64, 65, 127, 700, 4033])
@pytest.mark.parametrize("n_splits", [1, 4])
def test_nothing_behind_the_keys_is_read(d, n, n_splits):
    """A tile of NaN behind the last key, whatever part of its tile that one leaves empty."""
    import torch
    import paper_2604_12798_amd as vfa
    gen = torch.Generator(device="cuda").manual_seed(n)
    q, K, V = (torch.randn(s, generator=gen, device="cuda").bfloat16() for s in ((2, 8, d), (2, 2, n + 64, d), (2, 2, n + 64, d)))
    K[:, :, n:], V[:, :, n:] = float("nan"), float("nan")
    O, L = vfa.decode_fwd(q, K, V, n, use_minit=False, n_splits=n_splits)
    eO, eL = _exact(q, K, V, [n, n])
    assert (O.double() - eO).abs().max() <= O_MAX_ABS and (L.double() - eL).abs().max() <= LSE_ABS


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("tiles", [2, 5, 12, 20, 40])
def test_ranges_without_keys_change_nothing(d, tiles):
    """More ranges than tiles: one tile to a range, whatever their number, so the same partial sums and, in one, two or four rounds of the merge, the same bits."""
    import torch
    import paper_2604_12798_amd as vfa
    gen = torch.Generator(device="cuda").manual_seed(tiles)
    q, K, V = (torch.randn(s, generator=gen, device="cuda").bfloat16() for s in ((8, 32, d), (8, 4, 64 * tiles, d), (8, 4, 64 * tiles, d)))
    want = vfa.decode_fwd(q, K, V, 64 * tiles - 3, use_minit=False, n_splits=tiles)
    for n_splits in (8, 9, 16, 17, 32, 33, 64, 65, 130):
        if n_splits > tiles:
            got = vfa.decode_fwd(q, K, V, 64 * tiles - 3, use_minit=False, n_splits=n_splits)
            assert all(torch.equal(x, y) for x, y in zip(got, want)), n_splits
