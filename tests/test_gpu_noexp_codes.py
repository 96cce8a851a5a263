"""The weights of the forms without exponentials are E5M2 codes, one rounding away from the score: code by code against that
definition, with scores that come as close to the rounding's ties as the codes of whole-number operands can."""
import math

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

N = 64  # one tile of keys
E2M1 = np.array([0, 0.5, 1, 1.5, 2, 3, 4, 6])


def _expected(s, close):
    """Scores in log2 units, [rows, keys] -> weights / row sum: code = 4 (s - max - 4) + 119.8277 to the nearest whole one, at least 0.
    The offset's fraction leaves every score at least 4e-4 of a code away from a tie, ten times what 32 bits round at these sizes; `close`:
    some are that close."""
    c = 4.0 * (s - s.max(1, keepdims=True) - 4.0) + float(np.float32(119.8277))
    assert np.abs(c - np.floor(c) - 0.5).min() > 4e-4
    if close:
        assert (np.abs(c - np.floor(c) - 0.5) < 5e-4).sum() > 40
    k = np.clip(np.floor(c + 0.5), 0, 123).astype(np.int64)
    w = np.where(k >= 4, 2.0 ** (k // 4 - 15.0) * (1 + k % 4 / 4.0), 2.0 ** -14 * (k % 4) / 4.0)  # (E5M2's subnormal codes are 1 to 3)
    return w / w.sum(1, keepdims=True)


def _check(O, s, close=True):
    # the values are a unit vector for each key, so O holds the weights; half a unit of bf16's eight bits, 2^-8 (and a 64th of that for the
    # division in 32 bits), against steps of a seventh between one code's weight and the next
    want = _expected(s, close)
    err = np.abs(O.float().cpu().numpy().astype(np.float64)[0, 0, :, :N] - want)
    bad = np.argwhere(err > 2.0 ** -8 * (1 + 2.0 ** -6) * want)
    assert len(bad) == 0, (len(bad), bad[:4].tolist())


def _unit_values(vfa):
    import torch
    V = torch.zeros((1, 1, N, 128), dtype=torch.bfloat16, device="cuda")
    V[0, 0, torch.arange(N), torch.arange(N)] = 1.0
    return vfa.fp8_pack_v(V, 1.0)


@pytest.mark.parametrize("seed", [0, 1])
def test_fp8(seed):
    import torch
    import paper_2604_12798_amd as vfa
    rng = np.random.default_rng(seed)
    q, k = (rng.integers(-8, 9, (N, 128)).astype(np.float32) for _ in range(2))
    code = lambda x: vfa.fp8_quantize(torch.from_numpy(x).cuda().bfloat16().view(1, 1, N, 128), 1.0)
    # products times 2^-8: the codes' fractions are 64ths beside the offset's
    c = 2.0 ** -8
    O, _ = vfa.fp8_attn_fwd(code(q), code(k), _unit_values(vfa), descale_q=float(np.float32(c / math.log2(math.e))), descale_k=1.0, descale_v=1.0,
                            softmax_scale=1.0, noexp=True, causal=False, use_minit=False)
    _check(O, c * (q.astype(np.float64) @ k.T.astype(np.float64)))


# block scale bytes of the queries and the keys: the product of the two scales is what counts, wherever each of them lies
@pytest.mark.parametrize("qs,ks,features", [(127, 121, 128), (0, 248, 128), (5, 243, 128), (6, 242, 128), (128, 120, 128), (200, 48, 128), (248, 0, 128),
                                            (254, 0, 3)])
def test_mxfp4(qs, ks, features):
    import torch
    import paper_2604_12798_amd as vfa
    rng = np.random.default_rng(qs)
    qc, kc = (np.where(np.arange(128) < features, rng.integers(0, 16, (N, 128)), 0) for _ in range(2))
    value = lambda c: np.where(c & 8, -1.0, 1.0) * E2M1[c & 7]
    s = 2.0 ** (qs + ks - 254.0) * (value(qc) @ value(kc).T)
    pack = lambda c: torch.from_numpy((c[:, ::2] | c[:, 1::2] << 4).astype(np.uint8)).cuda().view(1, 1, N, 64)
    scales = lambda b: torch.full((1, 1, N, 4), b, dtype=torch.uint8, device="cuda")
    O, _, _ = vfa.mxfp4_attn_fwd(pack(qc), scales(qs), pack(kc), scales(ks), _unit_values(vfa), descale_v=1.0, softmax_scale=math.log(2.0), noexp=True,
                                 causal=False, use_minit=False)
    _check(O, s, features == 128)  # (three features and a scale of 1: quarters of a binade, none near a tie)
