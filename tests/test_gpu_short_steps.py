"""Alg. 1 on attn_short.hpp: every number of steps on either side of the six that its loop is unrolled by, list lengths and heads that
are no powers of two.  Every row of every head against exact attention."""
import pytest

from gpu_util import check_every_row

pytestmark = pytest.mark.gpu


def _check(d, B, Hq, Hkv, N, causal):
    import torch
    import paper_2604_12798_amd as vfa
    gen = torch.Generator(device="cuda").manual_seed(N + 7 * Hq + d)
    R = lambda h: torch.randn((B, h, N, d), generator=gen, device="cuda", dtype=torch.bfloat16)
    Q, K, V = R(Hq) * 2, R(Hkv), R(Hkv)
    O, L = torch.full_like(Q, float("nan")), torch.full(Q.shape[:3], float("nan"), device="cuda")
    vfa.vfa_attn_fwd(Q, K, V, causal=causal, out=O, lse=L)
    check_every_row(Q, K, V, O, L, causal)


# steps of 64 keys (two groups) and of 128 (four); lists of each XCD (KV heads in eights) and one for all
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("causal", [True, False])
@pytest.mark.parametrize("steps", list(range(1, 15)))
def test_steps(d, causal, steps):
    _check(d, 1, 6, 2, 64 * steps - (steps % 3), causal)
    _check(d, 2, 20, 4, 64 * steps, causal)
    if steps >= 5:
        _check(d, 1, 3, 1, 128 * steps - 5 * (steps % 2), causal)

