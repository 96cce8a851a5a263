"""Alg. 1 on attn_short.hpp: every number of steps on either side of the six that its loop is unrolled by, list lengths and heads that
are no powers of two, and sizes on both sides of the lines to the other kernels.  Every row of every head against exact attention."""
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


# the lines of short_groups on a chip of 256 units, the last length on this kernel and the next one
@pytest.mark.parametrize("d,Hq,Hkv,N,causal", [
    (128, 4, 2, 6144, True), (128, 14, 7, 5632, True), (128, 60, 15, 2176, True), (128, 45, 45, 3328, True), (128, 3, 3, 4096, False),
    (128, 16, 4, 2688, False), (128, 40, 10, 2176, False), (128, 80, 20, 1792, False), (128, 48, 12, 1152, False),
    (64, 16, 4, 6144, True), (64, 64, 16, 3648, True), (64, 96, 16, 2944, True), (64, 8, 8, 6144, False), (64, 20, 5, 3072, False), (64, 72, 18, 1664, False),
    (64, 36, 9, 3072, False), (64, 152, 38, 1280, False), (64, 84, 21, 2048, False), (64, 8, 2, 3008, False),
    # (other lengths about which calls change kernels, or did by number of tiles alone)
    (128, 64, 32, 3008, True), (128, 48, 48, 3840, True), (64, 320, 32, 2176, True), (128, 64, 16, 2048, True), (128, 64, 16, 1536, False),
    (128, 48, 16, 2048, False), (128, 4, 4, 4096, False), (64, 128, 32, 1536, False), (64, 32, 8, 3072, False)])
@pytest.mark.parametrize("behind", [0, 1])
def test_lines(d, Hq, Hkv, N, causal, behind):
    _check(d, 1, Hq, Hkv, N + behind, causal)


# KV heads that are no eights: lists for the eights and the rest (many items, no mask), one order for all (few), the last rows of a call
@pytest.mark.parametrize("d,B,Hq,Hkv,N,causal", [(128, 1, 45, 15, 1000, True), (128, 3, 18, 9, 600, False), (64, 2, 44, 11, 1500, True), (64, 1, 30, 15, 500, False),
                                                 (128, 1, 40, 20, 698, True), (64, 1, 20, 20, 1329, True), (128, 1, 30, 10, 2500, False)])
def test_kv_heads_that_are_no_eights(d, B, Hq, Hkv, N, causal):
    _check(d, B, Hq, Hkv, N, causal)


# full rounds of the other kernels stay with them, uneven ones do not (a chip of 256 units).  vfa_variant_fwd never runs on attn_short.hpp, so the
# same bits mean the same kernel
@pytest.mark.parametrize("d,Hq,Hkv,N,causal,short", [
    (128, 128, 128, 2048, True, False), (128, 128, 128, 3072, True, False), (128, 48, 48, 5632, True, False), (128, 64, 16, 2048, True, False),
    (128, 128, 32, 1536, False, False), (64, 40, 10, 3072, False, False), (128, 64, 16, 3600, True, True), (128, 24, 24, 5000, True, True),
    (128, 32, 8, 3328, True, False), (128, 32, 16, 3328, True, True)])
def test_rounds(d, Hq, Hkv, N, causal, short):
    import torch
    import paper_2604_12798_amd as vfa
    if torch.cuda.get_device_properties(0).multi_processor_count != 256:
        pytest.skip("lines of a chip of 256 units")
    gen = torch.Generator(device="cuda").manual_seed(N)
    Q, K, V = (torch.randn((1, h, N, d), generator=gen, device="cuda", dtype=torch.bfloat16) for h in (Hq, Hkv, Hkv))
    O, L = vfa.vfa_attn_fwd(Q, K, V, causal=causal)
    O2, L2, _ = vfa.vfa_variant_fwd(Q, K, V, causal=causal)
    assert (torch.equal(O, O2) and torch.equal(L, L2)) != short


# a slot's rows behind the last key are the next head's, or nothing: K and V come by requests whose range ends with the head's keys
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("N", [1, 33, 65, 100, 191, 700, 1025])
@pytest.mark.parametrize("Hkv,causal", [(2, True), (2, False), (40, True)])
def test_the_next_head_is_not_read(d, N, Hkv, causal):
    import torch
    import paper_2604_12798_amd as vfa
    gen = torch.Generator(device="cuda").manual_seed(N)
    Q, K, V = (torch.randn((1, Hkv, N, d), generator=gen, device="cuda", dtype=torch.bfloat16) for _ in range(3))
    O, L = vfa.vfa_attn_fwd(Q, K, V, causal=causal)
    K[:, 1::2], V[:, 1::2] = float("nan"), float("nan")
    O2, L2 = vfa.vfa_attn_fwd(Q, K, V, causal=causal)
    assert torch.equal(O2[:, ::2], O[:, ::2]) and torch.equal(L2[:, ::2], L[:, ::2])
    assert torch.isfinite(O[:, ::2].float()).all()
