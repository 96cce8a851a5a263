"""Rows whose scores are all -inf: nothing to attend to, so O = 0 and LSE = -inf, as for a row whose every tile was skipped."""
import math

import pytest

pytestmark = pytest.mark.gpu


def _empty(O, L, what):
    import torch
    torch.cuda.synchronize()
    assert (O == 0).all() and torch.isneginf(L).all(), what


# every row's blocks are sink or local ones, where all kernels take the exact max; at 600 rows the others too: vfa_attn_fwd runs on
# attn_short.hpp, vfa_variant_fwd on attn_frozen.hpp
@pytest.mark.parametrize("d,block_m", [(64, 64), (64, 128), (128, 64), (128, 128)])
@pytest.mark.parametrize("B,Hq,Hkv,N,kw", [(1, 4, 2, 128, {}), (2, 32, 8, 100, {}), (1, 32, 2, 300, dict(n_local=4)),
                                          (1, 32, 2, 300, dict(n_local=4, use_minit=False)), (1, 4, 2, 300, dict(n_sink=5)),
                                          (4, 64, 8, 64, dict(causal=False)), (1, 32, 2, 400, dict(n_sink=4, n_local=4)),
                                          (1, 4, 2, 600, {}), (1, 4, 2, 600, dict(use_minit=False))])
def test_bf16(d, block_m, B, Hq, Hkv, N, kw):
    _infinite_feature(d, block_m, B, Hq, Hkv, N, kw)


@pytest.mark.parametrize("block_m", [64, 128])
def test_bf16_d64_one_group_of_keys(block_m):
    _infinite_feature(64, block_m, 1, 64, 8, 600, {})


def _infinite_feature(d, block_m, B, Hq, Hkv, N, kw):
    """KV head 0: an infinite feature in every key.  The other heads are what they are without it."""
    import torch
    import paper_2604_12798_amd as vfa
    gen = torch.Generator(device="cuda").manual_seed(5)
    Q, K, V = (torch.randn((B, h, N, d), generator=gen, device="cuda").bfloat16() for h in (Hq, Hkv, Hkv))
    Q[..., 0] = 1.0
    g = Hq // Hkv
    clean = vfa.vfa_attn_fwd(Q, K, V, block_m=block_m, **kw)
    K[:, 0, :, 0] = -math.inf
    O, L = vfa.vfa_attn_fwd(Q, K, V, block_m=block_m, **kw)
    _empty(O[:, :g], L[:, :g], "vfa")
    assert torch.equal(O[:, g:], clean[0][:, g:]) and torch.equal(L[:, g:], clean[1][:, g:])
    O, L, _ = vfa.vfa_variant_fwd(Q, K, V, block_m=block_m, **kw)
    _empty(O[:, :g], L[:, :g], "vfa_variant")
    assert torch.isfinite(O[:, g:].float()).all() and torch.isfinite(L[:, g:]).all()
    O, L = vfa.fa_baseline_fwd(Q, K, V, block_m=block_m, causal=kw.get("causal", True))
    _empty(O[:, :g], L[:, :g], "fa")
    q = Q[:, :, -1].contiguous()
    for ns in (1, 3):
        O, L = vfa.decode_fwd(q, K, V, N, use_minit=False, n_splits=ns)
        _empty(O[:, :g], L[:, :g], "decode")


@pytest.mark.parametrize("N,n_local", [(64, 1), (100, 1), (300, 4), (500, 1)])
@pytest.mark.parametrize("use_minit", [True, False])
def test_quantised(N, n_local, use_minit):
    """Scores that leave the range of 32 bits downwards: through the descales (8-bit), through the block scales (4-bit)."""
    import torch
    import paper_2604_12798_amd as vfa
    H, d = 2, 128
    V8 = vfa.fp8_pack_v(torch.randn((1, H, N, d), device="cuda").bfloat16(), 1.0)
    fill = lambda c, b: torch.full((1, H, N, c), b, dtype=torch.uint8, device="cuda")
    one, minus_one = fill(d, 0x38), fill(d, 0xB8)  # E4M3
    O, L = vfa.fp8_attn_fwd(one, minus_one, V8, descale_q=1e19, descale_k=1e19, descale_v=1.0, n_local=n_local, use_minit=use_minit)
    _empty(O, L, "8-bit")
    q4, k4, s = fill(d // 2, 0x22), fill(d // 2, 0xAA), fill(d // 32, 200)  # E2M1 1 and -1, both under 2^73
    for scale, noexp in ((0.0, False), (math.log(2.0), False), (math.log(2.0), True)):
        O, L, _ = vfa.mxfp4_attn_fwd(q4, s, k4, s, V8, descale_v=1.0, softmax_scale=scale, noexp=noexp, n_local=n_local, use_minit=use_minit)
        _empty(O, L, "4-bit scale %g noexp %d" % (scale, noexp))
