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


# Alg. 2 on each of its kernels: attn_sparse_kernel, the generic one (d = 64, blocks of 64 rows, five sink blocks) and the ping-pong one
@pytest.mark.parametrize("d,block_m,Hq,Hkv,N,kw", [(128, 128, 4, 2, 600, {}), (128, 128, 4, 2, 1030, dict(causal=False)), (128, 128, 8, 8, 777, dict(n_sink=4, n_local=4)),
                                                  (128, 128, 4, 2, 900, dict(use_minit=False)), (128, 128, 3, 3, 4200, dict(n_sink=0, n_local=0)),
                                                  (128, 128, 4, 2, 600, dict(n_sink=5)), (128, 64, 4, 2, 600, {}), (64, 128, 4, 2, 600, {}),
                                                  (128, 128, 4, 2, 10300, dict(n_sink=5)), (128, 128, 2, 2, 10300, dict(n_sink=5))])
def test_skipping(d, block_m, Hq, Hkv, N, kw):
    """KV head 0: an infinite feature in every key, then in the first half of them only.  A tile without a finite score is dropped, and the
    other heads are what they are without it."""
    import torch
    import paper_2604_12798_amd as vfa
    gen = torch.Generator(device="cuda").manual_seed(6)
    Q, K, V = (torch.randn((1, h, N, d), generator=gen, device="cuda").bfloat16() for h in (Hq, Hkv, Hkv))
    Q[..., 0] = 1.0
    g = Hq // Hkv
    call = lambda k: vfa.vsa_attn_fwd(Q, k, V, block_m=block_m, skip_threshold_nats=2.0, **kw)
    clean = call(K)
    assert torch.isfinite(clean[0].float()).all() and torch.isfinite(clean[1]).all()
    for keys in (N, N // 128 * 64):
        K2 = K.clone()
        K2[:, 0, :keys, 0] = -math.inf
        O, L, M = call(K2)
        r = keys if kw.get("causal", True) else (N if keys == N else 0)  # rows that see nothing else
        _empty(O[:, :g, :r], L[:, :g, :r], "rows without a finite score")
        assert torch.isfinite(O[:, :g, r:].float()).all() and torch.isfinite(L[:, :g, r:]).all()
        # (a tile has a finite score if one of its keys from `keys` on is seen by the block)
        j, i = torch.arange(M.shape[3], device="cuda"), torch.arange(M.shape[2], device="cuda")
        last = torch.clamp((i + 1) * block_m, max=N) - 1 if kw.get("causal", True) else torch.full_like(i, N - 1)
        dropped = (64 * j[None] <= last[:, None]) & ((64 * j[None] + 64 <= keys) | (last[:, None] < keys))
        assert (M[0, :g][dropped.expand(g, -1, -1)] == 1).all()
        assert all(torch.equal(x[:, g:], y[:, g:]) for x, y in zip((O, L, M), clean))
        # the rows behind: exact attention over the other keys, nothing dropped
        if r < N:
            O, L, M = vfa.vsa_attn_fwd(Q, K2, V, block_m=block_m, skip_threshold_nats=1e4, **kw)
            q, k, v = Q[0, 0, N - 64:].double(), K[0, 0, keys:].double(), V[0, 0, keys:].double()
            S = q @ k.T * d ** -0.5
            if kw.get("causal", True):
                S = S.masked_fill(torch.arange(keys, N, device="cuda")[None] > torch.arange(N - 64, N, device="cuda")[:, None], -math.inf)
            P = (S - S.logsumexp(1, keepdim=True)).exp()
            o = P @ v
            assert ((O[0, 0, N - 64:].double() - o).abs() <= 2.0 ** -7 * (P @ v.abs() + o.abs()) + 1e-4).all()


# The keys and values behind a block of rows may hold anything (NaN, as in the padding of a cache), and so may other heads': attn_sparse_kernel
# and the ping-pong kernel
@pytest.mark.parametrize("Hq,Hkv,N,kw", [(4, 2, 777, {}), (6, 3, 1300, dict(n_sink=4, n_local=4)), (2, 2, 1100, dict(n_sink=0, n_local=0)), (4, 2, 10300, dict(n_sink=5))])
def test_skipping_blocks_do_not_see_later_keys(Hq, Hkv, N, kw):
    import torch
    import paper_2604_12798_amd as vfa
    gen = torch.Generator(device="cuda").manual_seed(7)
    Q, K, V = (torch.randn((1, h, N, 128), generator=gen, device="cuda").bfloat16() for h in (Hq, Hkv, Hkv))
    Q *= 2
    call = lambda k, v: vfa.vsa_attn_fwd(Q, k, v, skip_threshold_nats=3.0, **kw)
    O, L, M = call(K, V)
    Tr = -(-N // 128)
    for a in sorted({1, 2, Tr // 2, Tr - 1}):
        K2, V2 = K.clone(), V.clone()
        K2[:, :, 128 * a:], V2[:, :, 128 * a:] = 1e3, float("nan")
        O2, L2, M2 = call(K2, V2)
        assert torch.equal(O2[:, :, :128 * a], O[:, :, :128 * a]) and torch.equal(L2[:, :, :128 * a], L[:, :, :128 * a]), a
        assert torch.equal(M2[:, :, :a], M[:, :, :a]), a
    g = Hq // Hkv
    K[:, 1:], V[:, 1:] = float("nan"), float("nan")
    O2, L2, M2 = call(K, V)
    assert torch.equal(O2[:, :g], O[:, :g]) and torch.equal(L2[:, :g], L[:, :g]) and torch.equal(M2[:, :g], M[:, :g])


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
