"""block_m = 64 at d = 128 without skipping: on both sides of each line between items of 64 rows and blocks of 128 (one round of
items and less, a round more, the longest and the shortest sequences of the range), Alg. 1 against its oracle and the
baseline against exact attention, every row written.  (vfa_attn_fwd runs on attn_short.hpp at most of these sizes; vfa_variant_fwd, the same
call with a fixed max, on both sides of the lines.)"""
import numpy as np
import pytest

from paper_2604_12798_amd import workloads as wl

from gpu_util import check_o_lse, gpu_inputs, host_f32

pytestmark = pytest.mark.gpu

# (B, Hq, Hkv, N, causal)
SHAPES = [
    (1, 8, 1, 129, True), (1, 64, 8, 192, False), (1, 64, 8, 193, False),   # few items; three and four tiles
    (1, 64, 8, 256, True), (1, 64, 8, 257, True), (5, 32, 32, 200, True),     # four tiles and five; more than one round of four
    (3, 32, 8, 320, True), (3, 32, 32, 320, False), (6, 32, 32, 320, False),  # odd block counts
    (3, 32, 8, 384, True), (3, 32, 8, 385, True), (4, 32, 8, 320, True),     # an eighth, a quarter over one round
    (2, 32, 8, 640, True), (2, 32, 8, 641, True),                              # ten tiles and eleven
    (3, 32, 32, 640, True), (3, 32, 32, 641, True), (1, 32, 8, 768, True), (1, 32, 8, 769, True),
    (1, 32, 8, 896, False), (1, 32, 8, 897, False),                            # fourteen tiles and fifteen
    (1, 32, 8, 1024, True), (1, 32, 8, 1025, True), (1, 3, 1, 777, False),     # sixteen tiles and seventeen
    (4, 32, 8, 640, True), (4, 32, 8, 641, True),                              # two and a half rounds and more
]


@pytest.mark.parametrize("B,Hq,Hkv,N,causal", SHAPES)
def test_rows64(oracle, B, Hq, Hkv, N, causal):
    import torch
    import paper_2604_12798_amd as vfa
    w = wl.small(wl.CONFIGS["cfg3"], B=B, Hq=Hq, Hkv=Hkv, N=N, block_m=64, causal=causal)
    t = wl.generate(w)
    Q, K, V = gpu_inputs(t)
    Qh, Kh, Vh = host_f32(t)
    blocks = np.unique(np.concatenate([wl.sample_blocks(w, 6), [(B - 1, Hq - 1, w.Tr - 1), (0, 0, 0)]]), axis=0)
    kw = dict(block_m=64, block_n=w.block_n, causal=causal)
    Oe, Le, _ = oracle.exact(Qh, Kh, Vh, 64, causal, blocks)
    ref = oracle.blocks(Qh, Kh, Vh, 64, w.block_n, causal, blocks, n_sink=w.n_sink, n_local=w.n_local)
    outs = []
    for what, fn, Or, Lr, kws in (("fa", vfa.fa_baseline_fwd, Oe, Le, kw),
                                  ("vfa", vfa.vfa_attn_fwd, ref["O"], ref["LSE"], dict(n_sink=w.n_sink, n_local=w.n_local, **kw)),
                                  ("variant", vfa.vfa_variant_fwd, ref["O"], ref["LSE"], dict(n_sink=w.n_sink, n_local=w.n_local, **kw))):
        print(what, w.name, B, Hq, Hkv, N, causal, flush=True)
        O = torch.full_like(Q, float("nan"))
        L = torch.full((B, Hq, N), float("nan"), dtype=torch.float32, device=Q.device)
        fn(Q, K, V, out=O, lse=L, **kws)
        torch.cuda.synchronize()
        assert not torch.isnan(O.float()).any() and not torch.isnan(L).any(), what + ": rows left unwritten"
        print(check_o_lse(O, L, Or, Lr, blocks, 64, N, what), flush=True)
        outs.append((O, L))
    # every row of the three, which compute the same attention
    for O, L in outs[1:]:
        assert (outs[0][0].float() - O.float()).abs().max().item() <= 4e-2
        assert (outs[0][1] - L).abs().max().item() <= 2e-3


# What vfa_attn_fwd runs on at d = 128: attn_short.hpp (n_sink <= 4 and up to 777 rows), the ping-pong kernel in head pairs and in block pairs (n_sink =
# 5), attn_frozen.hpp (6272 rows); at d = 64 attn_short.hpp, the generic kernel (n_sink = 5), attn_frozen.hpp in one group of keys (4200 rows) and in two (6272).
# vfa_variant_fwd, the same call, keeps to the kernels with a fixed max: attn_frozen.hpp for the short ones (2113 and 4200 rows: long calls of attn_short.hpp).
LATER = [(2, 32, 8, 4200, dict(n_sink=1)), (1, 4, 2, 6272, dict(n_sink=1)), (2, 32, 8, 2113, dict(n_sink=1)), (1, 4, 2, 4200, dict(n_sink=1)),
         (1, 8, 2, 777, {}), (1, 4, 2, 1100, dict(n_sink=5)), (1, 3, 1, 1100, dict(n_sink=5)), (1, 3, 3, 1000, dict(n_sink=5, n_local=2)),
         (3, 32, 8, 320, {}), (5, 32, 32, 200, {}), (1, 8, 2, 128, dict(n_sink=0)), (1, 8, 2, 640, dict(n_sink=0, n_local=0))]


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("B,Hq,Hkv,N,kw", LATER)
def test_a_block_of_64_rows_does_not_see_the_next_one(d, B, Hq, Hkv, N, kw):
    """Causal: whatever the keys and values behind a block of 64 rows hold (keys whose estimate would drown every real score, NaN
    in the values, as in the padding of a cache), its rows come out bit for bit the same."""
    import torch
    import paper_2604_12798_amd as vfa
    gen = torch.Generator(device="cuda").manual_seed(7)
    R = lambda *s: torch.randn(s, generator=gen, device="cuda")
    Q, K, V = R(B, Hq, N, d).abs().bfloat16(), R(B, Hkv, N, d).bfloat16(), R(B, Hkv, N, d).bfloat16()
    calls = {"vfa": lambda k, v: vfa.vfa_attn_fwd(Q, k, v, block_m=64, **kw),
             "fa": lambda k, v: vfa.fa_baseline_fwd(Q, k, v, block_m=64),
             "lazy": lambda k, v: vfa.fa_lazy_rescale_fwd(Q, k, v, block_m=64),
             "softexp": lambda k, v: vfa.fa_lazy_rescale_softexp_fwd(Q, k, v, block_m=64)}
    if kw:
        calls = {"vfa": calls["vfa"]}
    calls["variant"] = lambda k, v: vfa.vfa_variant_fwd(Q, k, v, block_m=64, **kw)[:2]
    Tc = -(-N // 64)
    for what, call in calls.items():
        O, L = call(K, V)
        assert torch.isfinite(O.float()).all() and torch.isfinite(L).all()
        for a in sorted({1, 2, Tc // 2 | 1, Tc - 1}):
            if not 0 < a < Tc:
                continue
            print(what, d, B, Hq, Hkv, N, kw, "from block", a, flush=True)
            K2, V2 = K.clone(), V.clone()
            K2[:, :, 64 * a:] = 1e3
            V2[:, :, 64 * a:] = float("nan")
            O2, L2 = call(K2, V2)
            assert torch.equal(O2[:, :, :64 * a], O[:, :, :64 * a]) and torch.equal(L2[:, :, :64 * a], L[:, :, :64 * a]), (what, a)
