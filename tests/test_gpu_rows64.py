"""block_m = 64 at d = 128 without skipping: on both sides of each line between items of 64 rows and blocks of 128 (one round of
items and less, a round more, the longest and the shortest sequences of the range), Alg. 1 against its oracle and the
baseline against exact attention, every row written."""
import numpy as np
import pytest

from paper_2604_12798_amd import workloads as wl

from gpu_util import check_o_lse, gpu_inputs, host_f32

pytestmark = pytest.mark.gpu

# (B, Hq, Hkv, N, causal)
SHAPES = [
    (1, 8, 1, 129, True), (1, 64, 8, 192, False), (1, 64, 8, 193, False),   # few items; three and four tiles
    (3, 32, 8, 320, True), (3, 32, 32, 320, False), (6, 32, 32, 320, False),  # odd block counts
    (3, 32, 8, 384, True), (3, 32, 8, 385, True), (4, 32, 8, 320, True),     # an eighth, a quarter over one round
    (3, 32, 32, 640, True), (3, 32, 32, 641, True),                            # ten tiles and eleven
    (1, 32, 8, 768, True), (1, 32, 8, 769, True), (1, 3, 1, 777, False),       # twelve tiles and thirteen
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
                                  ("vfa", vfa.vfa_attn_fwd, ref["O"], ref["LSE"], dict(n_sink=w.n_sink, n_local=w.n_local, **kw))):
        print(what, w.name, B, Hq, Hkv, N, causal, flush=True)
        O = torch.full_like(Q, float("nan"))
        L = torch.full((B, Hq, N), float("nan"), dtype=torch.float32, device=Q.device)
        fn(Q, K, V, out=O, lse=L, **kws)
        torch.cuda.synchronize()
        assert not torch.isnan(O.float()).any() and not torch.isnan(L).any(), what + ": rows left unwritten"
        print(check_o_lse(O, L, Or, Lr, blocks, 64, N, what), flush=True)
        outs.append((O, L))
    # every row of the two, which compute the same attention
    assert (outs[0][0].float() - outs[1][0].float()).abs().max().item() <= 4e-2
    assert (outs[0][1] - outs[1][1]).abs().max().item() <= 2e-3
