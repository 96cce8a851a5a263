"""The kernel that fixes Alg. 1's max before the first softmax (attn_frozen.hpp), at the sizes where its tiles, groups of
keys and staging batches begin and end, against the float64 oracle; bars as in the other parity tests.  On short sequences vfa_attn_fwd
runs on attn_short.hpp, vfa_variant_fwd on this kernel (at d = 128 for up to one block of 128 rows per unit): every call is made of both
(`same`: both run on this one)."""
import numpy as np
import pytest

from paper_2604_12798_amd import workloads as wl

from gpu_util import check_every_row, check_o_lse, gpu_inputs, host_f32

pytestmark = pytest.mark.gpu


def _check(oracle, w, use_minit=True, sample=None, before=None, same=False):
    import torch
    import paper_2604_12798_amd as vfa
    t = wl.generate(w)
    Q, K, V = gpu_inputs(t)
    kw = dict(block_m=w.block_m, causal=w.causal, n_sink=w.n_sink, n_local=w.n_local, use_minit=use_minit)
    outs = {}
    for fn in (vfa.vfa_attn_fwd, vfa.vfa_variant_fwd):
        if before is not None:
            before(vfa)
        O, L = torch.full_like(Q, float("nan")), torch.full(Q.shape[:3], float("nan"), device="cuda")
        fn(Q, K, V, out=O, lse=L, **kw)
        outs[fn.__name__] = O, L
    torch.cuda.synchronize()
    if same:
        assert torch.equal(outs["vfa_attn_fwd"][0], outs["vfa_variant_fwd"][0]), "vfa_attn_fwd is not on this kernel"
    blocks = wl.all_blocks(w) if sample is None else wl.sample_blocks(w, sample)
    ref = oracle.blocks(*host_f32(t), w.block_m, w.block_n, w.causal, blocks, n_sink=w.n_sink, n_local=w.n_local, use_minit=use_minit)
    for name, (O, L) in outs.items():
        assert not torch.isnan(O.float()).any() and not torch.isnan(L).any(), name + ": rows left unwritten"
        check_o_lse(O, L, ref["O"], ref["LSE"], blocks, w.block_m, w.N, name)


def _w(**kw):
    kw.setdefault("F", 4 if kw.get("d") == 64 else 8)
    return wl.small(wl.CONFIGS["cfg2"], **kw)


# one to a few tiles (the second group of keys has none, one less or as many), ragged and whole, both head widths
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("N", [1, 64, 65, 129, 320, 385, 448])
@pytest.mark.parametrize("causal", [True, False])
def test_tile_counts(oracle, d, N, causal):
    _check(oracle, _w(B=2, Hq=16, Hkv=4, N=N, d=d, causal=causal), sample=6)


# d = 64: from a few blocks of 128 rows (two groups of keys) to more than one per unit of a chip of 256 (one group, three workgroups to a
# unit), tile counts even and odd
@pytest.mark.parametrize("B,Hq,N,causal", [(1, 8, 256, True), (1, 8, 257, True), (2, 32, 256, True), (3, 24, 256, False), (1, 8, 576, False),
                                           (1, 8, 577, True), (1, 8, 641, False), (2, 32, 512, True), (2, 32, 513, True), (2, 32, 600, False),
                                           (5, 32, 448, False), (5, 32, 512, True), (5, 32, 513, True), (3, 16, 1536, False),
                                           (3, 16, 1537, False), (3, 16, 1537, True)])
@pytest.mark.parametrize("block_m", [64, 128])
def test_tile_counts_d64(oracle, B, Hq, N, causal, block_m):
    _check(oracle, _w(B=B, Hq=Hq, Hkv=4, N=N, d=64, causal=causal, block_m=block_m), sample=6)


# the sets of blocks whose maxima are taken first: none, overlapping, more than four tiles in all, no estimate from the summaries
@pytest.mark.parametrize("d,block_m", [(64, 64), (64, 128), (128, 64), (128, 128)])
@pytest.mark.parametrize("n_sink,n_local,use_minit", [(0, 0, True), (0, 2, False), (1, 0, False), (3, 1, True), (4, 4, True), (2, 4, False)])
def test_sink_and_local_sets(oracle, d, block_m, n_sink, n_local, use_minit):
    for causal in (True, False):
        _check(oracle, _w(B=1, Hq=8, Hkv=8, N=600, d=d, block_m=block_m, causal=causal, n_sink=n_sink, n_local=n_local),
               use_minit=use_minit, sample=6)


@pytest.mark.parametrize("d", [64, 128])
def test_two_tiles_of_summaries(oracle, d):
    """More than 4096 keys: the summaries fill more than one tile, and the max phase takes more than one batch."""
    _check(oracle, _w(B=1, Hq=2, Hkv=1, N=4180, d=d, n_local=3), sample=6)


def test_three_rounds_without_a_causal_mask(oracle):
    """Between two and three items per compute unit of a 256-unit chip, not causal: the rule's second case at d = 128 (more than twelve
    tiles), and fewer tiles."""
    _check(oracle, _w(B=5, Hq=64, Hkv=8, N=200, causal=False), sample=8)
    _check(oracle, _w(B=1, Hq=48, Hkv=8, N=1500, causal=False), sample=8)


@pytest.mark.parametrize("d", [64, 128])
def test_what_lds_held_before_does_not_matter(oracle, d):
    """The call in front leaves NaN in every tile's memory; the first step multiplies its zero weights with an empty tile."""
    def poison(vfa):
        import torch
        x = torch.full((8, 32, 512, 128), float("nan"), dtype=torch.bfloat16, device="cuda")
        vfa.fa_baseline_fwd(x, x, x, causal=False)
    for b, n in ((1, 64), (1, 200), (1, 520), (1, 600), (6, 200), (6, 520)):  # (six: one group of keys at d = 64)
        _check(oracle, _w(B=b, Hq=32, Hkv=8, N=n, d=d, n_sink=1, n_local=0), sample=6, before=poison)
    for b, hq, n in ((2, 32, 4200), (1, 4, 6272)):  # calls of vfa_attn_fwd on this kernel (the first at d = 64: one group of keys)
        _check(oracle, _w(B=b, Hq=hq, Hkv=hq // 2, N=n, d=d), sample=4, before=poison, same=n == 6272 or d == 64)
    for b, hq, n in ((2, 32, 2113), (1, 4, 4200)):  # of vfa_variant_fwd only
        _check(oracle, _w(B=b, Hq=hq, Hkv=hq // 2, N=n, d=d), sample=4, before=poison)


# calls that are too long for the kernel of short sequences (attn_short.hpp): d = 64 with one group of keys (three workgroups to a unit)
# and with two, d = 128; staging batches of one to eight tiles, no estimate, blocks of 64
@pytest.mark.parametrize("B,Hq,N,d,causal,kw", [(2, 32, 4200, 64, True, {}), (2, 32, 4200, 64, True, dict(n_sink=4, n_local=4)), (2, 32, 2113, 64, False, {}),
                                                (2, 32, 2114, 64, False, dict(n_sink=0, n_local=3)), (1, 4, 6272, 64, True, {}), (1, 4, 6272, 64, False, {}),
                                                (1, 4, 4700, 128, False, {}), (1, 4, 4701, 128, False, dict(n_sink=3, n_local=0)),
                                                (1, 4, 6273, 64, True, {}), (1, 4, 6272, 128, True, {})])
@pytest.mark.parametrize("block_m,use_minit", [(128, True), (64, True), (128, False)])
def test_longer_calls(oracle, B, Hq, N, d, causal, kw, block_m, use_minit):
    _check(oracle, _w(B=B, Hq=Hq, Hkv=4, N=N, d=d, causal=causal, block_m=block_m, **kw), use_minit=use_minit, sample=4, same=True)


# lengths at which vfa_attn_fwd is still on attn_short.hpp and vfa_variant_fwd on this kernel
@pytest.mark.parametrize("B,Hq,N,d,causal,kw", [(2, 32, 2113, 64, True, {}), (2, 32, 2113, 64, True, dict(n_sink=4, n_local=4)), (2, 32, 1600, 64, False, {}),
                                                (2, 32, 1601, 64, False, dict(n_sink=0, n_local=3)), (1, 8, 4200, 64, True, {}), (1, 8, 4200, 64, False, {}),
                                                (1, 8, 2500, 128, False, {}), (1, 8, 2501, 128, False, dict(n_sink=3, n_local=0)),
                                                (1, 4, 4200, 64, True, {}), (1, 4, 4200, 128, True, {})])
@pytest.mark.parametrize("block_m,use_minit", [(128, True), (64, True), (128, False)])
def test_long_calls_of_the_short_kernel(oracle, B, Hq, N, d, causal, kw, block_m, use_minit):
    _check(oracle, _w(B=B, Hq=Hq, Hkv=4, N=N, d=d, causal=causal, block_m=block_m, **kw), use_minit=use_minit, sample=4)


# d = 64, many heads: on both sides of the lines to attn_short.hpp (of a chip of 256 units), and short calls, every row
@pytest.mark.parametrize("B,Hq,N,causal", [(16, 32, 448, False), (16, 32, 449, False), (8, 32, 704, False), (8, 32, 705, False), (4, 36, 1280, False), (4, 36, 1281, False),
                                           (4, 21, 2048, False), (4, 21, 2049, False), (16, 32, 896, True), (16, 32, 897, True), (6, 16, 2944, True), (6, 16, 2945, True),
                                           (4, 16, 3648, True), (4, 16, 3649, True), (5, 32, 960, False), (7, 16, 1025, False), (2, 32, 1345, False),
                                           (16, 32, 960, True), (6, 32, 1600, True), (6, 16, 1792, True), (6, 16, 1856, True)])
def test_many_heads(B, Hq, N, causal):
    import torch
    import paper_2604_12798_amd as vfa
    g = 4 if Hq % 4 == 0 else 3
    gen = torch.Generator(device="cuda").manual_seed(N)
    Q, K, V = (torch.randn((B, h, N, 64), generator=gen, device="cuda", dtype=torch.bfloat16) for h in (Hq, Hq // g, Hq // g))
    Q *= 2
    O, L = torch.full_like(Q, float("nan")), torch.full(Q.shape[:3], float("nan"), device="cuda")
    vfa.vfa_attn_fwd(Q, K, V, causal=causal, out=O, lse=L)
    check_every_row(Q, K, V, O, L, causal)
