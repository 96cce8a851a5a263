"""Alg. 2 at d = 128 in blocks of 128 rows, where its kernel can go wrong: one visible tile, tiles and blocks of one row more and
less, both parities of the tile count, the mask's words of 64 tiles, every count of sink and local blocks that it takes (and five,
which it does not), with and without the summaries' max, both item orders, and the two sides of the line at which short sequences
leave it.  Masks equal the oracle's outside the guard band around the threshold, LSE and the mean error of O are at the bars of
the other forward tests, and every row is written.

The bound on each element of O: a weight is rounded to bf16 (relative error up to 2^-8, the sum in the denominator is not rounded),
so O moves by at most 2^-8 max|V|, and O itself is rounded, 2^-8 |O|.  (A bar of 0.02 for all elements, as elsewhere, is short of
half a step of bf16 plus the weights' share once |O| passes 4: two batches of 6/3 heads have -4.04, which came back as -4.0625.)"""
import numpy as np
import pytest

from paper_2604_12798_amd import workloads as wl

from gpu_util import LSE_ABS, MASK_GUARD_NATS, O_MEAN_ABS, gather_blocks, gpu_inputs, host_f32

pytestmark = pytest.mark.gpu


def W(**kw):
    return wl.small(wl.CONFIGS["cfg3"], **dict(dict(B=1, Hq=2, Hkv=1, beta=6.0, kappa=3.0), **kw))


CASES = [("edge_%d%s" % (n, "c" if c else "n"), W(N=n, causal=c, n_sink=0, n_local=0), 5.0)
         for n in (1, 31, 63, 64, 65, 127, 128, 129, 191, 193, 257) for c in (True, False)]
# one and one: the line is at six tiles (causal) or four (non-causal), and at eighteen with many items
CASES += [("line_%d%s" % (n, "c" if c else "n"), W(N=n, causal=c), 5.0)
          for n, c in ((320, True), (321, True), (384, True), (385, True), (513, True), (640, True), (704, True), (192, False), (193, False),
                       (256, False), (449, False), (512, False))]
CASES += [("many_items_%d" % n, W(Hq=64, Hkv=8, N=n), 5.0) for n in (1151, 1217)]
CASES += [("lists_s%dl%d_%d%s%s" % (s, l, n, "c" if c else "n", "" if m else "_no_minit"), W(N=n, causal=c, n_sink=s, n_local=l), thr, m)
          for s, l, n, c, m, thr in ((4, 4, 1856, True, True, 5.0), (4, 4, 1793, True, True, 5.0), (4, 4, 1029, False, True, 9.0), (4, 0, 900, True, True, 5.0),
                                     (0, 4, 1500, True, False, 4.0), (2, 3, 1337, True, True, 5.0), (3, 2, 1000, False, False, 5.0), (1, 0, 800, True, False, 3.0),
                                     (0, 1, 700, True, False, 2.0), (1, 2, 1100, True, True, 5.0), (2, 1, 1100, False, True, 5.0))]
CASES += [("words_%d%s" % (n, "c" if c else "n"), W(N=n, causal=c), 4.0) for n, c in ((4095, False), (4096, False), (4097, False), (8256, True), (8257, False))]
CASES += [("items_b%d_%d_%d" % (b, hq, hkv), W(B=b, Hq=hq, Hkv=hkv, N=777), 5.0) for b, hq, hkv in ((2, 6, 3), (2, 12, 4), (1, 24, 8), (1, 7, 7), (3, 5, 1))]
# five sink or local blocks: the other kernels, the ping-pong one at these lengths
CASES += [("five_%s_%d" % (k, n), W(Hq=hq, Hkv=1, N=n, n_sink=s, n_local=l), 5.0)
          for k, hq, n, s, l in (("heads", 2, 10345, 5, 2), ("blocks", 1, 10367, 5, 1), ("local", 2, 10305, 1, 5), ("short", 2, 1500, 5, 5))]
CASES = [c if len(c) == 4 else c + (True,) for c in CASES]


@pytest.mark.parametrize("name,w,thr,minit", CASES, ids=[c[0] for c in CASES])
def test_sparse_blocks(oracle, name, w, thr, minit):
    import torch
    import paper_2604_12798_amd as vfa
    t = wl.generate(w)
    Q, K, V = gpu_inputs(t)
    Qh, Kh, Vh = host_f32(t)
    rows = sorted({i for i in [*range(0, 10), w.Tr // 2, w.Tr - 2, w.Tr - 1] if 0 <= i < w.Tr})
    blocks = [(b, h, i) for b in range(w.B) for h in sorted({0, w.Hq - 1}) for i in rows]
    print(name, flush=True)
    kw = dict(block_m=w.block_m, block_n=w.block_n, causal=w.causal, n_sink=w.n_sink, n_local=w.n_local, use_minit=minit, skip_threshold_nats=thr)
    O = torch.full_like(Q, float("nan"))
    L = torch.full((w.B, w.Hq, w.N), float("nan"), dtype=torch.float32, device=Q.device)
    M = torch.full((w.B, w.Hq, w.Tr, -(-w.N // w.block_n)), 9, dtype=torch.uint8, device=Q.device)
    vfa.vsa_attn_fwd(Q, K, V, out=O, lse=L, skip_mask=M, **kw)
    O2, _, M2 = vfa.vsa_attn_fwd(Q, K, V, want_mask=False, want_lse=False, **kw)
    torch.cuda.synchronize()
    assert not torch.isnan(O.float()).any() and not torch.isnan(L).any(), name + ": rows left unwritten"
    assert M2 is None and torch.equal(O, O2), name + ": the mask and the LSE change the result"
    got = M.cpu().numpy()
    assert got.max() <= 2, name + ": tiles of the mask left unwritten"
    ref = oracle.blocks(Qh, Kh, Vh, w.block_m, w.block_n, w.causal, blocks, n_sink=w.n_sink, n_local=w.n_local, use_minit=minit,
                        vsa=True, skip_threshold_nats=thr)
    got = np.stack([got[b, h, i] for b, h, i in blocks])
    near = np.abs(ref["margin"]) < MASK_GUARD_NATS
    clean = ~near.any(axis=1)  # (a tile inside the band may fall either way, and with it what follows in its block)
    assert clean.sum() >= 0.9 * len(clean) - 1, "too many tiles sit on the threshold"
    assert np.array_equal(got[clean], ref["mask"][clean]), (name, int((got[clean] != ref["mask"][clean]).sum()))
    at = np.asarray(blocks)[clean]
    want_o, want_l = ref["O"][clean], ref["LSE"][clean]
    got_o, got_l = gather_blocks(O, at, w.block_m, w.N), gather_blocks(L, at, w.block_m, w.N)
    valid = ~np.isnan(want_l)
    err = np.abs(got_o[valid] - want_o[valid])
    bound = 2.0 ** -8 * (np.abs(want_o[valid]) + np.abs(Vh).max()) + 1e-5
    assert (err <= bound).all(), (name, float((err / bound).max()))
    assert err.mean() <= O_MEAN_ABS and np.abs(got_l[valid] - want_l[valid]).max() <= LSE_ABS, (name, float(err.mean()))
