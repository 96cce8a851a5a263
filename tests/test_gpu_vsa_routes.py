"""Alg. 2 on both sides of the length at which its kernel changes (d = 128, block_m = 128): short sequences run one query
block per workgroup, long ones pairs of heads or of query blocks.  Masks bit-exact outside the guard band around the
threshold, O and LSE at the bars of the other forward tests, every row written."""
import numpy as np
import pytest

from paper_2604_12798_amd import workloads as wl

from gpu_util import MASK_GUARD_NATS, check_o_lse, gpu_inputs, host_f32

pytestmark = pytest.mark.gpu


def W(**kw):
    return wl.small(wl.CONFIGS["cfg3"], **dict(dict(B=1, beta=6.0, kappa=3.0), **kw))


# causal: up to 10240 tokens one block per workgroup; non-causal: up to 5120.  The visit lists of the first query blocks of
# the long causal cases are as short as a short sequence's, those of the last ones hold more than two words of mask bits.
CASES = [
    ("causal_10240", W(Hq=2, Hkv=1, N=10240), 4.0),
    ("causal_10241_head_pairs", W(Hq=4, Hkv=2, N=10241), 5.0),
    ("causal_10300_head_pairs_no_sink", W(Hq=2, Hkv=1, N=10300, n_sink=0, n_local=2), 4.0),
    ("causal_10500_block_pairs", W(Hq=2, Hkv=2, N=10500), 4.0),
    ("causal_10300_three_heads_no_local", W(Hq=3, Hkv=1, N=10300, n_local=0), 4.0),
    ("causal_10500_mha_local2", W(Hq=2, Hkv=2, N=10500, n_local=2), 4.0),
    ("noncausal_5120", W(Hq=2, Hkv=1, N=5120, causal=False), 5.0),
    ("noncausal_5121_head_pairs", W(Hq=2, Hkv=1, N=5121, causal=False), 5.0),
    ("noncausal_5700_head_pairs_sink2", W(Hq=2, Hkv=1, N=5700, causal=False, n_sink=2), 5.0),
    ("noncausal_5700_mha", W(Hq=2, Hkv=2, N=5700, causal=False), 5.0),
    ("generic_64_tiles", W(Hq=1, Hkv=1, N=4096, causal=False), 4.0),
    ("generic_65_tiles", W(Hq=1, Hkv=1, N=4097, causal=False), 4.0),
    ("generic_d64_rows64", W(Hq=2, Hkv=1, N=4200, d=64, F=4, block_m=64), 4.0),
]


# The ping-pong kernel runs a step in a general or in a fast form, chosen per step from the visit list's shape (sink / local visits
# at the head, masked or ragged tiles at the tail, five visits of look-ahead; two steps to a turn of the loop).  Non-causal lengths
# put the same visit count on every query block, so a sweep over consecutive counts with every head of the list walks the start and
# the end of the fast range and its parity; causal ones have every count from one up among their first query blocks.
STEP_FORMS = [("noncausal_tc%d%s_s%dl%d" % (tc, "r" if rag else "", s, l),
               W(Hq=2, Hkv=1, N=64 * tc - rag, causal=False, n_sink=s, n_local=l), thr)
              for tc, rag, s, l, thr in ((81, 0, 1, 1, 5.0), (82, 0, 1, 1, 5.0), (83, 0, 1, 1, 9.0), (84, 0, 0, 1, 5.0), (85, 0, 2, 1, 5.0),
                                         (86, 0, 1, 2, 5.0), (87, 0, 2, 2, 5.0), (82, 17, 1, 1, 5.0), (83, 40, 1, 1, 9.0),
                                         (84, 63, 0, 2, 5.0), (85, 1, 2, 0, 5.0), (88, 0, 1, 0, 5.0), (89, 5, 0, 0, 9.0), (90, 0, 2, 1, 9.0))]
STEP_FORMS += [("causal_%s_%d_s%dl%d" % ("blocks" if Hq == Hkv else "heads", N, s, l), W(Hq=Hq, Hkv=Hkv, N=N, n_sink=s, n_local=l), thr)
               for Hq, Hkv, N, s, l, thr in ((2, 2, 10304, 1, 1, 4.0), (2, 2, 10305, 0, 1, 4.0), (1, 1, 10400, 2, 1, 6.0), (1, 1, 10367, 1, 0, 4.0),
                                             (2, 1, 10304, 1, 1, 4.0), (2, 1, 10345, 2, 2, 4.0), (2, 1, 10432, 0, 1, 6.0), (2, 1, 10305, 2, 0, 4.0))]


@pytest.mark.parametrize("name,w,thr", STEP_FORMS, ids=[c[0] for c in STEP_FORMS])
def test_vsa_step_forms(oracle, name, w, thr):
    assert w.N > (10240 if w.causal else 5120) and w.block_m == 128, "a sequence that the generic kernel takes"
    rows = [0, 1, w.Tr // 2, w.Tr - 2, w.Tr - 1] if not w.causal else [*range(0, 16), w.Tr - 2, w.Tr - 1]
    _check(oracle, name, w, thr, rows)


@pytest.mark.parametrize("name,w,thr", CASES, ids=[c[0] for c in CASES])
def test_vsa_routes(oracle, name, w, thr):
    last = w.Tr - 1
    _check(oracle, name, w, thr, sorted(set([*range(0, 12), last // 2, last - 2, last - 1, last])))


def _check(oracle, name, w, thr, rows):
    import torch
    import paper_2604_12798_amd as vfa
    t = wl.generate(w)
    Q, K, V = gpu_inputs(t)
    Qh, Kh, Vh = host_f32(t)
    blocks = [(0, h, i) for h in range(min(w.Hq, 2)) for i in rows if 0 <= i < w.Tr]
    print(name, flush=True)
    O = torch.full_like(Q, float("nan"))
    L = torch.full((w.B, w.Hq, w.N), float("nan"), dtype=torch.float32, device=Q.device)
    _, _, M = vfa.vsa_attn_fwd(Q, K, V, block_m=w.block_m, block_n=w.block_n, causal=w.causal, n_sink=w.n_sink,
                               n_local=w.n_local, skip_threshold_nats=thr, out=O, lse=L)
    torch.cuda.synchronize()
    assert not torch.isnan(O.float()).any() and not torch.isnan(L).any(), name + ": rows left unwritten"
    ref = oracle.blocks(Qh, Kh, Vh, w.block_m, w.block_n, w.causal, blocks, n_sink=w.n_sink, n_local=w.n_local,
                        vsa=True, skip_threshold_nats=thr)
    got = M.cpu().numpy()
    got = np.stack([got[b, h, i] for b, h, i in blocks])
    near = np.abs(ref["margin"]) < MASK_GUARD_NATS
    assert near.sum() <= 4, "too many tiles sit on the threshold"
    # a tile inside the band may fall either way, and with it what follows in its block
    clean = ~near.any(axis=1)
    assert np.array_equal(got[clean], ref["mask"][clean]), (name, int((got[clean] != ref["mask"][clean]).sum()))
    stats = check_o_lse(O, L, ref["O"][clean], ref["LSE"][clean], np.asarray(blocks)[clean], w.block_m, w.N, name)
    kept, skipped = int((ref["mask"] == 0).sum()), int((ref["mask"] == 1).sum())
    print(name, "kept %d skipped %d" % (kept, skipped), stats, flush=True)
    assert kept > 0 and skipped > 0, "the case should mix kept and skipped tiles"
