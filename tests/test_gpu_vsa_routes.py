"""Alg. 2 at d = 128, block_m = 128 on each of its kernels: up to four sink and four local blocks on attn_sparse_kernel, more of them on the
generic kernel and, on long sequences, on the ping-pong kernel in pairs of heads or of query blocks.  Masks bit-exact outside the guard band
around the threshold, O and LSE at the bars of the other forward tests, every row written."""
import dataclasses

import pytest

from paper_2604_12798_amd import workloads as wl

from gpu_util import check_vsa, vsa_kernel

pytestmark = pytest.mark.gpu


def W(**kw):
    return wl.small(wl.CONFIGS["cfg3"], **dict(dict(B=1, beta=6.0, kappa=3.0), **kw))


# The lengths at which the kernels for more than four sink or local blocks change: causal 10240 tokens, non-causal 5120.  The visit lists of
# the first query blocks of the long causal cases are as short as a short sequence's, those of the last ones hold more than two words of mask bits.
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


def more(w):
    """With five sink blocks, or more, in front (five local ones where there was no sink and pairs of heads allow it)."""
    if w.n_sink == 0 and w.Hq // w.Hkv % 2 == 0:
        return dataclasses.replace(w, n_local=w.n_local + 4 if w.n_local else 5)
    return dataclasses.replace(w, n_sink=w.n_sink + 5)


# The kernel of each: as they are, and with more than four sink or local blocks
KERNELS = {"causal_10240": ("sparse", "generic"), "noncausal_5120": ("sparse", "generic"), "causal_10500_mha_local2": ("sparse", "generic"),
           "noncausal_5700_mha": ("sparse", "generic"), "generic_64_tiles": ("sparse", "generic"), "generic_65_tiles": ("sparse", "generic"),
           "generic_d64_rows64": ("generic", "generic")}

# The ping-pong kernel runs a step in a general or in a fast form, chosen per step from the visit list's shape (sink / local visits
# at the head, masked or ragged tiles at the tail, five visits of look-ahead; two steps to a turn of the loop).  Non-causal lengths
# put the same visit count on every query block, so a sweep over consecutive counts with every head of the list walks the start and
# the end of the fast range and its parity; causal ones have every count from one up among their first query blocks.  The same sweep as it is
# walks attn_sparse_kernel's two-step loop.
STEP_FORMS = [("noncausal_tc%d%s_s%dl%d" % (tc, "r" if rag else "", s, l),
               W(Hq=2, Hkv=1, N=64 * tc - rag, causal=False, n_sink=s, n_local=l), thr)
              for tc, rag, s, l, thr in ((81, 0, 1, 1, 5.0), (82, 0, 1, 1, 5.0), (83, 0, 1, 1, 9.0), (84, 0, 0, 1, 5.0), (85, 0, 2, 1, 5.0),
                                         (86, 0, 1, 2, 5.0), (87, 0, 2, 2, 5.0), (82, 17, 1, 1, 5.0), (83, 40, 1, 1, 9.0),
                                         (84, 63, 0, 2, 5.0), (85, 1, 2, 0, 5.0), (88, 0, 1, 0, 5.0), (89, 5, 0, 0, 9.0), (90, 0, 2, 1, 9.0))]
STEP_FORMS += [("causal_%s_%d_s%dl%d" % ("blocks" if Hq == Hkv else "heads", N, s, l), W(Hq=Hq, Hkv=Hkv, N=N, n_sink=s, n_local=l), thr)
               for Hq, Hkv, N, s, l, thr in ((2, 2, 10304, 1, 1, 4.0), (2, 2, 10305, 0, 1, 4.0), (1, 1, 10400, 2, 1, 6.0), (1, 1, 10367, 1, 0, 4.0),
                                             (2, 1, 10304, 1, 1, 4.0), (2, 1, 10345, 2, 2, 4.0), (2, 1, 10432, 0, 1, 6.0), (2, 1, 10305, 2, 0, 4.0))]


@pytest.mark.parametrize("kernel", ["sparse", "ping-pong"])
@pytest.mark.parametrize("name,w,thr", STEP_FORMS, ids=[c[0] for c in STEP_FORMS])
def test_vsa_step_forms(oracle, name, w, thr, kernel):
    if kernel == "ping-pong":
        w = more(w)
        if w.Hq == w.Hkv and w.n_local > 1:
            w = dataclasses.replace(w, n_local=1)  # (pairs of blocks take one local block at most)
    assert vsa_kernel(w) == kernel
    rows = [0, 1, w.Tr // 2, w.Tr - 2, w.Tr - 1] if not w.causal else [*range(0, 16), w.Tr - 2, w.Tr - 1]
    check_vsa(oracle, name, w, thr, _blocks(w, rows))


@pytest.mark.parametrize("many", [False, True])
@pytest.mark.parametrize("name,w,thr", CASES, ids=[c[0] for c in CASES])
def test_vsa_routes(oracle, name, w, thr, many):
    w = more(w) if many else w
    assert vsa_kernel(w) == KERNELS.get(name, ("sparse", "ping-pong"))[many]
    last = w.Tr - 1
    check_vsa(oracle, name, w, thr, _blocks(w, sorted(set([*range(0, 12), last // 2, last - 2, last - 1, last]))))


def _blocks(w, rows):
    return [(0, h, i) for h in range(min(w.Hq, 2)) for i in rows if 0 <= i < w.Tr]
