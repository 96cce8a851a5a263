"""Alg. 1 on the kernel for short sequences (attn_short.hpp) at the edges of its chunks of 32 keys, steps and items, and on the rows that
do not fill a round of the ping-pong kernel, against the float64 oracle; bars as in the other parity tests."""
import pytest

from paper_2604_12798_amd import workloads as wl

from gpu_util import check_every_row, check_o_lse, gpu_inputs, host_f32

pytestmark = pytest.mark.gpu


def _w(**kw):
    kw.setdefault("F", 4 if kw.get("d") == 64 else 8)
    return wl.small(wl.CONFIGS["cfg2"], **kw)


def _check(oracle, w, sample, **kw):
    import torch
    import paper_2604_12798_amd as vfa
    t = wl.generate(w)
    Q, K, V = gpu_inputs(t)
    ws = torch.zeros(vfa.workspace_bytes(w.B, w.Hkv, w.N, w.d, 64), dtype=torch.uint8, device="cuda")
    O, L = vfa.vfa_attn_fwd(Q, K, V, block_m=w.block_m, causal=w.causal, workspace=ws, **kw)
    R = vfa.kblock_summary(K)
    torch.cuda.synchronize()
    assert torch.equal(ws[:2 * R.numel()].view(torch.bfloat16), R.flatten())
    blocks = wl.sample_blocks(w, sample)
    ref = oracle.blocks(*host_f32(t), w.block_m, w.block_n, w.causal, blocks)
    check_o_lse(O, L, ref["O"], ref["LSE"], blocks, w.block_m, w.N, w.name)


# two groups of keys: chunks, steps of 64 keys, items of 64 rows; heads in eights or not
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("N", [1, 31, 32, 33, 64, 65, 95, 97, 128, 129, 193, 448, 513])
@pytest.mark.parametrize("causal", [True, False])
def test_two_groups(oracle, d, N, causal):
    _check(oracle, _w(B=2, Hq=8, Hkv=4, N=N, d=d, causal=causal), 6)
    _check(oracle, _w(B=1, Hq=6, Hkv=3, N=N, d=d, causal=causal, block_m=64), 6)


# four groups (from ten tiles on): steps of 128 keys, also where the last step has keys for some of the groups only
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("N", [577, 609, 640, 641, 672, 705, 767, 1025])
@pytest.mark.parametrize("causal", [True, False])
def test_four_groups(oracle, d, N, causal):
    _check(oracle, _w(B=1, Hq=8, Hkv=1, N=N, d=d, causal=causal), 6)


# the last rows of a call (32 heads: a round of the ping-pong kernel on 256 units is 2048 rows of each): one row, up to 512 in items of 64,
# up to 1024 on attn_frozen.hpp; pairs of heads, pairs of blocks.  Every row of every head, on both sides of the seam
@pytest.mark.parametrize("Hkv", [8, 32])
@pytest.mark.parametrize("N", [2049, 2113, 2560, 2561, 3000])
def test_last_rows(Hkv, N):
    import torch
    import paper_2604_12798_amd as vfa
    Q, K, V = gpu_inputs(wl.generate(_w(B=1, Hq=32, Hkv=Hkv, N=N, causal=False)))
    O, L = torch.full_like(Q, float("nan")), torch.full(Q.shape[:3], float("nan"), device="cuda")
    vfa.vfa_attn_fwd(Q, K, V, causal=False, out=O, lse=L)
    check_every_row(Q, K, V, O, L, False)


@pytest.mark.parametrize("d", [64, 128])
def test_what_lds_held_before_does_not_matter(oracle, d):
    import torch
    import paper_2604_12798_amd as vfa
    x = torch.full((8, 32, 512, 128), float("nan"), dtype=torch.bfloat16, device="cuda")
    for n in (20, 64, 200, 700):
        vfa.fa_baseline_fwd(x, x, x, causal=False)
        _check(oracle, _w(B=1, Hq=8, Hkv=8, N=n, d=d), 6)


@pytest.mark.parametrize("d,B,Hq,N", [(64, 1, 8, 256), (128, 1, 8, 256), (64, 1, 4, 700), (128, 1, 4, 700), (128, 2, 16, 448)])
@pytest.mark.parametrize("causal", [True, False])
def test_large_values(d, B, Hq, N, causal):
    """Scores that rise by 7.5 binades behind a wave's first keys, too little for it to move its max, and values near the largest of 32
    bits divided by the keys: a weight above 1 would overflow their sums, which exact attention's do not."""
    import torch
    import paper_2604_12798_amd as vfa
    Q, K = torch.zeros((B, Hq, N, d), device="cuda"), torch.zeros((B, Hq, N, d), device="cuda")
    Q[..., 0], K[:, :, N // 4:, 0] = 8.0, 1.0
    V = torch.full((B, Hq, N, d), 1e35, device="cuda").bfloat16()
    scale = 7.5 * 0.6931471805599453 / 8
    O, L = vfa.vfa_attn_fwd(Q.bfloat16(), K.bfloat16(), V, causal=causal, softmax_scale=scale)
    S = torch.where(torch.arange(N, device="cuda") < N // 4, 0.0, 8.0 * scale).double().expand(N, N)
    if causal:
        S = S.masked_fill(torch.ones(N, N, dtype=torch.bool, device="cuda").triu(1), -float("inf"))
    # all values are alike, so O is that value, but for the weights' rounding against their sum and its own: 2^-8 each
    assert ((O.double() / V.double() - 1).abs() <= 2.0 ** -7).all()
    assert (L.double() - S.logsumexp(1)).abs().max() <= 1e-3


# more heads of one token than a launch of 256 threads each can have workgroups (2^24); d = 128: pairs of heads, an odd number to a KV
# head; d = 64: the workgroups of blocks of 64 rows have 128 threads
@pytest.mark.parametrize("Hq,d,block_m", [(258, 128, 64), (257, 128, 128), (257, 64, 64)])
def test_very_many_heads_of_one_token(Hq, d, block_m):
    import torch
    import paper_2604_12798_amd as vfa
    B = 65528
    gen = torch.Generator(device="cuda").manual_seed(Hq)
    R = lambda h: torch.randn((B, h, 1, d), generator=gen, device="cuda", dtype=torch.bfloat16)
    Q, K, V = R(Hq), R(1), R(1)
    O, L = torch.full_like(Q, float("nan")), torch.full((B, Hq, 1), float("nan"), device="cuda")
    vfa.vfa_attn_fwd(Q, K, V, block_m=block_m, out=O, lse=L)
    # one key: its value, bit for bit (a weight that rounds to a power of two, divided by itself), and its score
    assert all((O[b:b + 4096] == V[b:b + 4096]).all() for b in range(0, B, 4096))
    for b in range(0, B, 4096):
        s = (Q[b:b + 4096, :, 0].float() @ K[b:b + 4096, 0, 0, :, None].float())[..., 0] * d ** -0.5
        assert (L[b:b + 4096, :, 0] - s).abs().max() <= 1e-3


def test_more_workgroups_than_a_launch_can_have_is_an_error():
    """Where no kernel covers that many heads the call fails and writes nothing (HIP would run a part of the launch, without an error)."""
    import torch
    import paper_2604_12798_amd as vfa
    B, Hq, d = 65528, 257, 64
    Q, K = torch.zeros((B, Hq, 1, d), device="cuda", dtype=torch.bfloat16), torch.zeros((B, 1, 1, d), device="cuda", dtype=torch.bfloat16)
    O, L = torch.full_like(Q, 7.0), torch.full((B, Hq, 1), 7.0, device="cuda")
    for call in (vfa.vfa_attn_fwd, vfa.fa_baseline_fwd):
        with pytest.raises(vfa.VfaError):
            call(Q, K, K, block_m=128, out=O, lse=L)
    q8, k8 = (torch.zeros((B, h, 1, 128), device="cuda", dtype=torch.uint8) for h in (Hq, 1))
    v8 = torch.zeros((B, 1, 1, 128, 64), device="cuda", dtype=torch.uint8)
    O8 = torch.full(q8.shape, 7.0, device="cuda", dtype=torch.bfloat16)
    with pytest.raises(vfa.VfaError):
        vfa.fp8_attn_fwd(q8, k8, v8, descale_q=1.0, descale_k=1.0, descale_v=1.0, out=O8, lse=L)
    torch.cuda.synchronize()
    assert (O == 7).all() and (L == 7).all() and (O8 == 7).all()
