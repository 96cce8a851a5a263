"""Key-block summaries at block lengths around the 64, 32 and 16 rows that a wave loads together, and ragged ends: the bits of torch's own maximum."""
import pytest

pytestmark = pytest.mark.gpu


def reference(K, block_n):
    """Per block and feature the element of largest magnitude, the positive one of a tie."""
    import torch
    out = []
    for j in range(0, K.shape[2], block_n):
        k = K[:, :, j:j + block_n].float()
        hi, lo = k.max(2).values, k.min(2).values
        out.append(torch.where(hi.abs() >= lo.abs(), hi, lo))
    return (torch.stack(out, 2) + 0.0).bfloat16()  # (a column of zeros of either sign: +0)


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("N,block_n", [(1, 64), (63, 64), (64, 64), (65, 64), (191, 64), (200, 1), (67, 7), (130, 63), (300, 65), (515, 128), (700, 200), (130, 8), (333, 16), (90, 17), (333, 32),
                                        (200, 33), (500, 96), (300, 97), (600, 160)])
def test_summaries(d, N, block_n):
    import torch
    import paper_2604_12798_amd as vfa
    gen = torch.Generator(device="cuda").manual_seed(1000 * d + N + block_n)
    K = torch.randn((2, 3, N, d), generator=gen, device="cuda").mul(4).round().div(4).bfloat16()  # (many ties of either sign)
    K[0, 0, N // 2, 3] = float("-inf")
    want = reference(K, block_n).view(torch.int16)
    assert torch.equal(vfa.kblock_summary(K, block_n).view(torch.int16), want)
    # grown in three steps, in a cache with more rows
    cap = torch.full((2, 3, N + 70, d), 99.0, dtype=torch.bfloat16, device="cuda")
    cap[:, :, :N] = K
    R = torch.zeros((2, 3, -(-(N + 70) // block_n), d), dtype=torch.bfloat16, device="cuda")
    for a, b in ((0, N // 3), (N // 3, N // 2), (N // 2, N)):
        vfa.kblock_summary_append(cap, R, a, b, block_n)
    assert torch.equal(R[:, :, :want.shape[2]].view(torch.int16), want)
    assert not R[:, :, want.shape[2]:].any()
    lens = lambda *n: torch.tensor(n, dtype=torch.int32, device="cuda")
    R2 = torch.zeros_like(R)
    vfa.kblock_summary_append_varlen(cap, R2, lens(0, 0), lens(N, N // 2), block_n)
    vfa.kblock_summary_append_varlen(cap, R2, lens(N, N // 2), lens(N, N), block_n)
    assert torch.equal(R2, R)


# more rows than the memory-side cache holds: sixteen loaded together at d = 128 (the line and behind it; both appends)
@pytest.mark.parametrize("N", [14336, 14337, 20000])
def test_many_blocks(N):
    import torch
    import paper_2604_12798_amd as vfa
    K = torch.randn((4, 8, N, 128), generator=torch.Generator(device="cuda").manual_seed(N), device="cuda").bfloat16()
    want = reference(K, 64).view(torch.int16)
    assert torch.equal(vfa.kblock_summary(K, 64).view(torch.int16), want)
    lens = lambda n: torch.full((4,), n, dtype=torch.int32, device="cuda")
    for append in (lambda R: vfa.kblock_summary_append(K, R, 0, N, 64), lambda R: vfa.kblock_summary_append_varlen(K, R, lens(0), lens(N), 64)):
        R = torch.zeros((4, 8, -(-N // 64), 128), dtype=torch.bfloat16, device="cuda")
        append(R)
        assert torch.equal(R.view(torch.int16), want)
