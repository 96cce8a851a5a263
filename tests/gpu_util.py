"""Helpers shared by the GPU parity tests: move seeded inputs to the GPU, call the C ABI
through the Python binding, and compare with the float64 oracle at the stated tolerances."""
import numpy as np

from paper_2604_12798_amd import workloads as wl

# parity bars (bf16 path vs float64 oracle)
O_MAX_ABS = 2e-2
O_MEAN_ABS = 2e-3
LSE_ABS = 1e-3
MASK_GUARD_NATS = 1e-3   # tiles whose oracle margin is closer to the threshold than this are not compared


def to_gpu(bits: np.ndarray):
    import torch
    return torch.from_numpy(bits.view(np.int16)).cuda().view(torch.bfloat16)


def gpu_inputs(t: dict):
    return to_gpu(t["Q"]), to_gpu(t["K"]), to_gpu(t["V"])


def host_f32(t: dict):
    return tuple(wl.bf16_bits_to_f32(t[k]) for k in "QKV")


def gather_blocks(x, blocks, block_m, N):
    """x: torch tensor [B,H,N,...] on GPU -> numpy float64 [nblk, block_m, ...], NaN-padded rows."""
    import torch
    xs = x.float().cpu().numpy().astype(np.float64)
    out = np.full((len(blocks), block_m) + xs.shape[3:], np.nan)
    for n, (b, h, i) in enumerate(blocks):
        r0, r1 = i * block_m, min(N, (i + 1) * block_m)
        out[n, : r1 - r0] = xs[b, h, r0:r1]
    return out


def check_o_lse(O_gpu, L_gpu, ref_O, ref_L, blocks, block_m, N, what=""):
    got_O = gather_blocks(O_gpu, blocks, block_m, N)
    got_L = gather_blocks(L_gpu, blocks, block_m, N)
    valid = ~np.isnan(ref_L)
    assert not np.isnan(got_O[valid]).any(), what + ": NaN in O"
    err = np.abs(got_O[valid] - ref_O[valid])
    fin = np.isfinite(ref_L) & valid
    lerr = np.abs(got_L[fin] - ref_L[fin]).max() if fin.any() else 0.0
    assert np.array_equal(np.isneginf(got_L[valid]), np.isneginf(ref_L[valid])), what + ": -inf LSE pattern"
    stats = dict(max_abs=float(err.max()), mean_abs=float(err.mean()), lse=float(lerr))
    assert stats["max_abs"] <= O_MAX_ABS and stats["mean_abs"] <= O_MEAN_ABS and stats["lse"] <= LSE_ABS, (what, stats)
    return stats


def check_every_row(Q, K, V, O, L, causal):
    """All rows of all heads against exact attention in 64 bits, element by element: a weight is off by up to 2^-8 of itself (bf16), so O by
    2^-8 of the same average of |v|, and by 2^-8 of itself for its own rounding (and 1e-4 for the sums in 32 bits)."""
    import torch
    B, Hq, N, d = Q.shape
    for b in range(B):
        for h in range(Hq):
            k, v = K[b, h * K.shape[1] // Hq].double(), V[b, h * K.shape[1] // Hq].double()
            S = Q[b, h].double() @ k.T * d ** -0.5
            if causal:
                S.masked_fill_(torch.ones(N, N, dtype=torch.bool, device=S.device).triu(1), -float("inf"))
            l = S.logsumexp(1)
            P = (S - l[:, None]).exp()
            o = P @ v
            assert ((O[b, h].double() - o).abs() <= 2.0 ** -8 * (P @ v.abs() + o.abs()) + 1e-4).all(), (b, h)
            assert (L[b, h].double() - l).abs().max() <= LSE_ABS, (b, h)


def vsa_kernel(w, n_cu=256):
    """The kernel that vsa_attn_fwd runs a workload on (launch_fwd in vfa_fwd.hip)."""
    if w.d != 128 or w.block_m != 128:
        return "generic"
    if w.n_sink <= 4 and w.n_local <= 4:
        again = max(w.n_sink - 1, 0) + (w.n_local + 1 if w.n_local else 0)
        Tc = -(-w.N // 64)
        if (Tc + 2 if w.causal else 2 * Tc) >= (10 if w.B * w.Hq * w.Tr > 2 * n_cu else 4) * again:
            return "sparse"
    head_pairs = w.Hq // w.Hkv % 2 == 0
    long = w.N > (10240 if w.causal else 5120)
    return "ping-pong" if long and (head_pairs or (w.causal and w.n_local <= 1)) else "generic"


def check_vsa(oracle, name, w, thr, blocks, use_minit=True):
    """vsa_attn_fwd: every row written, masks equal to the oracle's outside the guard band, mean error of O and LSE of the blocks at the bars.
    Each element of O: the usual bar up to |O| = 4, where half a step of bf16 is 2^-7.  Beyond, half a step is 2^-6 and more, and O_MAX_ABS has little
    room for the weights: a weight is rounded to bf16 (up to 2^-8 of it, the sum in the denominator is not rounded), so O moves by at most
    2^-8 max|V|, and O itself is rounded, 2^-8 |O|."""
    import torch
    import paper_2604_12798_amd as vfa
    t = wl.generate(w)
    Q, K, V = gpu_inputs(t)
    Qh, Kh, Vh = host_f32(t)
    print(name, vsa_kernel(w), flush=True)
    O = torch.full_like(Q, float("nan"))
    L = torch.full((w.B, w.Hq, w.N), float("nan"), dtype=torch.float32, device=Q.device)
    _, _, M = vfa.vsa_attn_fwd(Q, K, V, block_m=w.block_m, block_n=w.block_n, causal=w.causal, n_sink=w.n_sink,
                               n_local=w.n_local, use_minit=use_minit, skip_threshold_nats=thr, out=O, lse=L)
    torch.cuda.synchronize()
    assert not torch.isnan(O.float()).any() and not torch.isnan(L).any(), name + ": rows left unwritten"
    ref = oracle.blocks(Qh, Kh, Vh, w.block_m, w.block_n, w.causal, blocks, n_sink=w.n_sink, n_local=w.n_local, use_minit=use_minit,
                        vsa=True, skip_threshold_nats=thr)
    got = M.cpu().numpy()
    got = np.stack([got[b, h, i] for b, h, i in blocks])
    near = np.abs(ref["margin"]) < MASK_GUARD_NATS
    assert near.sum() <= 4, "too many tiles sit on the threshold"
    # a tile inside the band may fall either way, and with it what follows in its block
    clean = ~near.any(axis=1)
    assert np.array_equal(got[clean], ref["mask"][clean]), (name, int((got[clean] != ref["mask"][clean]).sum()))
    at = np.asarray(blocks)[clean]
    want_o, want_l = ref["O"][clean], ref["LSE"][clean]
    got_o, got_l = gather_blocks(O, at, w.block_m, w.N), gather_blocks(L, at, w.block_m, w.N)
    valid = ~np.isnan(want_l)
    err = np.abs(got_o[valid] - want_o[valid])
    size = np.abs(want_o[valid])
    worst = float((err / np.where(size < 4, O_MAX_ABS, 2.0 ** -8 * (size + np.abs(Vh).max()) + 1e-5)).max())
    stats = dict(of_bound=worst, mean_abs=float(err.mean()), lse=float(np.abs(got_l[valid] - want_l[valid]).max()))
    assert worst <= 1 and stats["mean_abs"] <= O_MEAN_ABS and stats["lse"] <= LSE_ABS, (name, stats)
    kept, skipped = int((ref["mask"] == 0).sum()), int((ref["mask"] == 1).sum())
    print(name, "kept %d skipped %d" % (kept, skipped), stats, flush=True)
    assert kept > 0 and skipped > 0, "the case should mix kept and skipped tiles"
