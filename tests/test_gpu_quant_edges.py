"""The quantising pre-passes at the edges of a workgroup's share (8192 elements), on values of every kind, byte for byte against
the oracle's codecs; and the 8-bit attention kernels' max phase (tiles of summaries, sink and local tiles, four at a time) where
it takes more than one batch, no summaries, or more than one tile of them."""
import math

import numpy as np
import pytest

from paper_2604_12798_amd import workloads as wl

from gpu_util import gpu_inputs, host_f32, to_gpu

pytestmark = pytest.mark.gpu


def _values(n):
    """bf16 patterns: every magnitude around the rounding ties of both formats, zeros of both signs, huge and tiny ones."""
    rng = np.random.default_rng(n)
    x = rng.standard_normal(n) * 2.0 ** rng.integers(-6, 6, n)
    x[::7] = rng.choice([0.0, -0.0, 0.25, 0.75, 1.25, 1.75, 2.5, 3.5, 5.0, -5.0, 6.0, 448.0, 464.0, 1e30, -1e-30], x[::7].shape)
    return wl.f32_to_bf16_bits(x.astype(np.float32))


@pytest.mark.parametrize("n", [32, 8160, 8192, 8224, 16416])
def test_quantisers_at_the_edges_of_a_workgroup(oracle, n):
    import torch
    import paper_2604_12798_amd as vfa
    bits = _values(n)
    x, xh = to_gpu(bits), wl.bf16_bits_to_f32(bits)
    assert np.array_equal(vfa.fp8_quantize(x, 0.5).cpu().numpy(), oracle.e4m3_quantize(xh, 0.5))
    for pre in (1.0, 0.1275):
        codes, scales = vfa.mxfp4_quantize(x.view(-1, 32), pre)
        want_c, want_s = oracle.mx_quantize(xh.reshape(-1, 32), 0, pre)
        assert np.array_equal(codes.cpu().numpy(), want_c) and np.array_equal(scales.cpu().numpy(), want_s)
    # a NaN takes the code of zero with its sign (and no part in the block's scale)
    nan = torch.full((1, 32), float("nan"), dtype=torch.bfloat16, device="cuda")
    nan[0, 1] = 3.0
    codes, scales = vfa.mxfp4_quantize(nan)
    assert int(scales[0, 0]) == 126 and (codes.cpu().numpy().view(np.uint8) & 0x77)[0, 1:].max() == 0 and int(codes[0, 0]) >> 4 == 7


@pytest.mark.parametrize("n", [1 << 22, (1 << 22) + 32, (1 << 26) - 32, 1 << 26, (1 << 26) + 32])
def test_quantisers_of_large_arrays(n):
    """Runs per thread and the kind of load change with the size: the same bytes as from small pieces."""
    import torch
    import paper_2604_12798_amd as vfa
    gen = torch.Generator(device="cuda").manual_seed(n)
    X = (torch.randn(n, generator=gen, device="cuda") * 3).bfloat16()
    pieces = torch.split(X, 1 << 20)
    assert torch.equal(vfa.fp8_quantize(X, 0.7), torch.cat([vfa.fp8_quantize(p, 0.7) for p in pieces]))
    got, want = vfa.mxfp4_quantize(X, 1.3), [vfa.mxfp4_quantize(p, 1.3) for p in pieces]
    assert torch.equal(got[0], torch.cat([w[0] for w in want])) and torch.equal(got[1], torch.cat([w[1] for w in want]))


@pytest.mark.parametrize("N,causal,n_sink,n_local,use_minit", [
    (1, True, 1, 1, True), (129, True, 4, 3, True), (700, False, 5, 6, False), (640, True, 2, 1, False), (4230, True, 1, 2, True)])
@pytest.mark.parametrize("path", ["fp8", "fp8_fold", "mxfp4", "mxfp4_fold"])
def test_max_phase_sets(oracle, path, N, causal, n_sink, n_local, use_minit):
    import torch
    import paper_2604_12798_amd as vfa
    w = wl.small(wl.CONFIGS["cfg2"], B=1, Hq=2, Hkv=1, N=N, causal=causal, n_sink=n_sink, n_local=n_local)
    t = wl.generate(w)
    Q, K, V = gpu_inputs(t)
    Qh, Kh, Vh = host_f32(t)
    p2 = lambda x: 2.0 ** math.ceil(math.log2(float(np.abs(x).max()) / 448.0))
    kw = dict(causal=causal, n_sink=n_sink, n_local=n_local, use_minit=use_minit)
    sv, scale = p2(Vh), 1.0 / math.sqrt(w.d)
    V8, Vd = vfa.fp8_pack_v(V, 1 / sv), oracle.e4m3_dequantize(oracle.e4m3_quantize(Vh, 1 / sv), sv)
    if path.startswith("fp8"):
        sk = p2(Kh)
        rest = sk * scale * math.log2(math.e)
        sq = float(np.float32(2.0 ** math.ceil(math.log2(float(np.abs(Qh).max()) / 448.0 * rest)) / rest)) if path == "fp8_fold" else p2(Qh)
        O, L = vfa.fp8_attn_fwd(vfa.fp8_quantize(Q, 1 / sq), vfa.fp8_quantize(K, 1 / sk), V8, descale_q=sq, descale_k=sk, descale_v=sv, **kw)
        Qd, Kd = (oracle.e4m3_dequantize(oracle.e4m3_quantize(x, 1 / s), s) for x, s in ((Qh, sq), (Kh, sk)))
        bound = 2.0 ** -4  # E4M3 weights: half a unit of three mantissa bits each, of one sign at worst
    else:
        pre = float(np.float32(scale) * np.float32(math.log2(math.e))) if path == "mxfp4_fold" else 1.0
        Q4, QS = vfa.mxfp4_quantize(Q, pre)
        K4, KS = vfa.mxfp4_quantize(K)
        scale = math.log(2.0) if path == "mxfp4_fold" else scale
        O, L, _ = vfa.mxfp4_attn_fwd(Q4, QS, K4, KS, V8, descale_v=sv, softmax_scale=scale, **kw)
        Qd, Kd = oracle.mx_dequantize(*oracle.mx_quantize(Qh, 0, pre)), oracle.mx_dequantize(*oracle.mx_quantize(Kh, 0))
        bound = 2.0 ** -3  # E5M2 weights
    torch.cuda.synchronize()
    o, l = O.float().cpu().numpy()[0], L.cpu().numpy()[0]
    rows = np.unique(np.linspace(0, N - 1, 40).astype(int))
    Qd, Kd, Vd = (np.asarray(x, np.float64)[0] for x in (Qd, Kd, Vd))
    for h in range(2):
        s = Qd[h, rows] @ Kd[0].T * scale
        if causal:
            s[np.arange(N)[None, :] > rows[:, None]] = -np.inf
        m = s.max(1, keepdims=True)
        p = np.exp(s - m)
        ref = p @ Vd[0] / p.sum(1, keepdims=True)
        # (and the bf16 output: half a unit of eight bits)
        assert np.abs(o[h, rows] - ref).max() <= (bound + 2.0 ** -8) * np.abs(Vd).max()
        assert np.abs(l[h, rows] - (m[:, 0] + np.log(p.sum(1)))).max() <= 1e-3
