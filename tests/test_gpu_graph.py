"""The entry points under HIP graph capture.  The library allocates nothing, records no memset and launches plain
kernels on the caller's stream, so a prefill call and a decode step can be captured once and replayed; every replay,
with the program's own eager work and synchronisations in between, must reproduce the eager result bit for bit."""
import numpy as np
import pytest

from paper_2604_12798_amd import workloads as wl

from gpu_util import gpu_inputs, to_gpu

pytestmark = pytest.mark.gpu


def test_prefill_and_decode_replay_from_a_graph():
    import torch
    import paper_2604_12798_amd as vfa
    vfa.lib()
    w = wl.small(wl.CONFIGS["cfg3"], B=1, Hq=4, Hkv=2, N=2048)
    Q, K, V = gpu_inputs(wl.generate(w, 1))
    dev = Q.device
    kw = dict(block_m=w.block_m, block_n=w.block_n, causal=w.causal, n_sink=w.n_sink, n_local=w.n_local)
    ws = torch.empty(vfa.workspace_bytes(w.B, w.Hkv, w.N, w.d, w.block_n), dtype=torch.uint8, device=dev)
    O, L = torch.empty_like(Q), torch.empty((w.B, w.Hq, w.N), dtype=torch.float32, device=dev)
    Os, Ls = torch.empty_like(Q), torch.empty_like(L)
    M = torch.empty((w.B, w.Hq, w.Tr, w.Tc), dtype=torch.uint8, device=dev)
    q1 = Q[:, :, -1].contiguous()                      # decode: the last token against the whole cache
    n_splits = 4
    R = torch.empty((w.B, w.Hkv, w.Tc, w.d), dtype=torch.bfloat16, device=dev)
    dws = torch.empty(vfa.decode_workspace_bytes(w.B, w.Hq, w.d, n_splits), dtype=torch.uint8, device=dev)
    Od, Ld = torch.empty_like(q1), torch.empty((w.B, w.Hq), dtype=torch.float32, device=dev)

    def step(o, l, os_, ls_, m, od, ld):
        vfa.vfa_attn_fwd(Q, K, V, out=o, lse=l, workspace=ws, **kw)
        vfa.vsa_attn_fwd(Q, K, V, out=os_, lse=ls_, skip_mask=m, workspace=ws, skip_threshold_nats=1.0, **kw)
        vfa.kblock_summary_append(K, R, 0, w.N, w.block_n)
        vfa.decode_fwd(q1, K, V, w.N, krepr=R, n_splits=n_splits, workspace=dws, out=od, lse=ld,
                       n_sink=w.n_sink, n_local=w.n_local)

    step(O, L, Os, Ls, M, Od, Ld)                      # eager once: one-time attribute calls happen outside the capture
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        step(O, L, Os, Ls, M, Od, Ld)
    eo, el = torch.empty_like(O), torch.empty_like(L)
    eos, els, em = torch.empty_like(Os), torch.empty_like(Ls), torch.empty_like(M)
    eod, eld = torch.empty_like(Od), torch.empty_like(Ld)
    for rnd in range(3):
        t = wl.generate(w, 10 + rnd)                   # new inputs into the captured buffers, by ordinary eager copies
        Q.copy_(to_gpu(t["Q"])); K.copy_(to_gpu(t["K"])); V.copy_(to_gpu(t["V"]))
        q1.copy_(Q[:, :, -1])
        for x in (O, L, Os, Ls, Od, Ld):
            x.fill_(float("nan"))
        M.fill_(7)
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        step(eo, el, eos, els, em, eod, eld)           # the same step eagerly, into other outputs
        torch.cuda.synchronize()
        for name, a, b in (("O", O, eo), ("LSE", L, el), ("VSA O", Os, eos), ("VSA LSE", Ls, els), ("mask", M, em),
                           ("decode O", Od, eod), ("decode LSE", Ld, eld)):
            assert torch.equal(a, b), (rnd, name)
        assert int((M == 1).sum().item()) > 0 and not torch.isnan(O.float()).any()


# the warm-up call and the captured one differ in size, blocks, switches, head width and entry point; each pair in a process of its
# own, where no other test has made the library's one-time attribute calls
PAIRS = {
    "d64_many_sinks_first": ("vfa_attn_fwd", 64, dict(N=200, n_sink=5), "vfa_attn_fwd", 64, dict(N=1000)),
    "d128_many_sinks_first": ("vfa_attn_fwd", 128, dict(N=200, n_sink=5, block_m=64), "vfa_attn_fwd", 128, dict(N=777)),
    "vsa_block_m_64_first": ("vsa_attn_fwd", 128, dict(N=200, block_m=64, skip_threshold_nats=4.0),
                             "vsa_attn_fwd", 128, dict(N=10304, skip_threshold_nats=4.0)),
    "variant_ascending_first": ("vfa_variant_fwd", 128, dict(N=200, reorder=False), "vfa_variant_fwd", 128, dict(N=2048)),
    "variant_skipping_last": ("vfa_variant_fwd", 128, dict(N=200), "vfa_variant_fwd", 128, dict(N=10304, skip_threshold_nats=4.0)),
    "baseline_at_d64_first": ("fa_baseline_fwd", 64, dict(N=64, block_m=64), "vfa_attn_fwd", 128, dict(N=4000, n_sink=6, block_m=64)),
}
CHILD = """
import sys, json, torch
import paper_2604_12798_amd as vfa
name1, d1, first, name2, d2, second = json.loads(sys.argv[1])
def call(name, d, N, **kw):
    gen = torch.Generator(device="cuda").manual_seed(N)
    Q, K, V = (torch.randn((1, h, N, d), generator=gen, device="cuda").bfloat16() for h in (4, 2, 2))
    bm = kw.get("block_m", 128)
    ws = torch.empty(vfa.workspace_bytes(1, 2, N, d, 64), dtype=torch.uint8, device="cuda")
    o, l = torch.empty_like(Q), torch.empty((1, 4, N), device="cuda")
    extra = {} if name == "fa_baseline_fwd" else dict(workspace=ws)
    if "skip_threshold_nats" in kw: extra.update(skip_mask=torch.empty((1, 4, -(-N // bm), -(-N // 64)), dtype=torch.uint8, device="cuda"))
    return (lambda: getattr(vfa, name)(Q, K, V, out=o, lse=l, **extra, **kw)), o, l
call(name1, d1, **first)[0]()
torch.cuda.synchronize()
fn, o, l = call(name2, d2, **second)
torch.cuda.synchronize()
g = torch.cuda.CUDAGraph()
with torch.cuda.graph(g):
    fn()
seen = []
for rnd in range(3):
    o.fill_(float("nan")); l.fill_(float("nan"))
    torch.cuda.synchronize()
    g.replay()
    torch.cuda.synchronize()
    seen.append((o.clone(), l.clone()))
fn()
torch.cuda.synchronize()
assert all(torch.equal(a, o) and torch.equal(b, l) for a, b in seen) and torch.isfinite(l).all()
print("captured", name2, flush=True)
"""


@pytest.mark.parametrize("name", PAIRS)
def test_warm_up_call_of_another_kind(name):
    import json
    import os
    import subprocess
    import sys
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    r = subprocess.run([sys.executable, "-c", CHILD, json.dumps(PAIRS[name])], cwd=root, timeout=100, capture_output=True, text=True)
    assert r.returncode == 0 and "captured" in r.stdout, r.stdout + r.stderr


DECODE_CHILD = """
import sys, json, torch
import paper_2604_12798_amd as vfa
B, Hq, Hkv, n, d, ns, ragged = json.loads(sys.argv[1])
gen = torch.Generator(device="cuda").manual_seed(n)
q, K, V = (torch.randn(s, generator=gen, device="cuda").bfloat16() for s in ((B, Hq, d), (B, Hkv, n, d), (B, Hkv, n, d)))
lens = torch.full((B,), n, dtype=torch.int32, device="cuda")
ws = torch.empty(vfa.decode_workspace_bytes(B, Hq, d, ns), dtype=torch.uint8, device="cuda")
o, l = torch.empty_like(q), torch.empty((B, Hq), device="cuda")
kw = dict(use_minit=False, n_splits=ns, workspace=ws, out=o, lse=l)
step = (lambda: vfa.decode_varlen_fwd(q, K, V, lens, **kw)) if ragged else (lambda: vfa.decode_fwd(q, K, V, n, **kw))
torch.cuda.synchronize()
g = torch.cuda.CUDAGraph()
with torch.cuda.graph(g, capture_error_mode="global"):
    step()
for rnd in range(3):
    o.fill_(float("nan")); l.fill_(float("nan"))
    torch.cuda.synchronize()
    g.replay()
    torch.cuda.synchronize()
    S = (K.double()[:, None] * q.double().view(B, Hkv, Hq // Hkv, 1, d).transpose(1, 2)).sum(-1) * d ** -0.5  # [B, g, Hkv, n]
    want = torch.logsumexp(S, -1).transpose(1, 2).reshape(B, Hq)
    assert (l.double() - want).abs().max() <= 1e-3 and torch.isfinite(o.float()).all(), rnd
print("captured", flush=True)
"""


# whole caches (four, two, eight waves to a workgroup) and ranges; the process makes no other call of the library before
@pytest.mark.parametrize("shape", [(1, 8, 2, 300, 128, 5, False), (1, 8, 2, 600, 64, 5, False), (33, 8, 8, 130, 128, 2, False), (1, 8, 2, 2048, 128, 16, False),
                                   (2, 8, 2, 300, 128, 5, True), (2, 8, 2, 2048, 64, 16, True)], ids=str)
def test_first_call_of_a_process_is_a_captured_decode_step(shape):
    import json
    import os
    import subprocess
    import sys
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    r = subprocess.run([sys.executable, "-c", DECODE_CHILD, json.dumps(shape)], cwd=root, timeout=100, capture_output=True, text=True)
    assert r.returncode == 0 and "captured" in r.stdout, r.stdout + r.stderr
