"""GPU parity where the ping-pong kernel runs as persistent workgroups (more work items than CUs) in the
forms the workload list does not reach: one item list for the whole chip (B * Hkv not a multiple of 8),
and a last round that only some workgroups take part in, for head pairs and for block pairs.
Besides the sampled oracle check, every output row must have been written exactly as the other entry
points write it: the two baselines and Alg. 1 compute the same attention, so their outputs have to agree
to rounding everywhere, which a work item that was dropped, done twice or decoded wrongly would break."""
import numpy as np
import pytest

from paper_2604_12798_amd import workloads as wl

from gpu_util import check_o_lse, check_vsa, gpu_inputs, host_f32, vsa_kernel

pytestmark = pytest.mark.gpu

# (name, base config, overrides), but for two over 96 tiles, where vfa_attn_fwd is not on attn_short.hpp: items = B * Hq/2 * Tr (head pairs) or B * Hq * ceil(Tr/2) (block pairs)
CASES = [
    ("chip_list_head_pairs", "cfg3", dict(B=3, Hq=4, Hkv=2, N=6272)),    # B*Hkv = 6: 294 items in one list
    ("xcd_lists_block_pairs", "cfg2", dict(B=1, Hq=8, Hkv=8, N=8448)),   # 8 lists of 33 items: partial round
    ("xcd_lists_head_pairs", "cfg3", dict(B=1, Hq=16, Hkv=8, N=6272)),   # 8 lists of 49 items: partial round
    ("chip_list_ragged", "cfg3", dict(B=1, Hq=6, Hkv=3, N=11300)),       # 267 items, ragged last block
    # (vfa_attn_fwd is on attn_short.hpp, vfa_variant_fwd and the baselines are not)
    ("chip_list_baselines", "cfg3", dict(B=3, Hq=4, Hkv=2, N=5632)),     # 264 items
    ("xcd_lists_baselines", "cfg3", dict(B=1, Hq=16, Hkv=8, N=4480)),    # 8 lists of 35 items
]


@pytest.mark.parametrize("name,base,over", CASES, ids=[c[0] for c in CASES])
def test_persistent_workgroups(oracle, name, base, over):
    import torch
    import paper_2604_12798_amd as vfa
    vfa.lib()
    w = wl.small(wl.CONFIGS[base], **over)
    n_cu = torch.cuda.get_device_properties(0).multi_processor_count
    g = w.Hq // w.Hkv
    items = w.B * (w.Hq // 2) * w.Tr if g % 2 == 0 else w.B * w.Hq * ((w.Tr + 1) // 2)
    assert items > n_cu, "shape no longer exceeds the CU count: the persistent path is not exercised"
    print(f"{name}: {items} items on {n_cu} CUs", flush=True)
    t = wl.generate(w)
    Q, K, V = gpu_inputs(t)
    Qh, Kh, Vh = host_f32(t)
    kw = dict(block_m=w.block_m, block_n=w.block_n, causal=w.causal)
    vkw = dict(n_sink=w.n_sink, n_local=w.n_local, **kw)
    blocks = wl.sample_blocks(w, 6)
    Oe, Le, _ = oracle.exact(Qh, Kh, Vh, w.block_m, w.causal, blocks)
    ref = oracle.blocks(Qh, Kh, Vh, w.block_m, w.block_n, w.causal, blocks, n_sink=w.n_sink, n_local=w.n_local)

    def run(fn, **kws):
        O = torch.full_like(Q, float("nan"))
        L = torch.full((w.B, w.Hq, w.N), float("nan"), dtype=torch.float32, device=Q.device)
        fn(Q, K, V, out=O, lse=L, **kws)
        torch.cuda.synchronize()
        assert not torch.isnan(O.float()).any() and not torch.isnan(L).any(), name + ": rows left unwritten"
        return O, L

    O_fa, L_fa = run(vfa.fa_baseline_fwd, **kw)
    print(name, "fa", check_o_lse(O_fa, L_fa, Oe, Le, blocks, w.block_m, w.N, "fa_baseline_fwd vs exact"), flush=True)
    O_v, L_v = run(vfa.vfa_attn_fwd, **vkw)
    print(name, "vfa", check_o_lse(O_v, L_v, ref["O"], ref["LSE"], blocks, w.block_m, w.N, "vfa_attn_fwd vs oracle"), flush=True)
    O_x, L_x = run(lambda *a, **k: vfa.vfa_variant_fwd(*a, **k)[:2], **vkw)  # (never on attn_short.hpp)
    print(name, "variant", check_o_lse(O_x, L_x, ref["O"], ref["LSE"], blocks, w.block_m, w.N, "vfa_variant_fwd vs oracle"), flush=True)
    assert torch.equal(O_v, O_x) == (w.Tc > 96), "vfa_attn_fwd is on another kernel"
    O_l, L_l = run(vfa.fa_lazy_rescale_fwd, rescale_tau=8.0, **kw)
    # every row, against each other (bf16 outputs of the same attention: a few ulps of bf16 apart at most)
    for what, (Oa, La) in {"vfa": (O_v, L_v), "fa_lazy": (O_l, L_l)}.items():
        do = (Oa.float() - O_fa.float()).abs().max().item()
        dl = (La - L_fa).abs().max().item()
        print(name, what, "vs fa over all rows: max |dO| %.4f max |dLSE| %.2e" % (do, dl), flush=True)
        assert do <= 4e-2 and dl <= 2e-3, (name, what, do, dl)
    # VSA with a threshold nothing reaches: the same attention again, every visited tile kept
    O_s, L_s, M = vfa.vsa_attn_fwd(Q, K, V, skip_threshold_nats=1e4, **vkw)
    torch.cuda.synchronize()
    assert int((M == 1).sum().item()) == 0
    assert (O_s.float() - O_v.float()).abs().max().item() <= 4e-2 and (L_s - L_v).abs().max().item() <= 2e-3


# Alg. 2's ping-pong kernel as persistent workgroups: more than four sink or local blocks and over 10240 tokens (causal) or 5120, both pairings
# with one list per XCD and with one for the whole chip, without a mask and without the summaries' max; thresholds that drop some tiles
VSA_CASES = [
    ("xcd_lists_head_pairs", "cfg3", dict(B=1, Hq=16, Hkv=8, N=10304, n_sink=5), 5.0, True),
    ("chip_list_head_pairs", "cfg3", dict(B=2, Hq=6, Hkv=3, N=10250, n_local=5), 5.0, True),
    ("xcd_lists_block_pairs", "cfg2", dict(B=1, Hq=8, Hkv=8, N=10304, n_sink=6), 4.0, True),
    ("chip_list_block_pairs", "cfg2", dict(B=1, Hq=7, Hkv=7, N=10500, n_sink=5), 4.0, True),
    ("xcd_lists_no_mask", "cfg3", dict(B=1, Hq=16, Hkv=8, N=5200, n_sink=5, causal=False), 5.0, True),
    ("chip_list_no_mask", "cfg3", dict(B=1, Hq=20, Hkv=10, N=5185, n_sink=1, n_local=5, causal=False), 5.0, True),
    ("xcd_lists_no_estimate", "cfg3", dict(B=1, Hq=16, Hkv=8, N=10304, n_sink=5), 5.0, False),
    ("chip_list_no_estimate", "cfg2", dict(B=1, Hq=7, Hkv=7, N=10500, n_sink=5), 4.0, False),
    # the same sizes with one sink and one local block: attn_sparse_kernel
    ("sparse_xcd_lists_16_heads", "cfg3", dict(B=1, Hq=16, Hkv=8, N=10304), 5.0, True),
    ("sparse_one_list_12_heads", "cfg3", dict(B=2, Hq=6, Hkv=3, N=10250), 5.0, True),
    ("sparse_xcd_lists_8_heads", "cfg2", dict(B=1, Hq=8, Hkv=8, N=10304), 4.0, True),
    ("sparse_one_list_7_heads", "cfg2", dict(B=1, Hq=7, Hkv=7, N=10500), 4.0, True),
]


@pytest.mark.parametrize("name,base,over,thr,minit", VSA_CASES, ids=[c[0] for c in VSA_CASES])
def test_persistent_workgroups_vsa(oracle, name, base, over, thr, minit):
    import torch
    import paper_2604_12798_amd as vfa
    w = wl.small(wl.CONFIGS[base], **dict(dict(beta=6.0, kappa=3.0), **over))
    n_cu = torch.cuda.get_device_properties(0).multi_processor_count
    items = w.B * (w.Hq // 2) * w.Tr if (w.Hq // w.Hkv) % 2 == 0 else w.B * w.Hq * ((w.Tr + 1) // 2)
    assert vsa_kernel(w) == ("sparse" if name.startswith("sparse") else "ping-pong") and items > n_cu, "not the persistent form of Alg. 2's ping-pong kernel"
    print(f"{name}: {items} items on {n_cu} CUs", flush=True)
    # blocks of the first round and of the later ones: long, short and the last
    blocks = [(w.B - 1, h, i) for h in sorted({0, w.Hq // 2, w.Hq - 1}) for i in sorted({0, 1, w.Tr // 3, w.Tr - 2, w.Tr - 1})]
    check_vsa(oracle, name, w, thr, blocks, use_minit=minit)
    # every row, where nothing is dropped
    Q, K, V = gpu_inputs(wl.generate(w))
    kw = dict(block_m=w.block_m, block_n=w.block_n, causal=w.causal, n_sink=w.n_sink, n_local=w.n_local, use_minit=minit)
    O_v, L_v = vfa.vfa_attn_fwd(Q, K, V, **kw)
    O = torch.full_like(Q, float("nan"))
    L = torch.full((w.B, w.Hq, w.N), float("nan"), dtype=torch.float32, device=Q.device)
    M = torch.full((w.B, w.Hq, w.Tr, w.Tc), 9, dtype=torch.uint8, device=Q.device)
    vfa.vsa_attn_fwd(Q, K, V, skip_threshold_nats=1e4, out=O, lse=L, skip_mask=M, **kw)
    torch.cuda.synchronize()
    j, i = torch.arange(w.Tc, device=M.device), torch.arange(w.Tr, device=M.device)
    seen = (j[None, :] * w.block_n < torch.clamp((i[:, None] + 1) * w.block_m, max=w.N)) | (not w.causal)
    assert torch.equal(M, torch.where(seen, 0, 2).to(torch.uint8).expand_as(M))
    assert (O.float() - O_v.float()).abs().max().item() <= 4e-2 and (L - L_v).abs().max().item() <= 2e-3
