"""Launches that combine the partials of cut key ranges, inside the launch (arrival counters, which every launch leaves at zero) or by
a merge launch, captured into a HIP graph and replayed with eager calls of the same plan and of others in between."""
import numpy as np
import pytest
import torch

from paper_2601_08743_amd import workloads as W

pytestmark = pytest.mark.gpu

# (dtype, query heads, KV heads, head dim, suffix, forced kernel, partitions, kernel of the plan)
CASES = [("bf16", 28, 4, 128, 17, 5, 7, 5), ("bf16", 28, 4, 128, 17, 5, 12, 5), ("bf16", 28, 4, 128, 1, 0, 12, 3),
         ("bf16", 32, 1, 128, 1, 0, 12, 3), ("f32", 8, 2, 64, 20, 0, 6, 0), ("f32", 8, 2, 128, 20, 0, 6, 0), ("bf16", 28, 4, 128, 100, 4, 3, 4)]


@pytest.mark.parametrize("dtype,hq,hkv,d,suffix,kernel,splits,plan", CASES)
def test_replays_match_eager(dtype, hq, hkv, d, suffix, kernel, splits, plan):
    import harness as H
    cfg = W.WorkloadConfig("g", 2, hq, hkv, d, dtype, 4, (300, 420), 3, (2, 3), "uniform", (suffix, suffix), 4, 337)
    wl = W.make_workload(cfg)
    dw = H.DeviceWorkload(wl)
    dw.ctx.tc_set_attn_kernel(kernel)
    dw.ctx.tc_set_kv_splits(splits)
    stream = torch.cuda.Stream()
    qkv = [tuple(H.to_dev(x, cfg) for x in wl.suffix_qkv(l)) for l in range(2)]
    outs = [torch.zeros_like(qkv[l][0]) for l in range(2)]

    def layers(bt, pl):
        for l in range(2):
            dw.ctx.tc_prefill_attn(l, *qkv[l], outs[l], wl.cu_seqlens, bt, pl, wl.suffix_len, wl.sm_scale, stream)

    bt, pl = dw.stitch(stream=stream)
    layers(bt, pl)
    torch.cuda.synchronize()
    assert dw.ctx.tc_attn_kernel() == plan and dw.ctx.tc_kv_splits() == splits
    eager = [o.clone() for o in outs]
    ref = H.oracle_attn_layer(wl, dw.tables_np, 1, wl.suffix_qkv(1))
    got = H.out_to_f64(outs[1], cfg)
    for i, r in ref.items():                 # 8 bits of a weight and of the output, values up to 5.5; fp32: sums of a thousand terms
        err = float(np.abs(got[int(wl.cu_seqlens[i]):int(wl.cu_seqlens[i + 1])] - r).max())
        assert err <= (2.2e-2 if dtype == "bf16" else 1e-5), (i, err)
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=stream):
        layers(bt, pl)
    for rep in range(4):
        if rep % 2:
            layers(bt, pl)                   # the same plan, eagerly
        for o in outs:
            o.fill_(float("nan"))
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        assert all(torch.equal(o, e) for o, e in zip(outs, eager)), rep
    dw.close()
