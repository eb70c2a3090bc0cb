"""The entry point that allocates nothing (tc_prefill_attn_noalloc): its plan and split-KV partials
live in the library's static workspace instead of allocated buffers.  Same kernels, same plan, so
its output must equal tc_prefill_attn's bit for bit - on two calls in a row, the second with a
smaller batch, which finds whatever the first call left in the workspace."""
import numpy as np
import pytest
import torch

from paper_2601_08743_amd import workloads as W

pytestmark = pytest.mark.gpu


def _case(H, cfg, force_kernel=0):
    wl = W.make_workload(cfg)
    dw = H.DeviceWorkload(wl)
    if force_kernel:
        dw.ctx.tc_set_attn_kernel(force_kernel)
    bt, pl = dw.stitch()
    res = []
    for layer in range(cfg.n_layers):
        q, k, v = (H.to_dev(x, cfg) for x in wl.suffix_qkv(layer))
        ref = torch.full_like(q, float("nan"))
        got = torch.full_like(q, float("nan"))
        dw.ctx.tc_prefill_attn(layer, q, k, v, ref, wl.cu_seqlens, bt, pl, wl.suffix_len, wl.sm_scale)
        splits = dw.ctx.tc_kv_splits()
        dw.ctx.tc_prefill_attn_noalloc(layer, q, k, v, got, wl.cu_seqlens, bt, pl, wl.suffix_len, wl.sm_scale)
        torch.cuda.synchronize()
        assert dw.ctx.tc_kv_splits() == splits
        assert torch.isfinite(ref.float()).all()
        res.append((splits, bool(torch.equal(ref.view(torch.int16), got.view(torch.int16))),
                    float((ref.float() - got.float()).abs().max())))
    # and against the checker, to the bf16 bar, on the last layer
    layer = cfg.n_layers - 1
    want = H.oracle_attn_layer(wl, dw.tables_np, layer, wl.suffix_qkv(layer))
    g64 = H.out_to_f64(got, cfg)
    err = max(float(np.abs(g64[int(wl.cu_seqlens[i]):int(wl.cu_seqlens[i + 1])] - r).max()) for i, r in want.items())
    dw.close()
    return res, err


def test_noalloc_matches_allocating_entry_point():
    import harness as H
    assert torch.cuda.is_available()
    base = W.CONFIGS["c2"]
    big = W.scaled(base, n_layers=2, n_tables=8, tables_per_query=(6, 6), capacity=8)          # P ~ 2.2k, split-KV
    small = W.scaled(base, n_layers=2, n_tables=8, tables_per_query=(2, 2), capacity=8, batch=3,
                     suffix_len=(17, 90), seed=base.seed + 5)                                   # shorter, three queries
    for name, cfg, kern in (("first call (larger)", big, 0), ("second call (smaller)", small, 0),
                            ("general kernel, split", big, 1)):
        res, err = _case(H, cfg, kern)
        print("no-alloc %s: per layer (splits, identical, max diff) %s; vs checker %.3e" % (name, res, err), flush=True)
        assert all(same for _, same, _ in res), res
        assert err <= 1e-2
        if cfg is big:
            assert all(s > 1 for s, _, _ in res), "the case is meant to use split-KV partials"


def test_noalloc_other_kernels():
    """The same through the long-launch kernel (split, so with partials in the workspace) and for a
    decode step (the decode kernels keep one partial per key range there)."""
    import harness as H
    base = W.CONFIGS["c2"]
    big = W.scaled(base, n_layers=1, n_tables=8, tables_per_query=(6, 6), capacity=8)
    res, err = _case(H, big, 4)
    print("no-alloc long-launch kernel: (splits, identical, max diff) %s; vs checker %.3e" % (res, err), flush=True)
    assert all(same for _, same, _ in res) and err <= 1e-2
    # decode: prefill first, then one token per query through both entry points
    cfg = W.scaled(base, n_layers=1, n_tables=8, tables_per_query=(3, 3), capacity=8, batch=3, suffix_len=(5, 40))
    wl = W.make_workload(cfg)
    P = np.array([int(wl.table_len[q].sum()) for q in wl.queries])
    S = wl.suffix_len.astype(int)
    dw = H.DeviceWorkload(wl, seq_blocks=int(sum(-(-(p + s + 1) // 16) for p, s in zip(P, S))) + 4)
    bt, pl = dw.stitch(max_blocks=int(max(-(-(p + s + 1) // 16) for p, s in zip(P, S))) + 1)
    dw.attn_layer(0, bt, pl)
    cur = (P + S).astype(np.int32)
    bt = dw.ctx.tc_grow_seqs(bt, cur + 1)
    rng = np.random.default_rng(3)
    q, k, v = (H.to_dev(W.f32_to_bf16_bits(rng.standard_normal(size=(cfg.batch, h, cfg.head_dim), dtype=np.float32)), cfg)
               for h in (cfg.n_q_heads, cfg.n_kv_heads, cfg.n_kv_heads))
    cu1, one = np.arange(cfg.batch + 1, dtype=np.int32), np.ones(cfg.batch, dtype=np.int32)
    ref, got = torch.full_like(q, float("nan")), torch.full_like(q, float("nan"))
    dw.ctx.tc_prefill_attn(0, q, k, v, ref, cu1, bt, cur, one, wl.sm_scale)
    assert dw.ctx.tc_attn_kernel() == 3 and dw.ctx.tc_kv_splits() > 1
    dw.ctx.tc_prefill_attn_noalloc(0, q, k, v, got, cu1, bt, cur, one, wl.sm_scale)
    torch.cuda.synchronize()
    assert dw.ctx.tc_attn_kernel() == 3
    assert torch.isfinite(ref.float()).all()
    assert torch.equal(ref.view(torch.int16), got.view(torch.int16))
    dw.ctx.tc_release_seqs(bt)
    dw.close()


def _ragged(H, dtype, hq, hkv, D, lens, suffix, kernel, splits=0):
    """One query per table, through both entry points; returns the partition count."""
    cfg = W.WorkloadConfig("n", 1, hq, hkv, D, dtype, len(lens), (1, max(lens)), len(lens), (1, 1), "uniform", (1, 9), len(lens), 317)
    wl = W.make_workload(cfg)
    wl.table_len[:] = lens
    wl.queries[:] = [np.array([i], dtype=np.int32) for i in range(len(lens))]
    wl.suffix_len[:] = suffix
    dw = H.DeviceWorkload(wl)
    dw.ctx.tc_set_kv_splits(splits)
    if kernel == 5:
        dw.ctx.tc_set_attn_kernel(5)
    bt, pl = dw.stitch()
    out, qkv = dw.attn_layer(0, bt, pl)
    assert dw.ctx.tc_attn_kernel() == kernel
    n, got = dw.ctx.tc_kv_splits(), torch.full_like(out, float("nan"))
    dw.ctx.tc_prefill_attn_noalloc(0, *(H.to_dev(x, cfg) for x in qkv), got, wl.cu_seqlens, bt, pl, wl.suffix_len, wl.sm_scale)
    torch.cuda.synchronize()
    assert dw.ctx.tc_attn_kernel() == kernel and dw.ctx.tc_kv_splits() == n
    assert torch.isfinite(out.float()).all() and torch.equal(out, got)
    ref = H.oracle_attn_layer(wl, dw.tables_np, 0, qkv)
    g64 = H.out_to_f64(got, cfg)
    err = max(float(np.abs(g64[int(wl.cu_seqlens[i]):int(wl.cu_seqlens[i + 1])] - r).max()) for i, r in ref.items() if r.size)
    assert err <= (1e-5 if dtype == "f32" else 2.2e-2), err      # as the kernels' own tests: fp32 sums; 8-bit weights and outputs, |v| < 5.5
    dw.close()
    return n


def test_noalloc_ragged_decode():
    """One long sequence among short ones: its many key ranges are its own, the others have one or two (all of them
    as often as the longest would be 20.9 M floats of partials where the workspace has 15.7 M)."""
    import harness as H
    assert _ragged(H, "bf16", 32, 1, 128, [20000] + [300] * 31, [1] * 32, 3) > 100


def test_noalloc_short_launch_and_fp32():
    """Kernels that keep their partials by row: queries in one range (written directly) among cut ones, a query without
    new tokens."""
    import harness as H
    assert _ragged(H, "bf16", 28, 4, 128, [3000, 40, 700, 1500], [5, 3, 0, 20], 5, splits=9) == 9
    assert _ragged(H, "f32", 8, 2, 64, [2100, 30, 500, 900], [23, 1, 0, 40], 0) > 1
    assert _ragged(H, "f32", 32, 8, 128, [7744, 2119], [23, 220], 0) >= 1


def test_noalloc_range_longer_than_the_block_id_table():
    """fp32, 563 key tiles where the kernel keeps the block ids of 512: the partials of two ranges (16.6 M floats) do not fit,
    so the entry point that allocates nothing runs it in one.  Against the other one's two ranges, every row."""
    import harness as H
    cfg = W.WorkloadConfig("n", 1, 32, 1, 128, "f32", 2, (1, 34000), 2, (1, 1), "uniform", (1, 9), 2, 318)
    wl = W.make_workload(cfg)
    wl.table_len[:] = [34000, 70]
    wl.queries[:] = [np.array([0], dtype=np.int32), np.array([1], dtype=np.int32)]
    wl.suffix_len[:] = [2000, 5]
    dw = H.DeviceWorkload(wl)
    bt, pl = dw.stitch()
    dw.ctx.tc_set_kv_splits(1)                   # (the kernel's block-id table still cuts it in two)
    out, qkv = dw.attn_layer(0, bt, pl)
    assert dw.ctx.tc_kv_splits() == 2
    got = torch.full_like(out, float("nan"))
    dw.ctx.tc_prefill_attn_noalloc(0, *(H.to_dev(x, cfg) for x in qkv), got, wl.cu_seqlens, bt, pl, wl.suffix_len, wl.sm_scale)
    torch.cuda.synchronize()
    assert dw.ctx.tc_kv_splits() == 1
    assert torch.isfinite(out).all()
    # the same sums in another order, each within 1e-5 of the exact value (as in the kernel's own tests; the rows of the first
    # query average 34 k values and are far closer)
    assert float((out - got)[:2000].abs().max()) <= 1e-5 and torch.equal(out[2000:], got[2000:])
    dw.close()


def test_noalloc_plan_of_least_space():
    """3302 rows of 313 block ids: with the rows padded to 316 and short-launch items the plan has more integers than the workspace
    (1 Mi), so the 30 queries that bring tokens go through another kernel, over unpadded (odd) table rows."""
    import harness as H
    n, total, blocks = 30, 3302, 313
    cfg = W.WorkloadConfig("n", 1, 4, 1, 128, "bf16", 1, (4992, 4992), n, (1, 1), "uniform", (8, 8), 1, 322)
    wl = W.make_workload(cfg)
    wl.table_len[:] = 4992
    wl.queries[:] = [np.array([0], dtype=np.int32)] * n
    wl.suffix_len[:] = 8
    dw = H.DeviceWorkload(wl)
    bt, pl = dw.stitch(max_blocks=blocks)
    out, qkv = dw.attn_layer(0, bt, pl)
    assert dw.ctx.tc_attn_kernel() == 5
    idle = total - n                             # queries without new tokens, over the first one's blocks
    bt, pl = np.concatenate([bt, np.repeat(bt[:1], idle, axis=0)]), np.concatenate([pl, np.full(idle, 5000, dtype=np.int32)])
    sl = np.concatenate([wl.suffix_len, np.zeros(idle, dtype=np.int32)]).astype(np.int32)
    cu = np.concatenate([[0], np.cumsum(sl)]).astype(np.int32)
    got = torch.full_like(out, float("nan"))
    dw.ctx.tc_prefill_attn_noalloc(0, *(H.to_dev(x, cfg) for x in qkv), got, cu, bt, pl, sl, wl.sm_scale)
    torch.cuda.synchronize()
    assert dw.ctx.tc_attn_kernel() in (1, 2) and dw.ctx.tc_kv_splits() == 1
    ref = H.oracle_attn_layer(wl, dw.tables_np, 0, qkv)
    for o in (out, got):
        g64 = H.out_to_f64(o, cfg)
        assert max(float(np.abs(g64[8 * i:8 * i + 8] - r).max()) for i, r in ref.items()) <= 1e-2
    dw.close()


def test_noalloc_counters_in_the_work_items():
    """A decode step of 64 sequences in four ranges each beside 3097 queries without new tokens, whose table rows leave the plan less room
    than 256 arrival counters take: they are counted in at their work items, with the bits of the counters behind the plan."""
    import harness as H
    n, total, blocks = 64, 3161, 320
    cfg = W.WorkloadConfig("n", 1, 28, 4, 128, "bf16", 8, (600, 640), n, (1, 1), "uniform", (1, 1), 8, 323)
    wl = W.make_workload(cfg)
    dw = H.DeviceWorkload(wl)
    dw.ctx.tc_set_kv_splits(4)
    bt, pl = dw.stitch(max_blocks=blocks)
    out, qkv = dw.attn_layer(0, bt, pl)
    assert dw.ctx.tc_attn_kernel() == 3 and dw.ctx.tc_kv_splits() == 4
    idle = total - n
    bt, pl = np.concatenate([bt, np.repeat(bt[:1], idle, axis=0)]), np.concatenate([pl, np.repeat(pl[:1], idle)])
    sl = np.concatenate([wl.suffix_len, np.zeros(idle, dtype=np.int32)]).astype(np.int32)
    cu = np.concatenate([[0], np.cumsum(sl)]).astype(np.int32)
    dev = [H.to_dev(x, cfg) for x in qkv]
    for _ in range(3):                           # the counters are found at zero again
        got = torch.full_like(out, float("nan"))
        dw.ctx.tc_prefill_attn_noalloc(0, *dev, got, cu, bt, pl, sl, wl.sm_scale)
        torch.cuda.synchronize()
        assert dw.ctx.tc_attn_kernel() == 3 and dw.ctx.tc_kv_splits() == 4
        assert torch.equal(got, out)
    ref = H.oracle_attn_layer(wl, dw.tables_np, 0, qkv)
    g64 = H.out_to_f64(out, cfg)
    assert max(float(np.abs(g64[i:i + 1] - r).max()) for i, r in ref.items()) <= 1e-2
    dw.close()


def test_noalloc_refuses_what_does_not_fit():
    """A batch whose partials exceed the fixed workspace is refused with TC_ERR_CAPACITY and
    enqueues nothing; the allocating entry point still serves it."""
    import harness as H
    from paper_2601_08743_amd import binding as B
    cfg = W.scaled(W.CONFIGS["c5"], n_layers=1, n_tables=12, tables_per_query=(4, 4), capacity=12, batch=48)
    wl = W.make_workload(cfg)
    dw = H.DeviceWorkload(wl)
    dw.ctx.tc_set_kv_splits(4)                 # 48 queries x 8 KV heads x 5 row tiles x 4 partitions: 65 MB of partials
    dw.ctx.tc_set_attn_kernel(1)
    bt, pl = dw.stitch()
    q, k, v = (H.to_dev(x, cfg) for x in wl.suffix_qkv(0))
    out = torch.full_like(q, float("nan"))
    with pytest.raises(B.TcError) as e:
        dw.ctx.tc_prefill_attn_noalloc(0, q, k, v, out, wl.cu_seqlens, bt, pl, wl.suffix_len, wl.sm_scale)
    assert e.value.code == B.TC_ERR_CAPACITY
    torch.cuda.synchronize()
    assert torch.isnan(out.float()).all()      # nothing ran
    dw.ctx.tc_prefill_attn(0, q, k, v, out, wl.cu_seqlens, bt, pl, wl.suffix_len, wl.sm_scale)
    torch.cuda.synchronize()
    assert torch.isfinite(out.float()).all()
    dw.close()
