"""The fp32 attention kernel at the sizes where it can go wrong: units of 32 keys that end the prefix,
straddle prefix and suffix or lie wholly in the suffix; row tiles of 32 that are ragged; ranges with fewer
units than waves; causal ends inside a split; key ranges longer than the block-id table.  Against the
fp64 checker on every row, the pool bit for bit."""
import numpy as np
import pytest

from paper_2601_08743_amd import workloads as W

pytestmark = pytest.mark.gpu

# Sums of n products of O(1) terms in fp32: |error| <= n * 2^-24 * sum|terms| in the worst case; with weights that
# sum to 1 and |v| < 5.5 the random-walk size is sqrt(n) * 2^-24 * 5.5 < 1e-5 up to n = 900 equal terms, and longer
# rows average the values down (outputs ~ 1/sqrt(n)).
TOL = 1e-5


@pytest.fixture(scope="module")
def H():
    import harness
    return harness


def _run(H, D, hq, hkv, lens, queries, suffix, splits):
    cfg = W.WorkloadConfig("f", 2, hq, hkv, D, "f32", len(lens), (1, max(lens)), len(queries), (0, 9), "uniform", (1, 9),
                           len(lens), 311)
    wl = W.make_workload(cfg)
    wl.table_len[:] = lens
    wl.queries[:] = [np.array(q, dtype=np.int32) for q in queries]
    wl.suffix_len[:] = suffix
    dw = H.DeviceWorkload(wl)
    for ns in splits:
        dw.ctx.tc_set_kv_splits(ns)
        bt, pl = dw.stitch()
        out, qkv = dw.attn_layer(1, bt, pl)
        got, ref = H.out_to_f64(out, cfg), H.oracle_attn_layer(wl, dw.tables_np, 1, qkv)
        for i, r in ref.items():
            sl = slice(int(wl.cu_seqlens[i]), int(wl.cu_seqlens[i + 1]))
            err = float(np.abs(got[sl] - r).max()) if r.size else 0.0
            assert err <= TOL, (ns, dw.ctx.tc_kv_splits(), i, err)
            n = int(pl[i]) + int(wl.suffix_len[i])
            k, v = dw.ctx.tc_read_seq_kv(1, bt[i, :-(-n // 16)], n, np.float32)
            ks, vs = H.oracle_sequences(wl, dw.tables_np, 1, i)
            np.testing.assert_array_equal(k, np.concatenate([ks, qkv[1][sl]]))
            np.testing.assert_array_equal(v, np.concatenate([vs, qkv[2][sl]]))
        dw.ctx.tc_release_seqs(bt)
    dw.close()


@pytest.mark.parametrize("D,hq,hkv", [(64, 8, 2), (64, 7, 1), (64, 3, 3), (128, 8, 2), (128, 5, 1)])
def test_edges(H, D, hq, hkv):
    """P: none, 1, one short of / exactly / one past a unit and a tile, several units per wave."""
    lens = [1, 31, 32, 33, 63, 64, 65, 129, 300]
    queries = [[], [0], [1], [2], [3], [4], [5], [6], [7], [8, 7, 5], [8, 8, 8, 2]]
    suffix = [33, 1, 2, 32, 31, 65, 8, 64, 9, 130, 7]
    _run(H, D, hq, hkv, lens, queries, suffix, (0, 1, 3, 7))


@pytest.mark.parametrize("D", [64, 128])
def test_range_longer_than_the_block_id_table(H, D):
    """513 key tiles of prefix where a work item may have 512: cut in two although one range is asked for."""
    _run(H, D, 2, 1, [32800, 40], [[0], [1]], [3, 17], (1, 0))


@pytest.mark.parametrize("D,splits", [(64, 1), (64, 3), (128, 1)])
def test_values_of_later_tokens_reach_no_earlier_row(H, D, splits):
    """An infinity and a NaN in the values of one suffix token: the rows before it are what they are
    without it, the rows from it on are not finite in exactly those columns."""
    cfg = W.WorkloadConfig("f", 1, 6, 2, D, "f32", 2, (1, 70), 2, (0, 2), "uniform", (1, 9), 2, 312)
    wl = W.make_workload(cfg)
    wl.table_len[:] = [70, 33]
    wl.queries[:] = [np.array([0, 1], dtype=np.int32), np.array([1], dtype=np.int32)]
    wl.suffix_len[:] = [45, 20]
    dw = H.DeviceWorkload(wl)
    dw.ctx.tc_set_kv_splits(splits)
    q, k, v = wl.suffix_qkv(0)
    ref = H.oracle_attn_layer(wl, dw.tables_np, 0, (q, k, v))
    at = 27                                      # token 27 of the first query, columns 3 and 5 of KV head 1
    bad = v.copy()
    bad[at, 1, 3], bad[at, 1, 5] = np.inf, np.nan
    bt, pl = dw.stitch()
    got = H.out_to_f64(dw.attn_layer(0, bt, pl, qkv=(q, k, bad))[0], cfg)
    want = np.concatenate([ref[0], ref[1]])
    hit = np.zeros(want.shape, dtype=bool)
    hit[at:45, 3:, 3] = hit[at:45, 3:, 5] = True
    assert not np.isfinite(got[hit]).any()
    assert float(np.abs(got - want)[~hit].max()) <= TOL
    dw.ctx.tc_release_seqs(bt)
    dw.close()


@pytest.mark.parametrize("hq,hkv,D", [(8, 2, 64), (6, 2, 128), (5, 1, 64), (3, 3, 128)])
def test_ranges_combined_inside_the_launch_and_by_one_of_its_own(hq, hkv, D):
    """Heads of 64: partition counts around the fold's rounds of four and its limit of eight; beyond, and for heads of 128, the
    merge launch.  Ragged row tiles, slots evenly spaced and packed, every plan twice (the arrival counters are found at zero again)."""
    import harness as H
    from paper_2601_08743_amd import workloads as W
    cfg = W.WorkloadConfig("fold", 1, hq, hkv, D, "f32", 4, (300, 420), 3, (1, 3), "uniform", (5, 40), 4, 331)
    for lens, suffix in ((None, None), ([20, 400, 900, 300], [60, 3, 5])):
        wl = W.make_workload(cfg)
        if lens:
            wl.table_len[:], wl.suffix_len[:] = lens, suffix
            wl.queries[:] = [np.array(q, dtype=np.int32) for q in ([0], [1, 2], [2, 3])]
        dw = H.DeviceWorkload(wl)
        ref = None
        for splits in (1, 2, 4, 5, 8, 9, 16, 0):
            dw.ctx.tc_set_kv_splits(splits)
            bt, pl = dw.stitch()
            outs = [dw.attn_layer(0, bt, pl) for _ in range(2)]
            got = H.out_to_f64(outs[0][0], cfg)
            np.testing.assert_array_equal(got, H.out_to_f64(outs[1][0], cfg))
            if ref is None:
                ref = H.oracle_attn_layer(wl, dw.tables_np, 0, outs[0][1])
            for i, r in ref.items():
                err = float(np.abs(got[int(wl.cu_seqlens[i]):int(wl.cu_seqlens[i + 1])] - r).max())
                assert err <= TOL, (splits, i, err)
            dw.ctx.tc_release_seqs(bt)
        dw.close()
