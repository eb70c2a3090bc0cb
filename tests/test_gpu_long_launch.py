"""The long-launch prefill kernel at the sizes where its way with the suffix can go wrong: prefixes that end on and around
block and tile edges (the block that a query shares with its prefix, tiles of both), suffixes of one token, of whole and
of ragged blocks, more blocks to append than a row tile has waves, key ranges that lie in the suffix alone, tables
read in place.  Against the fp64 checker on every row, the pool bit for bit."""
import numpy as np
import pytest

from paper_2601_08743_amd import workloads as W

pytestmark = pytest.mark.gpu

# Softmax weights and outputs carry 8 bits (2^-9 relative each, |v| < 5.5, weights that sum to 1): a row that one
# key dominates may be off by 2 * 2^-9 * 5.5 = 2.2e-2; with two keys or more the terms average below 1e-2 of these inputs.
TOL = 2.2e-2
LENS = [1, 15, 16, 17, 49, 63, 64, 65, 250]
QUERIES = [[], [0], [1], [2], [3], [4], [5], [6], [7], [8], [8, 7, 6], [8, 8, 1], [], [2]]
SUFFIX = [33, 1, 15, 16, 17, 31, 64, 65, 1, 300, 130, 2, 300, 200]


@pytest.fixture(scope="module")
def H():
    import harness
    return harness


@pytest.mark.parametrize("hq,hkv", [(28, 4), (8, 8), (5, 1), (64, 4)])
@pytest.mark.parametrize("alias", [False, True])
def test_suffix_from_the_new_rows(H, hq, hkv, alias):
    cfg = W.WorkloadConfig("l", 2, hq, hkv, 128, "bf16", len(LENS), (1, max(LENS)), len(QUERIES), (0, 2), "uniform", (1, 9),
                           len(LENS), 317)
    wl = W.make_workload(cfg)
    wl.table_len[:] = LENS
    wl.queries[:] = [np.array(q, dtype=np.int32) for q in QUERIES]
    wl.suffix_len[:] = SUFFIX
    dw = H.DeviceWorkload(wl, slot_layout=1 if alias else 0,
                          seq_blocks=sum(-(-(sum(LENS[t] for t in q) + s) // 16) + 1 for q, s in zip(QUERIES, SUFFIX)) + 8)
    dw.ctx.tc_set_attn_kernel(4)
    for ns in (1, 2, 5, 0):
        dw.ctx.tc_set_kv_splits(ns)
        bt, pl = dw.alias() if alias else dw.stitch()
        outs = [dw.attn_layer(1, bt, pl) for _ in range(2)]
        assert dw.ctx.tc_attn_kernel() == 4
        got, qkv = H.out_to_f64(outs[0][0], cfg), outs[0][1]
        np.testing.assert_array_equal(got, H.out_to_f64(outs[1][0], cfg))
        ref = H.oracle_attn_layer(wl, dw.tables_np, 1, qkv)
        for i, r in ref.items():
            sl = slice(int(wl.cu_seqlens[i]), int(wl.cu_seqlens[i + 1]))
            err = float(np.abs(got[sl] - r).max())
            assert err <= TOL, (ns, i, err)
            if alias:                                # the suffix has blocks of its own, behind the tables' ones
                first, n, k0, v0 = int(pl[i]) // 16, int(wl.suffix_len[i]), qkv[1][sl], qkv[2][sl]
            else:
                ks, vs = H.oracle_sequences(wl, dw.tables_np, 1, i)
                first, n, k0, v0 = 0, int(pl[i]) + int(wl.suffix_len[i]), np.concatenate([ks, qkv[1][sl]]), np.concatenate([vs, qkv[2][sl]])
            pad = -n % 16                            # behind the end the last block is zero
            k, v = dw.ctx.tc_read_seq_kv(1, bt[i, first:first - (-n // 16)], n + pad, np.uint16)
            for have, want in ((k, k0), (v, v0)):
                np.testing.assert_array_equal(have[:n].view(np.uint16), want.view(np.uint16))
                assert not have[n:].any()
        dw.ctx.tc_release_seqs(bt)
    dw.close()


@pytest.mark.parametrize("lens,suffix,cut", [([1400, 2600, 900, 2100], [128, 128, 128, 128], True), ([700, 700, 700, 700], [128] * 4, False)])
def test_values_beyond_fp16(H, lens, suffix, cut):
    """Values times 2^30 (exact in bf16): rows that average far above 65504, which a partial of a query that is only cut
    here must hold - with the scale taken out they are what they are without it."""
    def times_2_30(a):                               # bf16 bits: the exponent 30 more (zeros stay)
        return np.where(a.view(np.uint16) & 0x7f80, a.view(np.uint16) + (30 << 7), a.view(np.uint16)).astype(np.uint16).view(a.dtype)

    cfg = W.WorkloadConfig("v", 1, 40, 8, 128, "bf16", len(lens), (1, max(lens)), 8, (1, 2), "uniform", (1, 9), len(lens), 331)
    wl = W.make_workload(cfg)
    wl.table_len[:] = lens
    wl.queries[:] = [np.array(q, dtype=np.int32) for q in ([0], [1], [2], [1, 3], [0, 1], [3, 3], [1, 1], [2])]
    wl.suffix_len[:] = 2 * suffix
    plain = wl.table_kv
    wl.table_kv = lambda t: (plain(t)[0], times_2_30(plain(t)[1]))
    q, k, v = wl.suffix_qkv(0)
    dw = H.DeviceWorkload(wl)
    bt, pl = dw.stitch()
    dw.ctx.tc_set_attn_kernel(4)
    if not cut:
        dw.ctx.tc_set_kv_splits(1)
    out, qkv = dw.attn_layer(0, bt, pl, qkv=(q, k, times_2_30(v)))
    assert dw.ctx.tc_attn_kernel() == 4 and (dw.ctx.tc_kv_splits() > 1) == cut
    got, ref = H.out_to_f64(out, cfg) * 2.0 ** -30, H.oracle_attn_layer(wl, dw.tables_np, 0, qkv)
    for i, r in ref.items():
        err = float(np.abs(got[int(wl.cu_seqlens[i]):int(wl.cu_seqlens[i + 1])] - r * 2.0 ** -30).max())
        assert err <= TOL, (i, err)
    dw.ctx.tc_release_seqs(bt)
    dw.close()
