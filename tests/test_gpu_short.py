"""The short-launch prefill kernel at the sizes where it can go wrong: prefix units of 32 keys that are ragged,
fewer units than waves, one more than a round of the waves, the suffix in a wave's first and later units,
row tiles of 32 that are ragged, causal ends that leave suffix units out, key ranges of which some lie in the suffix
alone, tables read in place with unused block tails.  Against the fp64 checker on every row, the pool bit for bit."""
import numpy as np
import pytest

from paper_2601_08743_amd import workloads as W

pytestmark = pytest.mark.gpu

# Softmax weights and outputs carry 8 bits (2^-9 relative each, |v| < 5.5, weights that sum to 1): a row that one
# key dominates may be off by 2 * 2^-9 * 5.5 = 2.2e-2; with two keys or more the terms average below 1e-2 of these inputs.
TOL = 2.2e-2


@pytest.fixture(scope="module")
def H():
    import harness
    return harness


LENS = [1, 31, 32, 33, 63, 64, 65, 129, 300]
QUERIES = [[], [0], [1], [2], [3], [4], [5], [6], [7], [8], [8, 7, 5], [8, 8, 8, 2]]


def _run(H, hq, hkv, lens, queries, suffix, splits, alias=False, kind=5):
    cfg = W.WorkloadConfig("s", 2, hq, hkv, 128, "bf16", len(lens), (1, max(lens)), len(queries), (0, 2), "uniform", (1, 9),
                           len(lens), 313)
    wl = W.make_workload(cfg)
    wl.table_len[:] = lens
    wl.queries[:] = [np.array(q, dtype=np.int32) for q in queries]
    wl.suffix_len[:] = suffix
    dw = H.DeviceWorkload(wl, slot_layout=1 if alias else 0,
                          seq_blocks=sum(-(-(sum(lens[t] for t in q) + s) // 16) + 1 for q, s in zip(queries, suffix)) + 8)
    dw.ctx.tc_set_attn_kernel(kind)
    for ns in splits:
        dw.ctx.tc_set_kv_splits(ns)
        bt, pl = dw.alias() if alias else dw.stitch()
        out, qkv = dw.attn_layer(1, bt, pl)
        assert dw.ctx.tc_attn_kernel() == 5
        got, ref = H.out_to_f64(out, cfg), H.oracle_attn_layer(wl, dw.tables_np, 1, qkv)
        for i, r in ref.items():
            sl = slice(int(wl.cu_seqlens[i]), int(wl.cu_seqlens[i + 1]))
            err = float(np.abs(got[sl] - r).max()) if r.size else 0.0
            assert err <= TOL, (ns, dw.ctx.tc_kv_splits(), i, err)
            if alias:                            # the suffix has blocks of its own, behind the tables' ones
                first, n = int(pl[i]) // 16, int(wl.suffix_len[i])
                if n == 0:
                    continue
                k, v = dw.ctx.tc_read_seq_kv(1, bt[i, first:first - (-n // 16)], n, np.uint16)
                np.testing.assert_array_equal(k.view(np.uint16), qkv[1][sl].view(np.uint16))
                np.testing.assert_array_equal(v.view(np.uint16), qkv[2][sl].view(np.uint16))
                continue
            n = int(pl[i]) + int(wl.suffix_len[i])
            k, v = dw.ctx.tc_read_seq_kv(1, bt[i, :-(-n // 16)], n, np.uint16)
            ks, vs = H.oracle_sequences(wl, dw.tables_np, 1, i)
            np.testing.assert_array_equal(k.view(np.uint16), np.concatenate([ks, qkv[1][sl]]).view(np.uint16))
            np.testing.assert_array_equal(v.view(np.uint16), np.concatenate([vs, qkv[2][sl]]).view(np.uint16))
        dw.ctx.tc_release_seqs(bt)
    dw.close()


@pytest.mark.parametrize("hq,hkv", [(28, 4), (8, 8), (5, 1), (80, 2)])
@pytest.mark.parametrize("alias", [False, True])
def test_edges(H, hq, hkv, alias):
    suffix = [33, 1, 2, 32, 31, 65, 8, 64, 9, 17, 130, 7]
    _run(H, hq, hkv, LENS, QUERIES, suffix, (1, 2, 3, 7), alias)


def test_range_of_the_whole_block_id_table(H):
    """256 and 257 key tiles: the longest range a work item may have, and one tile more (cut in two)."""
    _run(H, 4, 2, [16384 - 64, 64, 40], [[0], [0, 1], [2]], [3, 40, 17], (1, 2))


def test_chosen_for_a_short_question(H):
    """The automatic choice takes it for a few tokens against a few tables, and leaves it where rows abound."""
    _run(H, 28, 4, [300, 401, 233], [[0, 1, 2]], [17], (0,), kind=0)


@pytest.mark.parametrize("hq,hkv", [(28, 4), (8, 8), (5, 1)])
def test_up_to_eight_ranges_and_more(H, hq, hkv):
    """Eight ranges are combined inside the launch, nine and more by one of its own: slots for the most ranges everywhere, or
    packed where a query has too few key tiles for that."""
    _run(H, hq, hkv, [1300, 700], [[0], [1], [0, 1]], [17, 33, 2], (7, 8, 9, 16, 17, 22))
    _run(H, hq, hkv, [1300, 100], [[0], [1], [0, 1]], [5, 60, 2], (9, 22))
