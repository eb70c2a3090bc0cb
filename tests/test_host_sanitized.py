"""The library's host-only logic, built with g++ under the address and undefined-behaviour
sanitizers and driven from a script (csrc/host_check.cpp): replacement rules (App. A) with pins,
the sequence-block allocator, the attention planner, the front end (Alg. 1, Eq. 1-2, the
Sec. 4.2.2 schedule).  Every answer is compared with the CPU checker's models or with the
invariants the kernels rely on; any sanitizer report fails the run.  No GPU needed."""
import os
import subprocess

import numpy as np
import pytest

import oracle

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(ROOT, "paper_2601_08743_amd", "csrc")

# key tiles whose block ids one work item may keep in LDS, per kernel (csrc/tc_types.h)
CAP_GENERAL, CAP_PIPE, CAP_PP, CAP_F32 = 256, 1024, 1024, 512


@pytest.fixture(scope="module")
def exe(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("hc") / "host_check")
    cmd = ["g++", "-std=c++17", "-O1", "-g", "-fsanitize=address,undefined", "-fno-sanitize-recover=all",
           "-I", os.path.join(ROOT, "include"), "-I", CSRC, "-o", out, os.path.join(CSRC, "host_check.cpp")]
    subprocess.check_call(cmd)
    return out


def run(exe, script: str):
    env = dict(os.environ, ASAN_OPTIONS="detect_leaks=1:abort_on_error=0", UBSAN_OPTIONS="print_stacktrace=1")
    env.pop("LD_PRELOAD", None)
    r = subprocess.run([exe], input=script, capture_output=True, text=True, env=env, timeout=300)
    assert r.returncode == 0 and "runtime error" not in r.stderr and "AddressSanitizer" not in r.stderr, r.stderr[-3000:]
    return r.stdout.splitlines()


@pytest.mark.parametrize("policy,model", [(0, oracle.LRUModel), (1, oracle.FIFOModel), (2, oracle.LFUModel)])
def test_rules_with_pins_equal_the_models(exe, policy, model):
    rng = np.random.default_rng(100 + policy)
    cap = 5
    m = model(cap)
    pins, script, want = {}, ["rule %d %d" % (policy, cap)], []
    for _ in range(3000):
        r = rng.random()
        t = int(rng.integers(0, 14))
        if r < 0.15 and sum(1 for v in pins.values() if v) < cap - 1:
            pins[t] = pins.get(t, 0) + 1
            script.append("p %d" % t)
        elif r < 0.3 and any(pins.values()):
            t = [k for k, v in pins.items() if v][int(rng.integers(0, sum(1 for v in pins.values() if v)))]
            pins[t] -= 1
            script.append("u %d" % t)
        else:
            hit, ev = m.access(t, pinned=[k for k, v in pins.items() if v])
            want.append("r %d %d %d" % (t, 1 if hit else 0, -1 if ev is None else ev))
            script.append("r %d" % t)
    assert run(exe, "\n".join(script) + "\n") == want


def test_rule_refuses_when_everything_is_pinned(exe):
    got = run(exe, "rule 0 2\nr 1\nr 2\np 1\np 2\nr 3\nu 2\nr 3\n")
    assert got == ["r 1 0 -1", "r 2 0 -1", "r 3 0 refused", "r 3 0 2"]


def test_allocator_equals_the_sorted_set_model(exe):
    rng = np.random.default_rng(7)
    first, n = 40, 300
    free = set(range(first, first + n))
    held, script, want = [], ["seq %d %d" % (first, first + n)], []
    for _ in range(400):
        if rng.random() < 0.55 or not held:
            k = int(rng.integers(1, 40))
            script.append("t %d" % k)
            if k > len(free):
                want.append("t oom")
                continue
            got = sorted(free)[:k]
            free -= set(got)
            held.append(got)
            want.append("t " + " ".join(map(str, got)))
        else:
            blk = held.pop(int(rng.integers(0, len(held))))
            free |= set(blk)
            script.append("f %d %s" % (len(blk), " ".join(map(str, blk))))
    script.append("f 1 5")                       # not a sequence block: refused, no crash
    want.append("f bad 5")
    assert run(exe, "\n".join(script) + "\n") == want


@pytest.mark.parametrize("cap", [1 << 20, 1 << 16, 131080, 65544])
def test_staged_plans_share_no_memory_with_an_upload_nobody_waited_for(exe, cap):
    """Plans longer than half the buffer between short ones, sizes at the half's edge: a plan may overlap an
    earlier one only if it waits for one of the events that the earlier one's upload recorded."""
    rng = np.random.default_rng(cap)
    half = cap // 2
    sizes = [int(x) for x in rng.choice([8, 4096, half - 64, half - 8, half, half + 8, cap - 8, cap], 300)]
    spots = [tuple(map(int, l.split()[1:])) for l in run(exe, "stage %d %d %s\n" % (cap, len(sizes), " ".join(map(str, sizes))))]
    assert len(spots) == len(sizes)
    pending = {}                                 # half -> index of the plan whose upload recorded its event last
    for i, ((at, parts), n) in enumerate(zip(spots, sizes)):
        assert parts in (1, 2, 3) and at % 4 == 0 and at + n <= cap
        over = {pending[k] for k in pending if parts >> k & 1}          # waited for
        for j in set(pending.values()) - over:
            (a, _), m = spots[j], sizes[j]
            assert at + n <= a or a + m <= at, (i, j)
        for k in (0, 1):
            if parts >> k & 1:
                pending[k] = i
    short = [p for (_, p), n in zip(spots, sizes) if n <= 4096]
    assert {1, 2} <= set(short)                  # and short ones do alternate


def test_staging_memory_names_its_coherence():
    """A kernel reads the pinned staging buffer, so what it may keep of it in a cache is not left to the environment
    (hipHostMallocDefault follows HIP_HOST_COHERENT)."""
    import re
    with open(os.path.join(CSRC, "tc_host.hip")) as f:
        src = f.read()
    flags = re.findall(r"hipHostMalloc\([^;]*, (\w+)\)", src)
    assert len(flags) == src.count("hipHostMalloc(") and set(flags) == {"kStagingFlags"}
    assert re.search(r"kStagingFlags = hipHostMallocCoherent;", src)


def _plan(exe, Hq, Hkv, PS, splits=0, rb=0, kernel=0, dtype=1, D=128, within=(0, 0)):
    lines = run(exe, "within %d %d\n" % within + "plan %d %d %d %d %d %d %d %d %s\n" % (dtype, Hq, Hkv, D, splits, rb, kernel, len(PS),
                                                          " ".join("%d %d" % ps for ps in PS)))
    head = list(map(int, lines[0].split()[1:]))
    rows = [tuple(map(int, l.split()[1:])) for l in lines[1:] if l.startswith("i ")]
    items = [r[:7] for r in rows]
    assert head[0] == len(items)
    ghead = [l for l in lines if l.startswith("groups ")][0].split()
    groups = [tuple(map(int, l.split()[1:])) for l in lines if l.startswith("g ")]
    info = dict(max_splits=head[1], decode=head[2], pingpong=head[3], pipelined=head[4], row_blocks=head[5], ok=head[6], brief=head[7],
                n_groups=int(ghead[2]), groups=groups, item_arrival=[r[7] for r in rows], item_holder=[r[10] for r in rows], item_part=[r[8:10] for r in rows])
    info["folds"] = int([l for l in lines if l.startswith("folds")][0].split()[1])
    info["merges"] = int([l for l in lines if l.startswith("merges")][0].split()[1])
    info["part_f32"] = int([l for l in lines if l.startswith("part_f32")][0].split()[1])
    info["ints"], info["compact"], info["counters"], info["counter_ints"] = map(int, [l for l in lines if l.startswith("ints")][0].split()[1:])
    info["part_floats"], info["part_stride"], *info["part_tab"] = map(int, [l for l in lines if l.startswith("parts")][0].split()[1:])
    assert int(ghead[1]) == len(groups)
    return info, items


def _check_plan(info, items, Hq, Hkv, PS, dtype=1):
    """What the kernels rely on: every (query, KV head, row tile) is covered by partitions that cut
    its key tiles [0, n_tiles) into consecutive non-empty ranges, and no range is longer than the
    block-id table of the kernel that runs it."""
    assert info["ok"] == 1
    G = Hq // Hkv
    if info["decode"]:
        cap, rt, unified = CAP_GENERAL, None, False
    else:
        cap = (10 ** 9 if info["compact"] else CAP_F32) if dtype == 0 else CAP_PP if info["pingpong"] else CAP_PIPE if info["pipelined"] else CAP_GENERAL
        rt = 32 if dtype == 0 or info["brief"] else 128 * info["row_blocks"]      # what the kernels stride their rows by
        unified = dtype == 0 or bool(info["pingpong"])
    cover = {}
    if not info["decode"] and dtype == 1 and not info["brief"]:
        # the merge launch goes by the group table: one entry per (query, KV head, row tile), each with the partition
        # count that its items carry and, where that is more than one, the slots that they write: of nobody else's
        base = np.cumsum([0] + [S for _, S in PS])
        table = {(cu, kvh, m0): (ns, S, part0) for kvh, m0, ns, cu, S, part0 in info["groups"]}
        assert len(table) == len(info["groups"]) == info["n_groups"]
        for (q, kvh, m0, tb, te, split, ns), (part0, _) in zip(items, info["item_part"]):
            if q >= 0:
                assert table[base[q], kvh, m0][:2] == (ns, PS[q][1])
                assert ns == 1 or table[base[q], kvh, m0][2] == part0
        slots = sorted((part0, ns) for ns, _, part0 in table.values() if ns > 1)
        assert all(a + n <= b for (a, n), (b, _) in zip(slots, slots[1:]))
    # where ranges are combined inside the launch, a row tile's items count in at a counter of their own: 128 bytes behind the plan,
    # or in one of those items
    counted = {}
    for (q, kvh, m0, tb, te, split, ns), at, holder in zip(items, info["item_arrival"], info["item_holder"]):
        assert (at >= 0) == (holder >= 0) == (q >= 0 and ns > 1 and info["folds"] == 1)
        if at >= 0:
            counted.setdefault((q, kvh, m0), []).append((at, ns, holder))
    for (q, kvh, m0), who in counted.items():
        assert len(set(who)) == 1 and len(who) == who[0][1] and items[who[0][2]][:3] == (q, kvh, m0)
    assert len({who[0][0] for who in counted.values()}) == len(counted)
    assert all(32 * who[0][0] + 32 <= info["counter_ints"] for who in counted.values())
    assert info["counters"] % 32 == 0 and info["counters"] >= info["ints"] and (info["folds"] or info["counter_ints"] == 0)
    for q, kvh, m0, tb, te, split, ns in items:
        if q < 0:
            continue
        empty_ok = info["decode"] and PS[q][0] == 0          # a decode step over an empty prefix: the token sees itself only
        assert (0 < te - tb or empty_ok) and te - tb <= cap, (q, tb, te, cap)
        cover.setdefault((q, kvh, m0), []).append((split, tb, te, ns))
    for i, (P, S) in enumerate(PS):
        if S == 0:
            assert not any(k[0] == i for k in cover)
            continue
        if info["decode"]:
            n_tiles, rows = -(-P // 64), [0]
        else:
            n_tiles = -(-(P + S) // 64) if unified else -(-P // 64) + -(-S // 64)
            rows = list(range(0, S * G, rt))
        assert {k[1:] for k in cover if k[0] == i} == {(kvh, m0) for kvh in range(Hkv) for m0 in rows}
        for kvh in range(Hkv):
            for m0 in rows:
                parts = sorted(cover[(i, kvh, m0)])
                assert [p[0] for p in parts] == list(range(len(parts))) and all(p[3] == len(parts) for p in parts)
                assert parts[0][1] == 0 and parts[-1][2] == n_tiles
                assert all(a[2] == b[1] for a, b in zip(parts, parts[1:]))
    return max([te - tb for q, _, _, tb, te, _, _ in items if q >= 0], default=0)


def _check_slots(info, items, Hq, D, PS):
    """Partials kept by row: every (token, partition) of a cut query, and no other, has a slot
    of its own inside the buffer, and the items write where the merge, going by its table, reads."""
    ns, base = {}, np.cumsum([0] + [S for _, S in PS])
    for it in items:
        if it[0] >= 0:
            ns[it[0]] = it[6]
    counts = [n if n > 1 else 0 for q, (_, S) in enumerate(PS) for n in [ns.get(q, 0)] * S]
    if info["part_stride"]:                      # evenly spaced
        assert info["part_tab"] == counts and info["part_stride"] == info["max_splits"]
        first, n_slots = [n * info["part_stride"] for n in range(len(counts))], len(counts) * info["part_stride"]
        assert n_slots <= 2 * sum(counts) and info["merges"]
    else:                                        # packed; only a merge launch has a table
        at = np.cumsum([0] + counts).tolist()
        assert info["part_tab"] == (at if info["merges"] else [])
        first, n_slots = at[:-1], sum(counts)
    assert info["part_floats"] == n_slots * Hq * (D + 2)
    for it, (part0, stride) in zip(items, info["item_part"]):
        if it[0] >= 0 and it[6] > 1:
            for t in range(PS[it[0]][1]):
                assert part0 + t * stride + it[5] == first[base[it[0]] + t] + it[5] < n_slots


# Batches of one long sequence among short ones, which the workspace of the entry point that allocates nothing
# (15 Mi floats of partials) holds: the long one's partition count is not everybody's.
WORKSPACE = 15 << 20


@pytest.mark.parametrize("Hq,Hkv,PS,kernel", [
    (32, 1, [(45776, 1)] + [(20, 1)] * 15, "decode"), (32, 2, [(300, 1)] * 63 + [(20000, 1)], "decode"),
    (32, 1, [(300, 1)] * 31 + [(20000, 1)], "decode"), (32, 1, [(300, 1)] * 63 + [(20000, 1)], "decode"),
    (28, 4, [(12800, 5)] + [(200, 4)] * 3, "brief")])
def test_partials_of_ragged_batches_stay_small(exe, Hq, Hkv, PS, kernel):
    info, items = _plan(exe, Hq, Hkv, PS, kernel=0 if kernel == "decode" else 5, splits=0 if kernel == "decode" else 40)
    assert info["ok"] and info[kernel]
    _check_slots(info, items, Hq, 128, PS)
    assert info["max_splits"] > 30 and info["part_floats"] <= WORKSPACE // 4


PLAN_INTS = 1 << 20                          # and of its plan


@pytest.mark.parametrize("Hq,Hkv,D,PS", [(32, 8, 128, [(7744, 23), (2119, 220)]), (8, 2, 128, [(15727, 652), (284, 992)]),
                                         (32, 8, 128, [(6000, 500)] * 3 + [(8000, 8)]), (8, 2, 64, [(20000, 1000)] * 6)])
def test_fp32_ranges_go_by_the_workspace(exe, Hq, Hkv, D, PS):
    """Where the partials of the fastest plan do not fit, a plan with fewer partitions whose partials do."""
    free, _ = _plan(exe, Hq, Hkv, PS, dtype=0, D=D)
    info, items = _plan(exe, Hq, Hkv, PS, dtype=0, D=D, within=(PLAN_INTS, WORKSPACE))
    _check_plan(info, items, Hq, Hkv, PS, dtype=0)
    assert not info["compact"] and info["ints"] <= PLAN_INTS and info["part_floats"] <= WORKSPACE
    assert info["max_splits"] == free["max_splits"] if free["part_floats"] <= WORKSPACE else info["max_splits"] < free["max_splits"]


def test_plan_of_least_space(exe):
    """What a fixed workspace cannot hold as planned for speed is planned for the least space: fp32 in one range
    however long (one partition never needs partials), no padded block table, no short-launch or extra partitions."""
    PS = [(40000, 2000), (50, 3)]                # 656 key tiles; two partitions would be 2000 x 32 x 2 rows of 130 floats = 16.6 M
    info, items = _plan(exe, 32, 8, PS, dtype=0, within=(PLAN_INTS, WORKSPACE))
    assert _check_plan(info, items, 32, 8, PS, dtype=0) == 657 and info["compact"] and info["max_splits"] == 1 and info["part_floats"] == 0
    PS = [(4992, 8)] * 30 + [(5008, 0)] * 3265   # 313 blocks a row, 316 padded: 3295 of those and the plan exceed 1 Mi integers
    free, _ = _plan(exe, 28, 4, PS)
    info, items = _plan(exe, 28, 4, PS, within=(PLAN_INTS, WORKSPACE))
    _check_plan(info, items, 28, 4, PS)
    assert free["brief"] and free["ints"] > PLAN_INTS and info["compact"] and info["ints"] <= PLAN_INTS
    # nothing of one partition and few rows is refused, whatever its shape
    rng = np.random.default_rng(23)
    for _ in range(60):
        dtype, Hkv, G = int(rng.random() < 0.5), int(rng.choice([1, 2, 8])), int(rng.choice([1, 4, 7, 32]))
        PS = [(int(2 ** rng.uniform(0, 16)), int(2 ** rng.uniform(0, 10))) for _ in range(int(rng.integers(1, 9)))]
        info, items = _plan(exe, Hkv * G, Hkv, PS, dtype=dtype, within=(PLAN_INTS, WORKSPACE))
        _check_plan(info, items, Hkv * G, Hkv, PS, dtype=dtype)
        rows = sum(S for _, S in PS) * Hkv * G
        if (rows <= 1e5 and dtype == 0) or rows <= 2e4:
            assert info["ints"] <= PLAN_INTS and info["part_floats"] <= WORKSPACE, (dtype, Hkv, G, PS)


def test_sequences_in_one_range_need_no_partials(exe):
    """A decode step writes the row of a sequence in one range directly: as many of them as the plan has room for fit the
    workspace, and beside cut ones they take no slots."""
    info, items = _plan(exe, 32, 1, [(300, 1)] * 3900, within=(PLAN_INTS, WORKSPACE))
    assert info["decode"] and not info["compact"] and info["max_splits"] == 1 and info["part_floats"] == 0
    info, items = _plan(exe, 32, 8, [(20000, 1)] + [(200, 1)] * 20)
    _check_slots(info, items, 32, 128, [(20000, 1)] + [(200, 1)] * 20)
    assert info["decode"] and info["part_floats"] == info["max_splits"] * 32 * 130 and info["max_splits"] > 1


def test_planner_partition_limit_with_forced_splits(exe):
    """A long prefix with a short suffix and a forced split count: the cut by weight used to leave
    a first partition of 259 tiles, three more than the general kernel's block-id table holds."""
    PS = [(32400, 168)]
    for splits in (1, 2, 3):
        for kernel in (1, 2, 4, 0):
            info, items = _plan(exe, 28, 4, PS, splits=splits, kernel=kernel)
            longest = _check_plan(info, items, 28, 4, PS)
            print("P=32400 S=168 forced splits %d kernel %d -> %d partitions, longest %d tiles" %
                  (splits, kernel, info["max_splits"], longest))
    info, items = _plan(exe, 28, 4, PS, splits=2, kernel=1)
    assert info["max_splits"] >= 3 and not info["pipelined"]
    # longer than every kernel's table (1095 key tiles): the pipelined kernel is planned twice (for
    # the general kernel's 256 tiles first, then for its own 1024), and the merge groups must be
    # those of the second pass - they once were the first pass's, with five partitions each
    PS = [(70001, 37), (100, 5)]
    for kernel, splits, want in ((2, 1, 2), (2, 4, 4), (4, 1, 2), (1, 2, 5), (0, 0, None)):
        info, items = _plan(exe, 4, 1, PS, splits=splits, kernel=kernel)
        _check_plan(info, items, 4, 1, PS)
        if want is not None:
            assert info["max_splits"] == want, (kernel, splits, info["max_splits"])


@pytest.mark.parametrize("splits", [1000, 10 ** 6, 2 * 10 ** 9])
@pytest.mark.parametrize("kernel,dtype", [(0, 1), (1, 1), (4, 1), (5, 1), (0, 0)])
def test_planner_takes_any_forced_partition_count(exe, splits, kernel, dtype):
    """tc_set_kv_splits accepts any count; more partitions than key tiles means one per key tile, and
    the planner's memory goes by that and not by the number asked for."""
    PS = [(2000, 128), (3000, 100)]
    lines = run(exe, "plan %d 28 4 128 %d 0 %d 2 2000 128 3000 100\n" % (dtype, splits, kernel))
    head = list(map(int, lines[0].split()[1:]))
    unified = dtype == 0 or head[3]
    want = [-(-(P + S) // 64) if unified else -(-P // 64) + -(-S // 64) for P, S in PS]
    assert head[6] == 1 and head[1] == max(want)
    ns = {}
    for l in lines:
        if l.startswith("i "):
            q, n = (int(l.split()[k]) for k in (1, 7))
            if q >= 0:
                ns[q] = n
    assert [ns[0], ns[1]] == want


def test_planner_paper_shapes(exe):
    c4 = [(24625, 512)] * 4
    info, items = _plan(exe, 32, 8, c4)
    _check_plan(info, items, 32, 8, c4)
    assert info["pingpong"] == 1 and info["max_splits"] == 1 and sum(1 for it in items if it[0] >= 0) == 256
    info, items = _plan(exe, 32, 8, c4, kernel=2)              # the pipelined kernel takes c4 unsplit as well
    _check_plan(info, items, 32, 8, c4)
    assert info["pipelined"] == 1 and info["max_splits"] == 1 and sum(1 for it in items if it[0] >= 0) == 512
    info, items = _plan(exe, 32, 8, c4, kernel=1)              # the general kernel must split
    _check_plan(info, items, 32, 8, c4)
    assert info["max_splits"] >= 2
    c2 = [(4086, 128)]
    info, items = _plan(exe, 28, 4, c2)
    _check_plan(info, items, 28, 4, c2)
    assert info["pipelined"] == 1 and info["max_splits"] == 8
    for PS, chosen in (([(1050, 17)], 1), ([(1050, 17)] * 8, 1), (c2, 0), (c4, 0)):     # a short question goes to the short-launch kernel
        info, items = _plan(exe, 28, 4, PS)
        _check_plan(info, items, 28, 4, PS)
        assert info["brief"] == chosen
    dec = [(5000, 1), (17, 1), (0, 1), (900, 0)]
    info, items = _plan(exe, 28, 4, dec)
    assert info["decode"] == 1
    _check_plan(info, items, 28, 4, dec)


def test_long_launch_kernel_up_to_a_fifth_of_padding(exe):
    """Launches of 14 .. 80 us go to the long-launch kernel if 256-row tiles make at most 6 / 5 of the rows of 128-row tiles,
    the limit itself (five 128-row tiles, three of 256 rows) included."""
    at = [(3000 + 17 * i, 128) for i in range(8)]           # 40 / 8 heads: 640 rows a KV head
    for PS, want in ((at, 1), (at + [(3000, 25)], 0), (at[:1], 0), ([(3000, 51)] * 8, 1)):
        info, items = _plan(exe, 40, 8, PS)
        _check_plan(info, items, 40, 8, PS)
        assert info["pingpong"] == want, PS


def test_decode_ranges_make_one_round_of_even_work_groups(exe):
    """A decode step is planned for one round of work-groups on the 256 CUs, all about equally long:
    the paper-shaped batches come out as at most 256 items, none longer than the shortest common
    range length that fits, and a long sequence is cut into more ranges than a short one."""
    import sys
    sys.path.insert(0, ROOT)
    from paper_2601_08743_amd import workloads as W
    for name, Hq, Hkv in (("c3", 28, 4), ("c4", 32, 8), ("c2", 28, 4)):
        wl = W.get(name)
        PS = [(int(wl.table_len[q].sum()) + int(s), 1) for q, s in zip(wl.queries, wl.suffix_len)]
        info, items = _plan(exe, Hq, Hkv, PS)
        assert info["decode"] == 1
        longest = _check_plan(info, items, Hq, Hkv, PS)
        real = [it for it in items if it[0] >= 0]
        tiles = [-(-P // 64) for P, _ in PS]
        assert len(real) <= 256, (name, len(real))
        # no shorter common range length would have fitted the 256 CUs (or the floor of two tiles was hit)
        L = longest
        fits = lambda L: sum(Hkv * max(1, -(-t // L)) for t in tiles) <= 256
        assert fits(L) and (L <= 2 or not fits(L - 1)), (name, L)
        per_q = {}
        for q, kvh, m0, tb, te, split, ns in real:
            per_q[q] = ns
        order = sorted(range(len(tiles)), key=lambda i: tiles[i])
        assert all(per_q[a] <= per_q[b] for a, b in zip(order, order[1:])), name
        lens = [te - tb for _, _, _, tb, te, _, _ in real]
        assert lens == sorted(lens, reverse=True), "longest items first"
        print("%s decode: %d items, ranges of %d..%d key tiles, %d..%d ranges per sequence" % (
            name, len(real), min(lens), max(lens), min(per_q.values()), max(per_q.values())))
    # short sequences: ranges of two tiles, a unit for each wave, and a lone odd tile
    info, items = _plan(exe, 28, 4, [(64 * 9, 1), (64 * 4 - 1, 1)])
    assert _check_plan(info, items, 28, 4, [(64 * 9, 1), (64 * 4 - 1, 1)]) == 2
    assert sorted({(q, te - tb) for q, _, _, tb, te, _, _ in items}) == [(0, 1), (0, 2), (1, 2)]
    # more (query, KV head) pairs than CUs: one range each, several rounds
    PS = [(3000 + 17 * i, 1) for i in range(100)]
    info, items = _plan(exe, 28, 4, PS)
    assert info["decode"] == 1 and info["max_splits"] == 1 and sum(1 for it in items if it[0] >= 0) == 400
    _check_plan(info, items, 28, 4, PS)
    # a sequence longer than one item's block-id table is cut whatever the batch looks like
    PS = [(64 * 700, 1)] + [(500, 1)] * 80
    info, items = _plan(exe, 28, 4, PS)
    _check_plan(info, items, 28, 4, PS)
    assert info["max_splits"] == 3


def test_planner_random_batches(exe):
    rng = np.random.default_rng(11)
    for _ in range(150):
        Hkv = int(rng.choice([1, 2, 4, 8]))
        G = int(rng.choice([1, 2, 4, 5, 7, 8]))
        B = int(rng.integers(1, 7))
        PS = [(int(rng.choice([0, 1, 63, 64, 65, int(rng.integers(0, 3000)), int(rng.integers(0, 70000))])),
               int(rng.choice([0, 1, 64, int(rng.integers(0, 600))]))) for _ in range(B)]
        dtype = int(rng.random() < 0.85)
        kw = dict(splits=int(rng.choice([0, 0, 1, 2, 5, 40])), rb=int(rng.choice([0, 0, 0, 1, 2])) if dtype else 0,
                  kernel=int(rng.choice([0, 0, 1, 2, 3, 4, 5])) if dtype else 0)
        info, items = _plan(exe, Hkv * G, Hkv, PS, dtype=dtype, D=128 if dtype else 64, **kw)
        _check_plan(info, items, Hkv * G, Hkv, PS, dtype=dtype)
        if info["part_tab"]:
            _check_slots(info, items, Hkv * G, 128 if dtype else 64, PS)


RAGGED = [(P, 128) for P in (1400, 2600, 900, 5200, 2000, 3100, 4300, 700)]


def test_partials_of_queries_cut_by_the_long_launch_kernel_alone_are_fp32(exe):
    """What one partition count for the batch, or the kernel that would take it otherwise, leaves whole is fp32 to the end:
    fp32 partials where the long-launch kernel cuts it.  Batches whose queries are cut with fp16 partials either way keep those, forced
    counts and plans of least space too, and what the short-launch kernel would take stays there."""
    for Hq, Hkv, PS, kw, cut, f32 in (
            (40, 8, RAGGED, {}, 1, 1), (40, 8, RAGGED, dict(kernel=4), 1, 1), (40, 8, RAGGED, dict(kernel=4, splits=3), 1, 0),
            (40, 8, RAGGED, dict(within=(1 << 30, 1 << 22)), 1, 1), (32, 8, [(70000, 200)] * 4, dict(within=(1 << 30, 4456448)), 1, 0),
            (28, 4, [(1727, 100), (4048, 160), (3773, 48), (2584, 90)], {}, 1, 0), (40, 8, [(4600, 128)], {}, 1, 0)):
        info, items = _plan(exe, Hq, Hkv, PS, **kw)
        _check_plan(info, items, Hq, Hkv, PS)
        assert info["pingpong"] and (info["max_splits"] > 1, info["part_f32"]) == (bool(cut), f32), (PS, kw)
        slots = sum(1 for it in items if it[0] >= 0 and it[6] > 1)
        assert info["part_floats"] == slots * 256 * ((128 if f32 else 64) + 2) <= kw.get("within", (0, 1 << 62))[1]
    info, items = _plan(exe, 40, 8, [(809, 100), (809, 160)])
    assert info["brief"] and info["max_splits"] == 1


def test_short_launch_plans(exe):
    """What the short-launch kernel relies on: 32-row tiles, every (query, KV head, row tile) covered by
    consecutive non-empty ranges of at most 256 key tiles; chosen by itself: at most 512 items, uncut
    beyond 256.  Forced, it serves any batch; chosen, few tokens against few tables, neither long nor wide ones."""
    rng = np.random.default_rng(17)
    batches = [[(1050, 17)], [(0, 5)], [(33000, 3)], [(4086, 128)], [(60, 1), (61, 0), (0, 2)], [(24600, 512)] * 4]
    for _ in range(60):
        n = int(rng.integers(1, 24))
        batches.append([(int(rng.integers(0, 12000)), int(2 ** rng.uniform(0, 8.5))) for _ in range(n)])
    chosen = []
    for (hq, hkv), kernel in [((28, 4), 0), ((28, 4), 5), ((40, 8), 0), ((3, 3), 5), ((96, 2), 5)]:
        for PS in batches:
            lines = run(exe, "short 32\nplan 1 %d %d 128 0 0 %d %d %s\n" % (hq, hkv, kernel, len(PS), " ".join("%d %d" % x for x in PS)))
            head = list(map(int, lines[0].split()[1:]))
            assert head[6] == 1                  # no range longer than its kernel's table
            if kernel == 0 and (hq, hkv) == (28, 4):
                chosen.append(head[7])
            if head[7] == 0:
                assert kernel == 0 or head[2]    # (a decode step)
                continue
            items = [tuple(map(int, l.split()[1:8])) for l in lines if l.startswith("i ")]
            items = [x for x in items if x[0] >= 0]
            G = hq // hkv
            if kernel == 0:
                assert len(items) <= 512 and (head[1] == 1 or len(items) <= 256)
            cover = {}
            for q, kvh, m0, tb, te, split, ns in items:
                assert 0 < te - tb <= 256 and m0 % 32 == 0
                cover.setdefault((q, kvh, m0), []).append((split, tb, te, ns))
            assert set(cover) == {(q, h, m) for q, (P, S) in enumerate(PS) for h in range(hkv) for m in range(0, S * G, 32)}
            for (q, _, _), parts in cover.items():
                parts.sort()
                P, S = PS[q]
                assert [x[0] for x in parts] == list(range(parts[0][3])) and parts[0][1] == 0
                assert all(a[2] == b[1] for a, b in zip(parts, parts[1:])) and parts[-1][2] == -(-P // 64) + -(-S // 64)
    assert chosen[0] == 1 and chosen[3] == 0 and chosen[5] == 0


def test_front_end_equals_the_checker(exe):
    rng = np.random.default_rng(5)
    tables, seen = {}, set()
    for t in range(40):
        toks = tuple(rng.integers(0, 4, size=int(rng.integers(1, 7))).tolist())
        if toks not in seen:
            seen.add(toks)
            tables[t] = list(toks)
    s = rng.integers(0, 4, size=4000).tolist()
    script = ["trie %d" % len(tables)] + ["%d %d %s" % (t, len(v), " ".join(map(str, v))) for t, v in tables.items()]
    script.append("match %d %s" % (len(s), " ".join(map(str, s))))
    sets = [sorted(rng.choice(30, size=int(rng.integers(1, 9)), replace=False).tolist()) for _ in range(120)]
    qs = "\n".join("%d %s" % (len(q), " ".join(map(str, q))) for q in sets)
    script.append("rerank %d 30 3\n%s" % (len(sets), qs))
    cases = [(12, 4, 4, 0, 0), (12, 4, 8, 0, 1), (10, 3, 0, 0, 0), (16, 8, 8, 1, 1)]
    for cap, bc, bm, keep, taper in cases:
        script.append("pipeline %d %d %d %d %d %d\n%s" % (len(sets), cap, bc, bm, keep, taper, qs))
    out = run(exe, "\n".join(script) + "\n")
    want = oracle.trie_match(tables, s)
    assert out[0] == "match %d" % len(want) + "".join(" %d %d" % m for m in want)
    assert out[1] == "rerank " + " ".join(map(str, oracle.rerank(sets, 3)))
    at = 2
    for cap, bc, bm, keep, taper in cases:
        steps = oracle.plan_pipeline(sets, cap, bc, bm, keep_pinned=bool(keep), taper=bool(taper))
        assert out[at] == "pipeline %d" % len(steps)
        got = [tuple(map(int, l.split()[1:])) for l in out[at + 1:at + 1 + len(steps)]]
        assert got == [tuple(st) for st in steps]
        at += 1 + len(steps)


def test_long_launch_ranges_go_by_each_query(exe):
    """One range length for the batch: a query has as many ranges as it takes, so long ones have more; batches that a cut
    does not promise 5 % stay whole; and the items placed longest first on 256 CUs end no later than uncut."""
    def ends(items):                                     # 7.8 us an item, 1.32 a key tile
        free = [0.0] * 256
        import heapq
        for n in sorted((it[4] - it[3] for it in items if it[0] >= 0), reverse=True):
            heapq.heapreplace(free, free[0] + 7.8 + 1.32 * n)
        return max(free)

    rng = np.random.default_rng(29)
    ragged = 0
    for _ in range(40):
        PS = [(int(rng.integers(200, 5000)), 128) for _ in range(int(rng.integers(2, 12)))]
        info, items = _plan(exe, 40, 8, PS, kernel=4)
        _check_plan(info, items, 40, 8, PS)
        whole, uncut = _plan(exe, 40, 8, PS, kernel=4, splits=1)
        ns = {it[0]: it[6] for it in items if it[0] >= 0}
        order = sorted(ns, key=lambda q: PS[q][0])
        assert all(ns[a] <= ns[b] for a, b in zip(order, order[1:]))
        assert ends(items) <= ends(uncut) + 1e-6
        ragged += len(set(ns.values())) > 1
    assert ragged >= 10
    info, items = _plan(exe, 28, 4, [(1500, 250)] * 60, kernel=4)      # many even items: nothing to gain
    assert info["max_splits"] == 1


@pytest.mark.parametrize("Hq,Hkv,PS", [(28, 4, [(4400, 400)]), (28, 4, [(3500, 370)]), (32, 8, [(5000, 500)]), (12, 1, [(9000, 300)] * 3)])
def test_long_launch_ranges_go_by_the_chiplets(exe, Hq, Hkv, PS):
    """The row tiles of a (query, KV head, range) stay on one of the eight XCDs (work-group id mod 8), 32 CUs each: of the
    equal range counts, the chosen one is as good as any by the placement that the launch will have - 7.8 us an item and 1.32 a key
    tile - to the 10 % that a range length in tenths, and a merge that grows with the count, may differ."""
    import heapq

    def ends(items):
        last = 0.0
        for x in range(8):
            free = [0.0] * 32
            for it in items[x::8]:
                if it[0] >= 0:
                    heapq.heapreplace(free, free[0] + 7.8 + 1.32 * (it[4] - it[3]))
            last = max(last, max(free))
        return last

    info, items = _plan(exe, Hq, Hkv, PS, kernel=4)
    _check_plan(info, items, Hq, Hkv, PS)
    assert info["max_splits"] > 1
    others = [ends(_plan(exe, Hq, Hkv, PS, kernel=4, splits=ns)[1]) for ns in range(1, 13)]
    assert ends(items) <= 1.1 * min(others) + 3.0, (info["max_splits"], ends(items), others)


def test_few_tokens_over_many_tables_stay_with_the_short_launch_kernel(exe):
    """Nine ranges and more are combined by a launch of its own, which costs no more than before there was any other way: such
    batches are not given to a kernel that keeps partials in fp16.  Up to eight need no table for that launch."""
    for Hq, Hkv in ((28, 4), (32, 8), (40, 8)):
        for PS in ([(2026, 7)], [(4800, 3)], [(8000, 8)]):
            info, items = _plan(exe, Hq, Hkv, PS)
            _check_plan(info, items, Hq, Hkv, PS)
            assert info["brief"] and info["max_splits"] > 8, (Hq, Hkv, PS)
    for PS, even in (([(1500, 17), (600, 3)], True), ([(1500, 3), (100, 17)], False)):
        for splits in (2, 8, 9, 30):
            info, items = _plan(exe, 28, 4, PS, kernel=5, splits=splits)
            _check_plan(info, items, 28, 4, PS)
            _check_slots(info, items, 28, 128, PS)
            assert info["brief"] and info["max_splits"] == min(splits, 25) and (info["part_stride"] > 0) == (even and splits > 8)


@pytest.mark.parametrize("Hq,Hkv,PS", [(28, 4, [(538, 22)]), (32, 8, [(528, 28)]), (40, 8, [(524, 9)]), (28, 4, [(456, 9)] * 2)])
def test_short_launches_of_three_units_a_wave_are_not_cut(exe, Hq, Hkv, PS):
    """In three ranges they take 0.5 .. 0.9 us longer than in one, also where those are combined inside the launch."""
    info, items = _plan(exe, Hq, Hkv, PS)
    _check_plan(info, items, Hq, Hkv, PS)
    assert info["brief"] == 1 and info["max_splits"] == 1


def test_decode_partials_are_folded_in_one_round_of_loads_or_merged(exe):
    """Up to 36 ranges of up to eight query heads per KV head, 72 of up to four, are combined inside the launch, any other cut by a launch that
    goes by the table of slots - and where that is needed, ranges are not made longer to have fewer of them."""
    for Hq, Hkv, P, splits, merged in ((8, 1, 64 * 40, 36, 0), (8, 1, 64 * 40, 37, 1), (9, 1, 64 * 40, 2, 1), (32, 1, 64 * 40, 36, 1),
                                       (64, 8, 64 * 40, 36, 0), (4, 1, 64 * 90, 72, 0), (4, 1, 64 * 90, 73, 1), (5, 1, 64 * 90, 37, 1), (28, 4, 4700, 0, 0), (32, 1, 4700, 0, 1), (8, 1, 18000, 0, 1)):
        info, items = _plan(exe, Hq, Hkv, [(P, 1), (100, 1), (0, 1)], splits=splits)
        _check_plan(info, items, Hq, Hkv, [(P, 1), (100, 1), (0, 1)])
        _check_slots(info, items, Hq, 128, [(P, 1), (100, 1), (0, 1)])
        assert info["decode"] and info["merges"] == merged, (Hq, Hkv, P, info["max_splits"])
    info, items = _plan(exe, 32, 1, [(18000, 1)])
    assert info["max_splits"] == -(-18000 // 128)          # ranges of two tiles: no fewer partials than CUs to read keys with


def test_fp32_partials_are_folded_or_merged(exe):
    """Up to eight ranges of heads of 64 are combined inside the launch; more, heads of 128 and plans of least space by the
    merge launch, from slots that are evenly spaced or, for one long query among short ones, packed."""
    for D, PS, splits, merged, even in ((64, [(1000, 60)] * 2, 8, 0, 0), (64, [(1000, 60)] * 2, 9, 1, 1), (128, [(1000, 60)] * 2, 2, 1, 1),
                                        (64, [(10, 60), (1300, 5)], 16, 1, 0), (128, [(10, 60), (1300, 5)], 16, 1, 0), (64, [(500, 60)], 1, 0, 0)):
        info, items = _plan(exe, 8, 2, PS, splits=splits, dtype=0, D=D)
        _check_plan(info, items, 8, 2, PS, dtype=0)
        assert info["max_splits"] == splits and (info["merges"], info["part_stride"] > 0) == (merged, bool(even)), (D, PS, splits)
        if splits > 1:
            _check_slots(info, items, 8, D, PS)


@pytest.mark.parametrize("dtype,kernel", [(0, 0), (1, 5)])
def test_partitions_are_not_limited_by_the_addresses_of_the_fold(exe, dtype, kernel):
    """A forced partition count is what a caller asked for, up to the key tiles, whatever the number of heads: where the
    partials of a row tile cannot be addressed inside the launch, the merge launch combines them."""
    for Hq, Hkv, P, splits, merged in ((128, 1, 64 * 1200 - 1, 1200, 1), (128, 1, 64 * 1200 - 1, 8, 0), (15000, 15000, 64 * 8 - 1, 8, 0),
                                       (16384, 16384, 64 * 8 - 1, 8, 1)):
        info, items = _plan(exe, Hq, Hkv, [(P, 1)], dtype=dtype, kernel=kernel, splits=splits, D=128 if dtype else 64)
        assert info["ok"] and not info["decode"] and (info["max_splits"], info["merges"]) == (splits, merged), (Hq, splits)


def test_counters_take_no_room_in_the_plan(exe):
    """The arrival counters are behind the plan where there is room and else in the work items: what fits the fixed workspace does not
    turn on how many (query, KV head) pairs are cut, and nothing but the items, the block table and (where a merge launch goes by it) the table of slots is uploaded."""
    for Hq, Hkv, n in ((32, 8, 640), (32, 8, 660), (28, 4, 790)):
        PS = [(17000, 1)] * n                    # two ranges each, in the plan of least space
        info, items = _plan(exe, Hq, Hkv, PS, within=(PLAN_INTS, WORKSPACE))
        assert info["decode"] and info["folds"] and info["max_splits"] == 2
        assert info["ints"] == len(items) * 32 + n * 1064 <= PLAN_INTS and info["part_floats"] <= WORKSPACE
    PS = [(1500, 100), (2800, 200), (700, 64), (3100, 256)]
    info, items = _plan(exe, 8, 2, PS, dtype=0, D=64)
    _check_plan(info, items, 8, 2, PS, dtype=0)
    up8 = lambda n: -(-n // 8) * 8
    nb, S = max(-(-(p + s) // 16) for p, s in PS), sum(s for _, s in PS)
    assert info["folds"] and info["ints"] == up8(4 * (-(-nb // 4) * 4)) + 3 * up8(4) + up8(S) + len(items) * 32


def test_counters_have_a_place_of_their_own_or_are_in_the_items(exe):
    """The batch of the GPU test of counters in the work items: its plan fits the fixed workspace, with the counters behind it it would not."""
    PS = [(620, 1)] * 64 + [(5120, 0)] + [(620, 0)] * 3096
    info, items = _plan(exe, 28, 4, PS, splits=4, within=(PLAN_INTS, WORKSPACE))
    _check_plan(info, items, 28, 4, PS)
    assert info["decode"] and info["folds"] and not info["compact"] and info["max_splits"] == 4
    assert info["ints"] <= PLAN_INTS < info["counters"] + info["counter_ints"]


def test_short_launches_that_gain_little_stay_with_the_other_kernels(exe):
    """Launches of 4 .. 14 us go to the long-launch kernel where its model is 20 % below the others': by 15 % it took the first four, each
    measured 2 .. 13 % slower in it; the fifth is 1.6 times as fast.  15 % are enough where nobody cuts the queries, or only this
    kernel does and they have the rows, as of the last three."""
    few = [416, 378, 842, 416, 794, 935, 416, 378, 795, 911, 911, 870]
    for Hq, Hkv, PS, want in ((32, 8, [(1168, 284)], 0), (28, 4, [(P, 60) for P in few], 0), (40, 8, [(1377, 239)], 0),
                              (28, 4, [(976, 154), (1258, 154)], 0), (32, 8, [(400, 226)] * 5, 1),
                              (32, 8, [(416, 269), (198, 324), (177, 297)], 1), (40, 8, [(265, 221), (160, 323)], 1),
                              (28, 4, [(654, 318), (454, 229), (436, 269)], 1)):
        info, items = _plan(exe, Hq, Hkv, PS)
        _check_plan(info, items, Hq, Hkv, PS)
        assert info["pingpong"] == want, PS
