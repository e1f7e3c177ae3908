"""Launch rules, on the CPU."""
import random

import pytest

from launch_rules import ask

LONG, MID, HALF, QUARTER, SHORT, TINY, PAIR, THIN = range(8)  # WideShape


def test_quantization_streams_large_inputs_only():
    # inputs that the kernel before has left in the caches lose by it below 64 MB
    short = [(64, 14336), (512, 8192), (2048, 3072), (16384, 256), (65535, 256)]
    assert ask(*(("quant_streams", m, k) for m, k in short)) == [[0]] * len(short)
    assert ask(("quant_streams", 65536, 256), ("quant_streams", 8192, 4096)) == [[1], [1]]


def test_quantization_workgroups_cover_rows_and_fit_the_grid():
    # a grid holds 2^32 - 1 threads; one long matrix among many short rows must
    # not push a grouped launch past it that 256 threads per row keep
    rows = [1, 64, (1 << 23) - 1, 1 << 23, (1 << 23) + 1, (1 << 24) - 1]
    ks = [4, 2048, 2052, 4096, 4100, 8192, 8196, 16384, 16388, 32768, 32772, 174720]
    cases = [(m, k) for m in rows for k in ks]
    for (m, k), (threads, pieces) in zip(cases, ask(*(("quant_shape", m, k) for m, k in cases))):
        assert m * threads < 1 << 32, (m, k)
        assert pieces == 0 or 4 * threads * pieces >= k, (m, k)
        assert threads == (256 if k <= 8192 or m >= 1 << 23 else 512), (m, k)


def test_window_kernel_splits_only_rows_that_gain():
    # (units, blocks, per-group scales)
    cases = [(1, 9, 0), (3, 128, 0), (4, 128, 0), (4, 9, 1), (8, 9, 1), (7, 129, 0), (8, 192, 0),
             (8, 192, 1), (12, 192, 1), (12, 193, 0), (112, 256, 0)]
    assert [v for v, in ask(*(("sm_splits",) + c for c in cases))] == [0, 0, 1, 0, 1, 0, 1, 0, 1, 0, 0]


def test_whole_rows_spread_over_the_gpu():
    # workgroup b goes to XCD b % 8 and there, in turn, to one of four engines
    subs = [v for v, in ask(*(("sm_whole_sub", b) for b in range(256)))]
    b = [4 * blk + sub for blk, sub in enumerate(subs)]
    places = [(v % 8, v // 8 % 4) for v in b]
    assert len(set(places)) == 32 and max(map(places.count, set(places))) <= 2 * 256 // 32


def test_xcd_order_is_a_permutation_in_eighths():
    for grid in (1, 7, 8, 9, 64, 203):
        blocks, = ask(("xcd_block", grid))
        assert sorted(blocks) == list(range(grid))
        for x in range(min(8, grid)):  # an XCD's blocks are neighbours, in order
            mine = blocks[x::8]
            assert mine == list(range(mine[0], mine[0] + len(mine)))


# blocks of a grouped launch, shape, workgroups per block, and the most tile
# groups that one workgroup may run in series
LAUNCHES = [(64, LONG, 1, 2), (64, MID, 2, 1), (64, HALF, 4, 1), (64, SHORT, 16, 1),
            (32, THIN, 2, 1), (32, PAIR, 4, 1), (32, SHORT, 8, 1),
            (33, MID, 1, 1), (33, HALF, 1, 1), (33, PAIR, 2, 1), (33, SHORT, 4, 1),
            # products without scales beside them
            (32, THIN, 1, 2)]


@pytest.mark.parametrize("kind,shape,per,series", LAUNCHES)
def test_grouped_workgroups_cover_every_product_once(kind, shape, per, series):
    rng = random.Random(kind * 100 + shape)
    launches = [[(m, R)] for m in (1, 31, 32, 33, 64, 65, 96, 127, 128, 129, 193) for R in (1, 3, 4, 5, 8, 13)]
    launches += [[(rng.choice([1, 17, 33, 65, 97, 129, 200]), rng.randint(1, 20)) for _ in range(6)]
                 for _ in range(40)]
    answers = ask(*(("cover", kind, shape, per) + tuple(v for p in ps for v in p) for ps in launches))
    for ps, (bad, most, active) in zip(launches, answers):
        assert bad == 0 and most <= series and active > 0, ps
        if shape == LONG and all(-(-m // 64) % 2 == 0 for m, _ in ps):
            assert most == 1, ps  # only an odd last token block is run in series


def test_no_shape_that_a_launch_leaves_half_idle():
    # 64-token workgroups with per-group scales take two 32-token blocks, which
    # launches of fewer than 32 tokens do not have
    totals = list(range(1, 4000, 7))
    few = ask(*(("wide_pick_batched_group", t, c, 31) for t in totals for c in (1, 9)))
    assert {v for v, in few} == {PAIR, SHORT}
    # 128-token workgroups run an odd last token block in twice the time: no
    # shape for few rounds of an odd number of token blocks
    for total in range(129, 513):
        (five,), (four,) = ask(("wide_pick_batched", total, 276), ("wide_pick_batched", total, 256))
        assert five == MID and four in (LONG, MID), total


def test_lines_of_the_grouped_shapes():
    # lines moved here move what the GPU cases below run
    def lines(name, *args):
        picks = [v for v, in ask(*((name, t) + args for t in range(1, 2100)))]
        return [(t + 1, p) for t, p in enumerate(picks) if t == 0 or picks[t - 1] != p]
    assert lines("wide_pick_batched32") == [(1, SHORT), (97, PAIR), (193, THIN)]
    assert lines("wide_pick_batched_group", 4, 32) == \
        [(1, SHORT), (129, PAIR), (769, HALF), (1537, MID)]
    assert lines("wide_pick_batched_group", 3, 32) == [(1, SHORT), (129, PAIR), (769, MID)]
    assert lines("wide_pick_batched", 64)[:3] == [(1, SHORT), (33, HALF), (65, MID)]
    assert lines("wide_pick_batched", 128)[:4] == [(1, SHORT), (33, HALF), (65, MID), (129, LONG)]


def test_gpu_cases_reach_every_shape():
    """The shapes that the GPU cases of the register-decoded kernel run."""
    pytest.importorskip("torch")
    import test_gpu_wide as wide
    lone = ask(*(("wide_pick",) + s for s in wide.LONE))
    assert {v for v, in lone} == {LONG, MID, HALF, QUARTER, SHORT, TINY}
    for aligned in (True, False):
        pieces = [aligned and -(-k // 128) % 4 == 0 for _, _, k in wide.LONE_GROUP]
        picks = ask(*(("wide_pick_group",) + s + (int(p),) for s, p in zip(wide.LONE_GROUP, pieces)))
        for chunk in ((True, False) if aligned else (False,)):
            assert {v for (v,), p in zip(picks, pieces) if p == chunk} == {MID, HALF, SHORT, TINY, PAIR}
    # grouped: the blocks that prepare counts, and the largest m
    def blocks(products, group):
        tok = wide_tokens(products, group)
        return sum(-(-(-(-n // 64)) // (4 if g else 8)) * -(-m // tok) for m, n, _, g in products)

    def wide_tokens(products, group):
        return 32 if group or max(m for m, _, _, _ in products) <= 32 else 64
    got = set()
    for shapes, low, high in wide.GROUPED:
        ps = [s + (False,) for s in shapes]
        total = blocks(ps, False)
        assert low <= total <= high
        got.add(ask(("wide_pick_batched", total, max(m for m, _, _ in shapes)))[0][0])
    assert got == {SHORT, HALF, MID, LONG}
    got, with_groups, beside = set(), set(), set()
    for shapes, low, high in wide.GROUPED32:
        group = any(g for _, _, _, g in shapes)
        total = blocks(shapes, group)
        assert low <= total <= high
        if not group:
            got.add(ask(("wide_pick_batched32", total))[0][0])
        else:
            v = ask(("wide_pick_batched_group", total, len(shapes),
                     max(m for m, _, _, _ in shapes)))[0][0]
            with_groups.add(v)
            if not all(g for _, _, _, g in shapes):
                beside.add(v)
    assert got == {SHORT, PAIR, THIN} and with_groups == {SHORT, PAIR, HALF, MID} == beside
