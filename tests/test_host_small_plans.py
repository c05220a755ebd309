"""Plans of small decode batches and of prefill parts hidden behind a decode part (CPU: the planner's dry run)."""
import numpy as np
import pytest

from paper_2511_21862_amd import binding as B


def dry(heads, q_lens, ctx_lens, **kw):
    ql, cx = np.asarray(q_lens, np.int32), np.asarray(ctx_lens, np.int32)
    qsl = np.zeros(len(ql) + 1, np.int32)
    qsl[1:] = np.cumsum(ql)
    return B.ooco_plan_dry_run(*heads, 16, 8192, 256, kw.pop("workspace", 128 << 20), cx + ql, qsl, cx, **kw)


def check_cover(r, q_lens, ctx_lens):
    pieces = r["decode_pieces"]
    for i, (q, c) in enumerate(zip(q_lens, ctx_lens)):
        mine = sorted((int(p[1]), int(p[2])) for p in pieces if p[0] == i)
        if q != 1:
            assert not mine
            continue
        assert mine[0][0] == 0 and mine[-1][1] == (c + 1 + 15) // 16 and all(a[1] == b[0] for a, b in zip(mine, mine[1:]))


@pytest.mark.parametrize("heads,limit", [((32, 8, 128), 768), ((28, 4, 128), 768), ((32, 4, 64), 1536)])
def test_short_sequences_are_taken_whole_up_to_the_limit(heads, limit):
    for longest, whole in ((limit, True), (limit + 1, False)):
        q, c = [1, 1, 20, 1], [longest - 1, 33, 100, 0]
        r = dry(heads, q, c)
        assert (r["decode_runs"] == len(q) and all(int(p[3]) < 0 for p in r["decode_pieces"])) == whole
        check_cover(r, q, c)
    # four workgroups per unit, two beside a prefill part
    per_unit = 256 // heads[1]
    for n, chunk, whole in ((4 * per_unit, 0, True), (4 * per_unit + 1, 0, False), (2 * per_unit - 1, 1, True), (2 * per_unit, 1, False)):
        q, c = [1] * n + [20] * chunk, [63 + i % 9 for i in range(n)] + [0] * chunk
        r = dry(heads, q, c)
        assert all(int(p[3]) < 0 for p in r["decode_pieces"]) == whole and (r["decode_runs"] == n + chunk) == whole
        check_cover(r, q, c)


def whole(heads, lens, chunk=None):
    q, c = [1] * len(lens), [n - 1 for n in lens]
    if chunk:
        q.append(chunk[0])
        c.append(chunk[1])
    r = dry(heads, q, c)
    check_cover(r, q, c)
    return r["decode_runs"] == len(q) and all(int(p[3]) < 0 for p in r["decode_pieces"]) and \
        [int(p[4]) for p in sorted(r["decode_pieces"], key=lambda p: p[4])] == [i for i, x in enumerate(q) if x == 1]


def mixed_lengths(n, longest, shortest=None):
    return [longest] + [(shortest or longest // 2) + 16 * (i % 3) for i in range(n - 1)]


@pytest.mark.parametrize("heads", [(32, 8, 128), (64, 8, 128), (32, 32, 128), (32, 4, 64)], ids=lambda h: "-".join(map(str, h)))
def test_batches_of_several_workgroups_per_unit(heads):
    # measured against single waves: equal lengths only up to one workgroup per unit with head_dim 128 (single waves, one run
    # per sequence, cut nothing there either), long outliers up to 1.5, more than two per unit by the group's size
    per_unit, hd, g = 256 // heads[1], heads[2], heads[0] // heads[1]
    n = lambda r: int(per_unit * r)
    assert whole(heads, [240] * n(1)) and whole(heads, mixed_lengths(n(1), 700, 64))
    # (a line of equal sequences in as many runs as sequences cuts nothing, but its workgroups would be cooperative)
    for r in (1.5, 2):
        assert whole(heads, mixed_lengths(n(r), 500))
        assert whole(heads, mixed_lengths(n(r), 600 * 128 // hd, 64)) == (r <= 1.5)
        assert whole(heads, mixed_lengths(n(r) - 1, 600 * 128 // hd, 64), (40, 100))
    assert whole(heads, mixed_lengths(n(4), 100)) and not whole(heads, mixed_lengths(n(4) + per_unit // 8, 100))
    assert whole(heads, mixed_lengths(n(4), 600)) == (g >= 6)
    assert whole(heads, mixed_lengths(n(2.5), 600)) == (g >= 4)
    assert not whole(heads, mixed_lengths(n(3) - 1, 100), (40, 100))


@pytest.mark.parametrize("heads,n,longest,runs", [((64, 8, 128), 24, 1000, 48), ((32, 8, 128), 40, 768, 40), ((32, 8, 128), 35, 1536, 64),
                                                  ((32, 32, 128), 12, 1000, 12), ((32, 8, 128), 48, 1536, 48)])
def test_equal_sequences_get_as_many_runs_each(heads, n, longest, runs):
    # ... unless that leaves too few waves for long sequences
    r = dry(heads, [1] * n, [longest - 1] * n)
    assert r["decode_runs"] == runs
    check_cover(r, [1] * n, [longest - 1] * n)
    if runs % n == 0:
        assert len(r["decode_pieces"]) == runs
    uneven = [longest - 1 - 16 * (i % 2) for i in range(n)]
    assert dry(heads, [1] * n, uneven)["decode_runs"] >= runs


@pytest.mark.parametrize("heads", [(32, 8, 128), (28, 4, 128), (32, 4, 64), (16, 1, 128)])
@pytest.mark.parametrize("workspace", [128 << 20, 1 << 20, 40000])
def test_lines_with_larger_pads_cover_every_block_once(heads, workspace):
    rng = np.random.default_rng(7)
    for n in (1, 2, 5, 16):
        q = [1] * n
        c = [int(x) for x in rng.integers(800, 6000, size=n)]
        if n > 2:
            q.insert(2, 50)
            c.insert(2, 17)
        check_cover(dry(heads, q, c, workspace=workspace), q, c)


def test_prefill_parts_hidden_behind_a_long_decode_part_stay_few():
    dec = [2250] * 48
    alone = dry((32, 8, 128), [60] * 4, [1500] * 4, prefill_groups=1)["prefill_parts"]
    beside = dry((32, 8, 128), [60] * 4 + [1] * 48, [1500] * 4 + dec, prefill_groups=1)["prefill_parts"]
    few = dry((32, 8, 128), [60] * 4 + [1] * 8, [1500] * 4 + dec[:8], prefill_groups=1)["prefill_parts"]
    assert beside < min(alone, few)
    # ... but a chunk that would outlast the decode part is still cut
    assert dry((32, 8, 128), [100] + [1] * 48, [10000] + dec)["prefill_parts"] >= 5


@pytest.mark.parametrize("heads,default,grown", [((32, 8, 128), 3, 12), ((32, 4, 64), 6, 24)])
def test_a_piece_pad_that_is_set_to_the_default_is_taken_as_it_is(heads, default, grown):
    # (cooperative plans charge a piece's start four times as much unless the option says otherwise)
    rng = np.random.default_rng(8)
    q, c = [1] * 16, [int(x) for x in rng.integers(2000, 4000, size=16)]
    pieces = lambda pad: dry(heads, q, c, decode_piece_pad=pad)["decode_pieces"].tolist()
    assert pieces(-1) == pieces(grown)
    assert pieces(default) != pieces(grown)
    check_cover(dry(heads, q, c, decode_piece_pad=default), q, c)


@pytest.mark.parametrize("heads", [(16, 1, 128), (28, 4, 128), (64, 8, 128), (32, 8, 128), (32, 4, 64)], ids=lambda h: "-".join(map(str, h)))
def test_one_long_sequence_among_short_ones_is_not_cut_into_crumbs(heads):
    # its parts are merged by one wave, one after the other
    rng = np.random.default_rng(9)
    n = 256 // heads[1]
    for longest in (2500, 8000):
        q, c = [1] * n, [int(x) for x in rng.integers(30, 250, size=n - 1)] + [longest - 1]
        r = dry(heads, q, c)
        check_cover(r, q, c)
        parts = sum(int(p[0]) == n - 1 for p in r["decode_pieces"])
        assert 4 <= parts <= (40 if longest == 8000 else 20), (longest, parts)


def test_parts_of_prefill_tiles_at_head_dim_64():
    # 32/4 heads of 64: whole tiles below 16 steps and from two workgroups per unit on, parts in between, never past three
    # workgroups per unit by more than one part per tile
    def plan(n, rows, ctx):
        ql, cx = np.full(n, rows, np.int32), np.full(n, ctx, np.int32)
        qsl = np.arange(n + 1, dtype=np.int32) * rows
        return B.ooco_plan_dry_run(32, 4, 64, 16, 4096, 256, 256 << 20, cx + ql, qsl, cx)
    for n, rows, ctx, want in ((1, 615, 1500, 3), (1, 1036, 1598, 2), (8, 112, 3800, 2), (8, 256, 768, 1), (8, 250, 700, 1)):
        r = plan(n, rows, ctx)
        t = r["prefill_tiles"]
        assert r["prefill_parts"] == want, (n, rows, ctx, r["prefill_parts"])
        assert t[:, 2].sum() == n * rows and t[:, 4].sum() * 4 <= 3 * 256 + 4 * len(t)
