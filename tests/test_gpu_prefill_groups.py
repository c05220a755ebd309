"""Prefill workgroups of key groups (option "prefill_groups"): the float64 oracle and the four-wave workgroups at the edges
of their tiles, steps and parts, and the planner's list of such tiles (CPU)."""
import numpy as np
import pytest

from oracle import ref_c
from paper_2511_21862_amd import binding as B
from paper_2511_21862_amd import workloads as W

HEADS = [(32, 8, 128), (28, 4, 128), (16, 1, 128), (4, 4, 128), (32, 4, 64), (4, 1, 64)]
FORCED, AUTO = 4 << 32, 0          # "prefill_groups" in the dry run's prefill_split


def dry(heads, q_lens, ctx_lens, **kw):
    ql, cx = np.asarray(q_lens, np.int32), np.asarray(ctx_lens, np.int32)
    qsl = np.zeros(len(ql) + 1, np.int32)
    qsl[1:] = np.cumsum(ql)
    return B.ooco_plan_dry_run(*heads, 16, 8192, 256, kw.pop("workspace", 128 << 20), cx + ql, qsl, cx, **kw)


@pytest.mark.parametrize("heads", HEADS, ids=str)
def test_tiles_of_64_columns_cover_every_row_once(heads):
    rows = 64 // (heads[0] // heads[1])
    rng = np.random.default_rng(heads[0])
    for q, c in (([2], [0]), ([rows, rows + 1, 2 * rows - 1], [0, 127, 4000]), (rng.integers(2, 90, size=7), rng.integers(0, 9000, size=7))):
        for split, parts in ((FORCED, 0), (FORCED + 3, 3), (AUTO + 1, 1)):
            r = dry(heads, q, c, prefill_split=split)
            t = r["prefill_tiles"]
            for i, (n, cx) in enumerate(zip(q, c)):
                mine = t[t[:, 0] == i]
                mine = mine[np.argsort(mine[:, 1])]
                assert mine[:, 2].sum() == n and (mine[:, 3] == cx + np.r_[0, np.cumsum(mine[:-1, 2])]).all()
                steps = (mine[:, 3] + mine[:, 2] + 127) // 128
                if split >> 32 == 4:
                    assert (mine[:-1, 2] == rows).all() and (mine[:, 4] >= 1).all() and (mine[:, 4] <= np.minimum(steps, 64)).all()
                    assert parts == 0 or (mine[:, 4] == np.minimum(parts, steps)).all()
            # the parts fit the units, and the workspace bounds them
            if parts == 0:
                assert t[:, 4].sum() * heads[1] <= max(256, len(t) * heads[1])
        small = dry(heads, q, c, prefill_split=FORCED, workspace=20 * 64 * (heads[2] + 2) * 4)
        split_tiles = small["prefill_tiles"][small["prefill_tiles"][:, 4] > 1]
        assert split_tiles[:, 4].sum() * heads[1] <= 20


def test_key_groups_are_planned_where_they_pay():
    rows4 = lambda q, c, heads=(32, 8, 128), **kw: int(dry(heads, q, c, prefill_split=AUTO, **kw)["prefill_tiles"][:, 2].max())
    # the dry run without them keeps the four-wave tiles
    assert dry((32, 8, 128), [40], [1000], prefill_groups=1)["prefill_tiles"][:, 2].max() == 32
    assert rows4([40], [1000]) == 16
    # three steps (head_dim 64: two) at least, at most one workgroup per unit
    assert rows4([40], [216]) == 32 and rows4([40], [217]) == 16
    assert rows4([16], [112], (32, 4, 64)) == 16 and rows4([16], [113], (32, 4, 64)) == 8
    assert rows4([512], [300]) == 16 and rows4([513], [300]) == 32
    # a load of 10 steps per unit; up to 25 for few tiles without many unused columns
    assert rows4([512], [760]) == 16 and rows4([512], [900]) == 32
    assert rows4([128], [8192]) == 16 and rows4([144], [8192]) == 32
    assert rows4([64], [12000]) == 16 and rows4([16], [40000]) == 16 and rows4([18], [40000]) == 18 and rows4([18] * 4, [12000] * 4) == 18
    # beside decode work: where every decode sequence finds a unit, three steps (four where one wave holds all columns), and
    # the decode part does not decide the time by itself; any load where tiles stay whole ("prefill_split" 1)
    assert rows4([40, 1], [1000, 50]) == 16 and rows4([40, 1], [216, 50]) == 32 and rows4([8, 1], [370, 50]) == 8
    assert dry((32, 8, 128), [8, 1], [370, 50], prefill_split=AUTO)["prefill_tiles"][0, 2] == 8
    assert rows4([40] + [1] * 8, [1000] + [50] * 8) == 16 and rows4([40] + [1] * 30, [1000] + [50] * 30) == 32
    assert rows4([40] + [1] * 4, [1000] + [8000] * 4) == 32
    whole = lambda q, c: int(dry((32, 8, 128), q, c, prefill_split=AUTO + 1)["prefill_tiles"][:, 2].max())
    assert rows4([300, 1], [16000, 50]) == 32 and whole([300, 1], [16000, 50]) == 16 and whole([300], [16000]) == 16
    # what the cooperative decode workgroups do not take
    assert dry((32, 8, 128), [40, 1], [1000, 50], prefill_split=AUTO, decode_tail_pct=20)["prefill_tiles"][:, 2].max() == 32


@pytest.mark.parametrize("heads", HEADS, ids=str)
def test_decode_parts_beside_key_groups_cover_every_block_on_the_units_that_are_left(heads):
    rng = np.random.default_rng(5)
    for n, top in ((1, 40), (3, 769), (9, 5000), (20, 300)):
        if (n + 3) * heads[1] > 256:
            continue
        lens = rng.integers(1, top, size=n)
        q, c = [3] + [1] * n, [3000] + [int(x) for x in lens]
        for split in (FORCED, FORCED + 1):
            r = dry(heads, q, c, prefill_split=split)
            p = r["decode_pieces"]
            for i in range(n):
                mine = sorted((int(x[1]), int(x[2])) for x in p if x[0] == i + 1)
                assert mine[0][0] == 0 and mine[-1][1] == (c[i + 1] + 1 + 15) // 16 and all(a[1] == b[0] for a, b in zip(mine, mine[1:]))
            wgs = r["decode_runs"] * heads[1] + int(r["prefill_tiles"][:, 4].sum()) * heads[1]
            assert wgs <= 256 and r["slots"] in (0, r["decode_runs"] + n + 1)


def batch(heads, q_lens, ctx_lens, seed):
    seq = np.asarray(q_lens) + np.asarray(ctx_lens)
    return W.build_batch(Hq=heads[0], Hkv=heads[1], hd=heads[2], q_lens=q_lens, ctx_lens=ctx_lens,
                         num_blocks=int(((seq + 15) // 16).sum()) + 5, seed=seed, poison=True)


@pytest.mark.gpu
@pytest.mark.parametrize("heads", HEADS, ids=str)
def test_edges_of_tiles_and_steps(heads):
    from gpu_util import assert_parity, run_gpu, say
    rows = 64 // (heads[0] // heads[1])
    # rows: one wave's columns, a tile and one more; keys: the edges of a group's 32 and of a step's 128
    q = [2, max(2, rows // 2), max(2, rows // 2 + 1), rows, rows + 1, 2 * rows + 1, 3]
    for c in ([0, 30, 31, 126, 127, 128, 300], [29, 0, 93, 1000, 255, 17, 2047]):
        b = batch(heads, q, c, seed=61)
        want = ref_c.attn_mixed(b.q, b.k_cache, b.v_cache, b.block_tables, b.seq_lens, b.query_start_loc, b.ctx_lens)
        for opts in ({}, {"prefill_split": 1}, {"prefill_split": 2}, {"prefill_split": 16}, {"prefill_split": 3, "prefill_sorted": 0}):
            say(f"case: {heads} q={q} ctx={c} {opts}")
            assert_parity(run_gpu(b, options=dict(opts, prefill_groups=4)), want, str(opts))


@pytest.mark.gpu
@pytest.mark.parametrize("heads,rows,ctx", [((28, 4, 128), 3, 17000), ((4, 1, 64), 9, 25000)], ids=str)
def test_more_parts_than_sixteen_and_a_small_workspace(heads, rows, ctx):
    from gpu_util import assert_parity, run_gpu, say
    b = batch(heads, [rows], [ctx], seed=62)
    want = ref_c.attn_mixed(b.q, b.k_cache, b.v_cache, b.block_tables, b.seq_lens, b.query_start_loc, b.ctx_lens)
    with B.Context(*heads, 16, b.num_blocks, b.max_blocks_per_seq) as ctx_:
        ctx_.plan(b.seq_lens, b.query_start_loc, b.ctx_lens)
        assert ctx_.plan_info()["prefill_parts"] > 16 and ctx_.plan_kernels() == [f"prefill_kernel_groups<{heads[2]}>"]
        say(f"case: {heads} {rows} rows on {ctx} tokens, {ctx_.plan_info()}")
        outs = [run_gpu(b, ctx=ctx_) for _ in range(3)]       # (the arrival counters are clean for every call)
    assert_parity(outs[0], want, "many parts")
    assert all(np.array_equal(o, outs[0]) for o in outs[1:])
    for ws in (0, 1 << 20):
        assert_parity(run_gpu(b, workspace_bytes=ws or 256), want, f"workspace {ws}")


@pytest.mark.gpu
@pytest.mark.parametrize("heads", HEADS, ids=str)
def test_step_of_key_groups_and_eight_wave_decode_workgroups(heads):
    from gpu_util import assert_parity, run_gpu, say
    g = heads[0] // heads[1]
    # decode sequences whole, cut, of one block and of none of the waves' second step; an empty sequence; two chunks
    for q, c in (([1, 5, 1, 0, 1], [15, 700, 255, 9, 256]), ([1, 64 // g + 1, 1, 2, 1], [5000, 1000, 767, 3000, 770])):
        if (len(q) + 3) * heads[1] > 256:
            continue
        b = batch(heads, q, c, seed=63)
        want = ref_c.attn_mixed(b.q, b.k_cache, b.v_cache, b.block_tables, b.seq_lens, b.query_start_loc, b.ctx_lens)
        with B.Context(*heads, 16, b.num_blocks, b.max_blocks_per_seq) as ctx:
            ctx.set_option("prefill_groups", 4)
            ctx.plan(b.seq_lens, b.query_start_loc, b.ctx_lens)
            assert ctx.plan_kernels() == [f"step_kernel_groups<{heads[2]}, {256 // heads[2]}>"]
        outs = []
        for opts in ({}, {"overlap": 0}, {"overlap": 2}, {"mixed_step": 0}, {"trace": 1}, {"prefill_split": 1}, {"prefill_split": 4}):
            say(f"case: {heads} q={q} ctx={c} {opts}")
            outs.append(run_gpu(b, options=dict(opts, prefill_groups=4)))
            assert_parity(outs[-1], want, str(opts))
        assert all(np.array_equal(o, outs[0]) for o in outs[1:5])       # one launch gives the bits of two
        for ws in (1 << 20, 4096):                                       # too small for the plan: the four-wave workgroups
            assert_parity(run_gpu(b, options={"prefill_groups": 4}, workspace_bytes=ws), want, f"workspace {ws}")


# (one workgroup per tile whatever its length: key groups from eight steps of 128 keys on also beside more decode sequences
# than units; 7 and 8 steps, decodes whole and cut, of one block and empty)
@pytest.mark.gpu
@pytest.mark.parametrize("heads", [(32, 8, 128), (28, 4, 128), (32, 4, 64), (64, 8, 128)], ids=str)
@pytest.mark.parametrize("keys", [896, 897, 2500])
def test_static_entry_with_more_decode_sequences_than_units(heads, keys):
    import torch
    from gpu_util import assert_parity, device_meta, say
    rng = np.random.default_rng(keys)
    n = 256 // heads[1] + 9
    q = [1] * n + [2, 21]
    ctx = rng.integers(0, 300, size=n).tolist() + [keys - 2, keys - 700]
    ctx[3], ctx[5] = 0, 1900
    ql, cx = np.asarray(q), np.asarray(ctx)
    b = W.build_batch(Hq=heads[0], Hkv=heads[1], hd=heads[2], q_lens=q, ctx_lens=ctx, num_blocks=int(((ql + cx + 15) // 16).sum()) + 5,
                      seed=91, poison=True)
    want = ref_c.attn_mixed(b.q, b.k_cache, b.v_cache, b.block_tables, b.seq_lens, b.query_start_loc, b.ctx_lens)
    d, meta = W.to_device(b), device_meta(b)
    for _ in range(3):
        say(f"case: {heads} {n} decodes, {keys} keys")
        out = torch.full((b.total_q, b.Hq, b.hd), float("nan"), dtype=torch.bfloat16, device="cuda")
        B.ooco_attn_mixed_static(*heads, 16, b.max_blocks_per_seq, 0.0, b.seq_lens, b.query_start_loc, b.ctx_lens, d.q, d.k_cache,
                                 d.v_cache, *meta, out, b.num_seqs, b.total_q)
        torch.cuda.synchronize()
        assert_parity(out.view(torch.int16).cpu().numpy().view(np.uint16), want, "static")
