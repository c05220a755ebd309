"""Plans of key groups (CPU: the planner's dry run): the dry run is what a context plans, and what the kernels will write of
partial results lies inside the workspace, whatever "decode_segments" asks for."""
import numpy as np
import pytest

from paper_2511_21862_amd import binding as B

FORCED, OFF, AUTO = 4 << 32, 1 << 32, 0          # "prefill_groups" in the dry run's prefill_split


def dry(heads, q_lens, ctx_lens, **kw):
    ql, cx = np.asarray(q_lens, np.int32), np.asarray(ctx_lens, np.int32)
    qsl = np.zeros(len(ql) + 1, np.int32)
    qsl[1:] = np.cumsum(ql)
    return B.ooco_plan_dry_run(*heads, 16, 8192, 256, kw.pop("workspace", 128 << 20), cx + ql, qsl, cx, **kw)


def workspace_used(r, heads):
    """Bytes of the decode slots and, 256-byte aligned behind them, of the prefill parts: 64 columns each in tiles of key
    groups.  (A tile of few rows may be one of four waves, whose parts have 128: then this is less than the plan uses.)"""
    Hq, Hkv, hd = heads
    t = r["prefill_tiles"]
    cols = 64 if int(t[:, 2].max()) * (Hq // Hkv) <= 64 else 128
    return (r["slots"] * Hq * (hd + 2) * 4 + 255) // 256 * 256 + int(t[t[:, 4] > 1][:, 4].sum()) * Hkv * cols * (hd + 2) * 4


@pytest.mark.parametrize("groups", [AUTO, FORCED])
@pytest.mark.parametrize("heads,q,ctx,segments,workspace", [((64, 8, 128), [40, 1, 1], [9000, 20000, 20000], 500, 16 << 20),
                                                            ((32, 8, 128), [2, 1, 1], [17000, 16000, 16000], 1500, 24 << 20)])
def test_forced_segments_beside_key_groups_fit_the_workspace(heads, q, ctx, segments, workspace, groups):
    r = dry(heads, q, ctx, prefill_split=groups, decode_segments=segments, workspace=workspace)
    assert workspace_used(r, heads) <= workspace
    if groups == AUTO:                     # the number of runs that the option asks for holds
        assert r["decode_runs"] == segments


def test_random_plans_fit_the_workspace_and_cover_every_block():
    rng = np.random.default_rng(20256)
    for case in range(4000):
        heads = [(32, 8, 128), (28, 4, 128), (64, 8, 128), (16, 1, 128), (32, 4, 64), (4, 1, 64)][rng.integers(6)]
        n = int(rng.integers(1, 1 + max(1, 40 // heads[1])))
        q = [int(x) for x in np.exp(rng.uniform(np.log(2), np.log(300), size=rng.integers(1, 4)))] + [1] * n
        c = [int(x) for x in 2.0 ** rng.uniform(4, 15, size=len(q))]
        kw = dict(workspace=int(2.0 ** rng.uniform(20, 28)) // 256 * 256, decode_segments=int(rng.choice([0, 1, 7, 150, 500, 1500])),
                  prefill_split=int(rng.choice([AUTO, FORCED, AUTO + 1, FORCED + 3])))
        r = dry(heads, q, c, **kw)
        assert workspace_used(r, heads) <= kw["workspace"], (case, heads, q, c, kw)
        for i in range(len(q) - n, len(q)):
            mine = sorted((int(p[1]), int(p[2])) for p in r["decode_pieces"] if p[0] == i)
            assert mine[0][0] == 0 and mine[-1][1] == (c[i] + 16) // 16 and all(a[1] == b[0] for a, b in zip(mine, mine[1:]))


@pytest.mark.parametrize("heads,chunks,cached,decodes,longest,taken", [
    ((32, 8, 128), [6], 1057, 42, 850, False), ((32, 8, 128), [6], 1250, 42, 850, True), ((32, 4, 64), [6], 1057, 84, 850, True),
    ((28, 4, 128), [21, 16], 970, 156, 290, False), ((28, 4, 128), [21, 16], 970, 120, 200, True),
    ((64, 8, 128), [55, 69, 83], 1700, 71, 118, False), ((64, 8, 128), [15, 19, 13], 1700, 71, 118, True)])
def test_key_groups_whose_decode_part_would_be_the_longer_one(heads, chunks, cached, decodes, longest, taken):
    # whole tiles beside more decode sequences than units: chains of eight and nine steps, and of more with few units left
    q, c = chunks + [1] * decodes, [cached] * len(chunks) + [longest // 4 + i * longest * 3 // (4 * decodes) for i in range(decodes)]
    plans = [dry(heads, q, c, prefill_split=split)["decode_pieces"].tolist() for split in (AUTO + 1, OFF + 1)]
    assert (plans[0] != plans[1]) == taken


def test_the_dry_run_takes_key_groups_as_a_context_does():
    rows = lambda **kw: int(dry((32, 8, 128), [40], [1000], **kw)["prefill_tiles"][:, 2].max())
    assert rows() == rows(prefill_groups=0) == rows(prefill_groups=4) == 16 and rows(prefill_groups=1) == 32
    assert rows(prefill_split=70000) == 32          # (forced parts: four waves, however many are asked for)
    for groups in (2, 3, 5, 15, 1 << 20):
        with pytest.raises(B.OocoError) as e:
            rows(prefill_groups=groups)
        assert e.value.status == B.OOCO_EINVAL


@pytest.mark.gpu
def test_the_dry_run_is_what_a_context_plans():
    import torch
    units = torch.cuda.get_device_properties(0).multi_processor_count
    rng = np.random.default_rng(20257)
    for case in range(150):
        heads = [(32, 8, 128), (28, 4, 128), (64, 8, 128), (16, 1, 128), (32, 4, 64), (4, 1, 64)][rng.integers(6)]
        q = [int(x) for x in np.exp(rng.uniform(np.log(2), np.log(600), size=rng.integers(0, 4)))] + [1] * int(rng.integers(0, 60))
        q = np.asarray(q or [1], np.int32)
        c = (2.0 ** rng.uniform(2, 14, size=len(q))).astype(np.int32)
        args = q + c, np.r_[0, np.cumsum(q)].astype(np.int32), c
        opts = dict(prefill_groups=int(rng.choice([0, 0, 1, 4])), prefill_split=int(rng.choice([0, 0, 1, 3])),
                    decode_segments=int(rng.choice([0, 0, 20])))
        r = B.ooco_plan_dry_run(*heads, 16, 2048, units, 128 << 20, *args, **opts)
        with B.Context(*heads, 16, 64, 2048) as ctx:
            for k, v in opts.items():
                ctx.set_option(k, v)
            ctx.plan(*args)
            info = ctx.plan_info()
        got = (info["decode_waves"], info["prefill_tiles"], info["prefill_parts"])
        assert got == (r["decode_runs"], len(r["prefill_tiles"]), r["prefill_parts"]), (case, heads, q, c, opts)


# 16/1 heads: chunks of a tile each; arrays of num_seqs + 1 and 2 * chunks + 1 + tiles entries, together up to 961
def two_kernels(chunks, decodes):
    return [3] * chunks + [1] * decodes, [1500 - 7 * i % 500 for i in range(chunks)] + [60 + 9 * i % 300 for i in range(decodes)]


@pytest.mark.parametrize("chunks,decodes,fit", [(180, 239, True), (180, 240, False), (235, 159, False)])
def test_decode_runs_of_plans_in_two_kernels_are_those_of_all_units(chunks, decodes, fit):
    q, c = two_kernels(chunks, decodes)
    r, four = (dry((16, 1, 128), q, c, prefill_split=groups + 1, workspace=32 << 20) for groups in (AUTO, OFF))
    assert chunks + decodes + 1 + 3 * chunks + 1 <= 961 if fit else chunks + decodes + 1 + 3 * chunks + 1 > 961
    assert r["decode_runs"] == 256 - chunks if fit else (r["decode_pieces"] == four["decode_pieces"]).all()


@pytest.mark.gpu
def test_two_kernels_beside_key_groups():
    import torch
    from gpu_util import assert_parity, device_meta, run_gpu, say
    from oracle import ref_c
    from paper_2511_21862_amd import workloads as W
    q, c = two_kernels(235, 159)
    b = W.build_batch(Hq=16, Hkv=1, hd=128, q_lens=q, ctx_lens=c, num_blocks=sum((x + y + 15) // 16 for x, y in zip(q, c)) + 5, seed=92,
                      poison=True)
    want = ref_c.attn_mixed(b.q, b.k_cache, b.v_cache, b.block_tables, b.seq_lens, b.query_start_loc, b.ctx_lens)
    d, meta = W.to_device(b), device_meta(b)
    say("case: static entry, arrays too large for one launch")
    out = torch.full((b.total_q, b.Hq, b.hd), float("nan"), dtype=torch.bfloat16, device="cuda")
    B.ooco_attn_mixed_static(16, 1, 128, 16, b.max_blocks_per_seq, 0.0, b.seq_lens, b.query_start_loc, b.ctx_lens, d.q, d.k_cache, d.v_cache,
                             *meta, out, b.num_seqs, b.total_q)
    torch.cuda.synchronize()
    assert_parity(out.view(torch.int16).cpu().numpy().view(np.uint16), want, "static")
    for opts in ({}, {"prefill_groups": 4}, {"prefill_split": 1}):
        say(f"case: plan {opts}")
        assert_parity(run_gpu(b, options=opts), want, str(opts))
