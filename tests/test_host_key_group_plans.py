"""Plans of key groups beside decode work (CPU: the planner's dry run): what the kernels will write of partial results lies
inside the workspace, whatever "decode_segments" asks for."""
import numpy as np
import pytest

from paper_2511_21862_amd import binding as B

FORCED, AUTO = 4 << 16, 15 << 16          # "prefill_groups" in the dry run's prefill_split


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
