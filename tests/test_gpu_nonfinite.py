"""NaN and infinities in q and K, prefill and decode: what is not finite stays in the (row, head) whose scores it reaches.  The columns of a
wave share matrix products, in which 0 * NaN and 0 * inf are NaN, so every column of the batch that has only finite scores is
compared with the float64 oracle, and every other one has to be NaN there and here."""
import numpy as np
import pytest

from oracle import ref_c
from paper_2511_21862_amd import binding as B
from paper_2511_21862_amd import workloads as W

pytestmark = pytest.mark.gpu

NAN, INF = 0x7FC0, 0x7F80
# options, decode sequences beside the chunks, the kernel's name
FORMS = [({"prefill_groups": 1, "prefill_split": 1}, 0, "prefill_kernel<"), ({"prefill_groups": 1, "prefill_split": 3}, 0, "prefill_kernel<"),
         ({"prefill_groups": 1, "prefill_split": 5}, 0, "prefill_kernel<"), ({"prefill_sorted": 0}, 0, "prefill_kernel<"),
         ({"prefill_groups": 1, "prefill_waves": 8}, 0, "prefill_kernel<"),
         ({"prefill_groups": 4, "prefill_split": 1}, 0, "prefill_kernel_groups<"), ({"prefill_groups": 4, "prefill_split": 2}, 0, "prefill_kernel_groups<"),
         ({"prefill_groups": 1, "mixed_step": 2}, 3, "step_kernel<"), ({"prefill_groups": 4, "mixed_step": 2}, 3, "step_kernel_groups<"),
         ({"mixed_fused": 1}, 3, "mixed_kernel<"), ({"mixed_lean": 2}, 3, "lean")]


def batch(heads, decodes):
    Hq, Hkv, hd = heads
    return W.build_batch(Hq=Hq, Hkv=Hkv, hd=hd, q_lens=[75, 40, 9] + [1] * decodes, ctx_lens=[30, 700, 0] + [90] * decodes, num_blocks=80, seed=23, poison=True)


def query_columns(b, value, dims):
    # the first, a middle and the last column of the halves that a product holds side by side, in different waves
    g = b.Hq // b.Hkv
    for c in (0, 32 + 15, 64 + 16, 96 + 31, 160 + 5):
        b.q[c // g, c % g, dims] = value
    b.q[75 + 39, b.Hq - 1, dims] = value          # the last row of the second chunk


def key(b, value):
    # of a token that the earlier rows of its chunk do not see, one kv head; and of one in the middle of the next chunk's first tile
    for seq, token in ((0, 30 + 20), (1, 700 + 13)):
        k, v = W.gather_logical(b, seq)
        k = k.copy()
        k[token, b.Hkv - 1, 3] = value
        W.scatter_logical(b, seq, k, v)


KINDS = {"nan query": lambda b: query_columns(b, NAN, slice(None)), "nan of one dim": lambda b: query_columns(b, NAN, 5),
         "inf query": lambda b: query_columns(b, INF, 7), "nan key": lambda b: key(b, NAN), "inf key": lambda b: key(b, INF)}


@pytest.mark.parametrize("kind", KINDS)
@pytest.mark.parametrize("heads", [(16, 4, 128), (14, 2, 128), (16, 2, 64), (6, 2, 64)], ids=str)
def test_other_columns_stay_finite(heads, kind):
    from gpu_util import MAX_ABS, MEAN_ABS, REL_L2, run_gpu, say
    wrong = []
    for decodes in (0, 3):
        b = batch(heads, decodes)
        KINDS[kind](b)
        want = ref_c.attn_mixed(b.q, b.k_cache, b.v_cache, b.block_tables, b.seq_lens, b.query_start_loc, b.ctx_lens)
        lost = np.isnan(want).all(axis=2)                       # (row, head)
        if kind == "inf key":
            # a score of +inf is lost, one of -inf is a weight of 0: by the query's sign in that dim
            assert lost.any() and not lost.all()
        assert lost.any() and lost.mean() < 0.4 and (np.isnan(want).any(axis=2) == lost).all()
        for opts, n, name in FORMS:
            if n != decodes or (heads[2] == 64 and "mixed_lean" in opts):   # (the lean pair: head_dim 128)
                continue
            say(f"case: {heads} {kind} {opts}")
            with B.Context(*heads, 16, b.num_blocks, b.max_blocks_per_seq) as ctx:
                for k, v in opts.items():
                    ctx.set_option(k, v)
                ctx.plan(b.seq_lens, b.query_start_loc, b.ctx_lens)
                kernels = ";".join(ctx.plan_kernels())
                assert name in kernels, (opts, kernels)
                got = W.bf16_bits_to_f32(run_gpu(b, ctx=ctx, plan=False)).astype(np.float64)
            assert np.isnan(got[lost]).all(), (opts, "a lost column is not NaN")
            fine = got[~lost]
            if not np.isfinite(fine).all():
                wrong.append((opts, "other columns not finite", np.argwhere(~np.isfinite(got).all(axis=2) & ~lost)[:6].tolist()))
                continue
            diff = np.abs(fine - want[~lost])
            rel = np.sqrt((diff ** 2).sum() / (want[~lost] ** 2).sum())
            if diff.max() > MAX_ABS or diff.mean() > MEAN_ABS or rel > REL_L2:
                wrong.append((opts, diff.max(), diff.mean(), rel))
    for w in wrong:
        say(f"  {w}")
    assert not wrong


@pytest.mark.parametrize("kind", ["nan query", "inf query", "nan key", "inf key"])
@pytest.mark.parametrize("heads", [(32, 4, 128), (14, 2, 128), (16, 2, 64)], ids=str)
def test_other_heads_of_a_decode_row_stay_finite(heads, kind):
    from gpu_util import MAX_ABS, REL_L2, run_gpu, say
    Hq, Hkv, hd = heads
    b = W.build_batch(Hq=Hq, Hkv=Hkv, hd=hd, q_lens=[1] * 5, ctx_lens=[3, 60, 333, 900, 2600], num_blocks=300, seed=29, poison=True)
    value = NAN if "nan" in kind else INF
    if "query" in kind:
        b.q[1:, 1, 9] = value
        b.q[0, Hq - 1, 9] = value
    else:
        for seq, token in ((1, 60), (2, 0), (3, 500), (4, 2599)):
            k, v = W.gather_logical(b, seq)
            k = k.copy()
            k[token, 0, 3] = value
            W.scatter_logical(b, seq, k, v)
    want = ref_c.attn_mixed(b.q, b.k_cache, b.v_cache, b.block_tables, b.seq_lens, b.query_start_loc, b.ctx_lens)
    lost = np.isnan(want).all(axis=2)
    assert lost.any() and not lost.all() and (np.isnan(want).any(axis=2) == lost).all()
    for opts in ({}, {"decode_coop": 0}, {"decode_coop": 2}, {"decode_coop": 0, "decode_segments": 7}, {"decode_coop": 0, "decode_segments": 60}):
        say(f"case: {heads} {kind} {opts}")
        got = W.bf16_bits_to_f32(run_gpu(b, options=opts)).astype(np.float64)
        assert np.isnan(got[lost]).all() and np.isfinite(got[~lost]).all(), opts
        diff = np.abs(got[~lost] - want[~lost])
        assert diff.max() <= MAX_ABS and np.sqrt((diff ** 2).sum() / (want[~lost] ** 2).sum()) <= REL_L2, opts
