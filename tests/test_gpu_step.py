"""Batches with both kinds of work in one launch (the step kernel): same bits as the two kernels one after the other, and
the float64 oracle, at the edges of its launch rule."""
import numpy as np
import pytest
import torch

from oracle import ref_c
from paper_2511_21862_amd import binding as B
from paper_2511_21862_amd import workloads as W

from gpu_util import assert_parity, device_meta, run_gpu, say

pytestmark = pytest.mark.gpu


def batch(Hq, Hkv, hd, q_lens, ctx_lens, seed):
    seq = np.asarray(q_lens) + np.asarray(ctx_lens)
    return W.build_batch(Hq=Hq, Hkv=Hkv, hd=hd, q_lens=q_lens, ctx_lens=ctx_lens, num_blocks=int(((seq + 15) // 16).sum()) + 5,
                         seed=seed, poison=True)


def oracle(b):
    return ref_c.attn_mixed(b.q, b.k_cache, b.v_cache, b.block_tables, b.seq_lens, b.query_start_loc, b.ctx_lens)


def planned_kernels(b, options):
    with B.Context(b.Hq, b.Hkv, b.hd, b.BS, b.num_blocks, b.max_blocks_per_seq) as ctx:
        for k, v in options.items():
            ctx.set_option(k, v)
        ctx.plan(b.seq_lens, b.query_start_loc, b.ctx_lens)
        return ctx.plan_kernels()


CASES = {
    # one decode wave in all beside one query tile; the last decode workgroup partly filled (3 runs x 1 head, 5 x 3)
    "one-wave": ((4, 1, 64), [1, 2], [0, 0]),
    "odd-items": ((12, 3, 64), [1, 33, 1, 1, 1, 1], [16, 5, 700, 513, 1, 2000]),
    "g16": ((16, 1, 128), [9, 1, 1, 17], [40, 3000, 15, 260]),
    # more than one decode wave per workgroup, cut sequences, a split chunk
    "waves": ((32, 8, 128), [1] * 20 + [150], [1400 + 97 * i for i in range(20)] + [3000]),
    # a sequence in so many parts that the lean pair's decode waves are spread too
    "one-long": ((64, 8, 128), [40, 1, 1], [100, 30000, 500]),
    "qwen": ((28, 4, 128), [105, 1, 1, 132, 1, 1], [858, 4095, 130, 268, 17, 2222]),
}


@pytest.mark.parametrize("opts", [{}, {"mixed_lean": 2}, {"decode_nbi": 1}, {"trace": 1}, {"prefill_sorted": 0, "prefill_split": 2}],
                         ids=["default", "lean", "nbi1", "trace", "unsorted-split2"])
@pytest.mark.parametrize("name", list(CASES))
def test_one_launch_gives_the_bits_of_two(name, opts):
    heads, q_lens, ctx_lens = CASES[name]
    b = batch(*heads, q_lens, ctx_lens, seed=41)
    opts = {k: v for k, v in opts.items() if heads[2] == 128 or k != "mixed_lean"}
    say(f"case: {name} {opts}")
    one = planned_kernels(b, opts)
    # (head_dim 64 has the step kernel with two blocks per softmax step only)
    assert len(one) == (2 if opts.get("decode_nbi") == 1 and heads[2] == 64 else 1), one
    assert len(planned_kernels(b, dict(opts, mixed_step=0))) == 2 and len(planned_kernels(b, dict(opts, overlap=2))) == 2
    got = run_gpu(b, options=opts)
    two = run_gpu(b, options=dict({k: v for k, v in opts.items() if k != "trace"}, overlap=0))
    assert np.array_equal(got, two)
    assert_parity(got, oracle(b), name)


@pytest.mark.parametrize("n_dec,one", [(955, True), (956, False), (958, False)])
def test_arrays_that_do_not_fit_the_arguments_together_run_as_two_kernels(n_dec, one):
    # 961 entries: n + 2 of the decode array, 3 of the prefill array of one chunk, one (tile, part) entry
    q_lens, ctx_lens = [1] * n_dec + [8], [i % 40 for i in range(n_dec)] + [50]
    b = batch(4, 1, 64, q_lens, ctx_lens, seed=42)
    say(f"case: {n_dec} decodes and a chunk")
    assert len(planned_kernels(b, {})) == (1 if one else 2)
    assert_parity(run_gpu(b), oracle(b), f"{n_dec} decodes")


def test_weights_and_tails_run_as_two_kernels():
    b = batch(32, 8, 128, [1] * 12 + [64], [3000 + 31 * i for i in range(12)] + [10], seed=43)
    say("case: XCD weights, dynamic tail")
    want = oracle(b)
    for opts in ({"decode_tail_pct": 30, "decode_tail_blocks": 2}, {"xcd_weights": 0x0807060505060708, "decode_segments": 32}):
        assert len(planned_kernels(b, opts)) == 2, opts
        assert_parity(run_gpu(b, options=opts), want, str(opts))


@pytest.mark.parametrize("name", ["one-wave", "odd-items", "waves"])
def test_static_entry_runs_both_kinds_in_one_launch(name):
    heads, q_lens, ctx_lens = CASES[name]
    b = batch(*heads, q_lens, ctx_lens, seed=44)
    say(f"case: static {name}")
    d = W.to_device(b)
    bt, sl, qsl, cl = device_meta(b)
    want = oracle(b)
    for _ in range(2):      # (the arrival counters of the first call are clean for the second)
        out = torch.full((b.total_q, b.Hq, b.hd), float("nan"), dtype=torch.bfloat16, device="cuda")
        B.ooco_attn_mixed_static(b.Hq, b.Hkv, b.hd, b.BS, b.max_blocks_per_seq, 0.0, b.seq_lens, b.query_start_loc, b.ctx_lens, d.q,
                                 d.k_cache, d.v_cache, bt, sl, qsl, cl, out, len(b.seq_lens), b.total_q)
        torch.cuda.synchronize()
        assert_parity(out.view(torch.int16).cpu().numpy().view(np.uint16), want, name)


def test_long_decode_parts_run_on_two_streams_with_the_same_bits():
    # more than 180 us of decode K/V beside more than half a prefill workgroup per unit: two kernels, as "mixed_step" 2 is not
    seqs = 96
    q_lens, ctx_lens = [1] * seqs + [300, 300], [3600 + 7 * i for i in range(seqs)] + [40, 0]
    b = W.build_batch(Hq=32, Hkv=8, hd=128, q_lens=q_lens, ctx_lens=ctx_lens,
                      num_blocks=int(sum((q + c + 15) // 16 for q, c in zip(q_lens, ctx_lens))) + 5, seed=45, device="cuda")
    say("case: long decode part")
    assert len(planned_kernels(b, {})) == 2 and len(planned_kernels(b, {"mixed_step": 2})) == 1
    short = W.build_batch(Hq=32, Hkv=8, hd=128, q_lens=q_lens[60:], ctx_lens=ctx_lens[60:],
                          num_blocks=b.num_blocks, seed=45, device="cuda")
    assert len(planned_kernels(short, {})) == 1
    bt, sl, qsl, cl = device_meta(b)
    outs = []
    for opts in ({}, {"mixed_step": 2}):
        out = torch.zeros((b.total_q, 32, 128), dtype=torch.bfloat16, device="cuda")
        with B.Context(32, 8, 128, 16, b.num_blocks, b.max_blocks_per_seq) as ctx:
            for k, v in opts.items():
                ctx.set_option(k, v)
            ctx.plan(b.seq_lens, b.query_start_loc, b.ctx_lens)
            ctx.attn_mixed(b.q, b.k_cache, b.v_cache, bt, sl, qsl, cl, out)
            torch.cuda.synchronize()
        outs.append(out.view(torch.int16))
    assert torch.equal(outs[0], outs[1]) and bool((outs[0] != 0).any())
