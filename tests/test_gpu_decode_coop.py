"""Decode runs shared by workgroups of four waves (small batches): against the oracle at the edges of their rule, and against
single waves on the same batch."""
import numpy as np
import pytest
import torch

from oracle import ref_c
from paper_2511_21862_amd import binding as B
from paper_2511_21862_amd import workloads as W

from gpu_util import assert_parity, device_meta, run_gpu, say

pytestmark = pytest.mark.gpu

HEADS = [(32, 8, 128), (28, 4, 128), (16, 1, 128), (4, 1, 64), (32, 4, 64), (3, 3, 64)]


def decode_batch(heads, lens, seed, chunk=None):
    lens = np.asarray(lens, np.int32)
    q, cx = [1] * len(lens), list(lens - 1)
    if chunk:
        q.insert(len(q) // 2, chunk[0])
        cx.insert(len(cx) // 2, chunk[1])
    nb = int(((np.asarray(q) + np.asarray(cx) + 15) // 16).sum())
    return W.build_batch(Hq=heads[0], Hkv=heads[1], hd=heads[2], q_lens=q, ctx_lens=cx, num_blocks=nb + 3, seed=seed, poison=True)


def oracle(b):
    return ref_c.attn_mixed(b.q, b.k_cache, b.v_cache, b.block_tables, b.seq_lens, b.query_start_loc, b.ctx_lens)


def kernels(b, options):
    with B.Context(b.Hq, b.Hkv, b.hd, b.BS, b.num_blocks, b.max_blocks_per_seq) as ctx:
        for k, v in options.items():
            ctx.set_option(k, v)
        ctx.plan(b.seq_lens, b.query_start_loc, b.ctx_lens)
        return ctx.plan_kernels(), ctx.plan_info()["decode_waves"]


# lengths: one token, a block and its neighbours, less and more than a step of the four waves, and past the limit up to
# which a sequence is taken whole (768 tokens, with head_dim 64 1536)
LENS = {"one": [1], "edges": [1, 15, 16, 17, 127, 128, 129, 255, 257], "whole-limit": [768, 3, 700], "cut": [769, 40, 1537, 200],
        "long": [9000, 33], "many-parts": [20011]}


@pytest.mark.parametrize("lens", list(LENS))
@pytest.mark.parametrize("heads", HEADS, ids=lambda h: "-".join(map(str, h)))
def test_small_batches(heads, lens):
    b = decode_batch(heads, LENS[lens], seed=51)
    names, runs = kernels(b, {})
    say(f"case: {heads} {lens}: {names}, {runs} runs")
    assert names[0].startswith("decode_coop_kernel")
    whole = max(LENS[lens]) <= 768 * 128 // heads[2]
    assert (runs == len(LENS[lens])) == (whole or (lens == "one"))
    got = run_gpu(b)
    assert_parity(got, oracle(b), "four waves")
    assert_parity(run_gpu(b, options={"decode_coop": 0}), oracle(b), "single waves")
    assert np.array_equal(got, run_gpu(b))


@pytest.mark.parametrize("heads", [(32, 8, 128), (32, 4, 64)], ids=lambda h: "-".join(map(str, h)))
@pytest.mark.parametrize("lens", ["equal", "unequal"])
def test_two_workgroups_per_unit(heads, lens):
    # equal lengths: single waves, one run per sequence (head_dim 128), unequal ones: whole sequences in four waves
    n = 2 * 256 // heads[1]
    b = decode_batch(heads, [100] * n if lens == "equal" else [40 + 16 * (i % 5) for i in range(n)], seed=55)
    names, runs = kernels(b, {})
    say(f"case: {n} {lens} sequences, {heads}: {names}, {runs} runs")
    assert names[0].startswith("decode_kernel" if lens == "equal" and heads[2] == 128 else "decode_coop_kernel") and runs == n
    assert_parity(run_gpu(b), oracle(b), lens)


@pytest.mark.parametrize("opts", [{"decode_coop": 2, "decode_segments": 1}, {"decode_coop": 2, "decode_segments": 7},
                                  {"decode_coop": 2, "decode_segments": 10 ** 6}, {"decode_coop": 2, "rotate_heads": 0}, {"decode_nbi": 1}],
                         ids=["1run", "7runs", "block-runs", "no-rotate", "nbi1"])
@pytest.mark.parametrize("chunk", [None, (37, 500)], ids=["decode", "mixed"])
def test_forced_layouts(chunk, opts):
    for heads in ((32, 8, 128), (32, 4, 64)):
        b = decode_batch(heads, [5, 300, 17, 1200, 16, 33, 2000], seed=52, chunk=chunk)
        say(f"case: {heads} {opts} chunk {chunk}")
        assert_parity(run_gpu(b, options=opts), oracle(b), str(opts))


@pytest.mark.parametrize("chunk", [None, (20, 100)], ids=["decode", "mixed"])
@pytest.mark.parametrize("opts", [{}, {"decode_coop": 2, "decode_segments": 300}, {"decode_coop": 2}], ids=["whole", "300runs", "runs"])
def test_batches_whose_plan_is_read_from_device_memory(opts, chunk):
    # more than 960 sequences: the plan's arrays do not fit the kernel arguments.  "runs" has lengths past the limit up to
    # which sequences are taken whole
    top = 1600 if opts == {"decode_coop": 2} else 90
    b = decode_batch((4, 1, 64), [1 + (37 * i) % 90 for i in range(979)] + [top], seed=56, chunk=chunk)
    names, runs = kernels(b, opts)
    say(f"case: {len(b.seq_lens)} sequences, {opts}: {names}, {runs} runs")
    if opts or not chunk:
        assert names[0].startswith("decode_coop_kernel") and len(names) == (2 if chunk else 1)
    assert_parity(run_gpu(b, options=opts), oracle(b), str(opts))
    assert_parity(run_gpu(b, plan=False, options=opts), oracle(b), f"{opts}, planned in the call")


@pytest.mark.parametrize("chunk", [None, (20, 100)], ids=["decode", "mixed"])
def test_replays_and_later_calls_find_clean_counters(chunk):
    # sequences cut into parts: the arrival counters are zero again after every launch, also inside a captured graph
    b = decode_batch((32, 8, 128), [5000, 1500, 64], seed=53, chunk=chunk)
    say(f"case: replayed, chunk {chunk}")
    d = W.to_device(b)
    bt, sl, qsl, cl = device_meta(b)
    out = torch.zeros((b.total_q, b.Hq, b.hd), dtype=torch.bfloat16, device="cuda")
    with B.Context(b.Hq, b.Hkv, b.hd, b.BS, b.num_blocks, b.max_blocks_per_seq) as ctx:
        ctx.set_option("plan_persistent", 1)
        ctx.plan(b.seq_lens, b.query_start_loc, b.ctx_lens)
        side = torch.cuda.Stream()
        with torch.cuda.stream(side):
            ctx.attn_mixed(d.q, d.k_cache, d.v_cache, bt, sl, qsl, cl, out)
            side.synchronize()
            want = out.clone()
            g = torch.cuda.CUDAGraph()
            with torch.cuda.graph(g, stream=side):
                ctx.attn_mixed(d.q, d.k_cache, d.v_cache, bt, sl, qsl, cl, out)
        for _ in range(3):
            out.zero_()
            g.replay()
            torch.cuda.synchronize()
            assert torch.equal(out.view(torch.int16), want.view(torch.int16))
            ctx.attn_mixed(d.q, d.k_cache, d.v_cache, bt, sl, qsl, cl, out)
            torch.cuda.synchronize()
            assert torch.equal(out.view(torch.int16), want.view(torch.int16))
    assert_parity(want.view(torch.int16).cpu().numpy().view(np.uint16), oracle(b), "replayed")


# K blocks whose scores overflow to -inf in fp32 (their weight is zero): the first steps of a piece, of one wave, of all but
# one wave of four, all of a piece but its last block
MASKED = {"start": [(0, 4)], "one-wave": [(2, 4), (10, 12)], "middle": [(8, 16)], "second-half": [(0.5, 1.0)], "all-but-last": [(0, -1)],
          "all-but-first": [(1, 1.0)]}


@pytest.mark.parametrize("opts", [{}, {"decode_coop": 0}, {"decode_coop": 2, "decode_segments": 9}, {"decode_nbi": 1}],
                         ids=["default", "single", "9runs", "nbi1"])
@pytest.mark.parametrize("masked", list(MASKED))
def test_keys_whose_scores_are_minus_infinity_weigh_nothing(masked, opts):
    for heads, chunk in (((32, 8, 128), None), ((4, 1, 64), None), ((28, 4, 128), (37, 100))):
        b = decode_batch(heads, [600, 40, 3000], seed=54, chunk=chunk)
        say(f"case: {heads} {masked} {opts} chunk {chunk}")
        b.q = np.where(b.q == b.q, np.uint16(0x3F80), np.uint16(0))                  # ones
        for i, (n, ql) in enumerate(zip(b.seq_lens, b.q_lens)):
            nb = (int(n) + 15) // 16
            if ql > 1 or nb < 16:
                continue
            for lo, hi in MASKED[masked]:
                lo = int(lo * nb) if isinstance(lo, float) else lo
                hi = int(hi * nb) if isinstance(hi, float) else hi % nb
                b.k_cache[b.block_tables[i, lo:hi]] = 0xFF61                        # -2.98e38: scores below -FLT_MAX
        assert_parity(run_gpu(b, options=opts), oracle(b), masked)
