"""Split prefill tiles whose parts share the merge: the float64 oracle at the fewest and the most parts, tiles with unused
columns and parts without visible keys, one bit pattern whoever merges -- also where early parts leave at once or after one
look --, counters ready for the next call and under replay, and a launch too large for it."""
import numpy as np
import pytest
import torch

from oracle import ref_c
from paper_2511_21862_amd import binding as B
from paper_2511_21862_amd import workloads as W

pytestmark = pytest.mark.gpu


def batch(heads, q_lens, ctx_lens, seed=83):
    seq = np.asarray(q_lens) + np.asarray(ctx_lens)
    return W.build_batch(Hq=heads[0], Hkv=heads[1], hd=heads[2], q_lens=q_lens, ctx_lens=ctx_lens,
                         num_blocks=int(((seq + 15) // 16).sum()) + 5, seed=seed, poison=True)


@pytest.mark.parametrize("heads", [(32, 8, 128), (28, 4, 128), (4, 1, 64), (32, 4, 64), (7, 7, 128)], ids=str)
@pytest.mark.parametrize("parts", [3, 4, 5, 16])
def test_parity_and_the_same_bits_every_time(heads, parts):
    from gpu_util import assert_parity, device_meta, say
    b = batch(heads, [2, 37, 3], [1100, 1021, 250])      # the last tile has fewer steps than parts
    want = ref_c.attn_mixed(b.q, b.k_cache, b.v_cache, b.block_tables, b.seq_lens, b.query_start_loc, b.ctx_lens)
    d, meta = W.to_device(b), device_meta(b)
    with B.Context(*heads, 16, b.num_blocks, b.max_blocks_per_seq) as ctx:
        ctx.set_option("prefill_groups", 1)
        ctx.set_option("prefill_split", parts)
        ctx.set_option("plan_persistent", 1)
        ctx.plan(b.seq_lens, b.query_start_loc, b.ctx_lens)
        say(f"case: {heads} {parts} parts {ctx.plan_kernels()}")
        outs = []
        for looks in (12, 0, 12, 1, 0, 1, 100, 0, 3, 12, 12, 12):
            ctx.set_option("prefill_merge_looks", looks)
            out = torch.full((b.total_q, b.Hq, b.hd), float("nan"), dtype=torch.bfloat16, device="cuda")
            ctx.attn_mixed(d.q, d.k_cache, d.v_cache, *meta, out)
            outs.append(out)
        torch.cuda.synchronize()
        outs = [o.view(torch.int16).cpu().numpy().view(np.uint16) for o in outs]
        assert_parity(outs[0], want, f"{parts} parts")
        assert all(np.array_equal(outs[0], o) for o in outs)


def test_replays_and_a_launch_that_is_too_large():
    from gpu_util import assert_parity, device_meta, say
    heads = (32, 8, 128)
    for n, parts, looks in ((2, 8, 12), (2, 8, 0), (2, 8, 1), (12, 6, 12)):      # 128 workgroups; 576, more than 256 units hold
        b = batch(heads, [20] * n, [1500 + 64 * i for i in range(n)], seed=84)
        want = ref_c.attn_mixed(b.q, b.k_cache, b.v_cache, b.block_tables, b.seq_lens, b.query_start_loc, b.ctx_lens)
        d, meta = W.to_device(b), device_meta(b)
        out = torch.empty((b.total_q, b.Hq, b.hd), dtype=torch.bfloat16, device="cuda")
        with B.Context(*heads, 16, b.num_blocks, b.max_blocks_per_seq) as ctx:
            for k, v in dict(prefill_groups=1, prefill_split=parts, plan_persistent=1).items():
                ctx.set_option(k, v)
            ctx.set_option("prefill_merge_looks", looks)
            ctx.plan(b.seq_lens, b.query_start_loc, b.ctx_lens)
            say(f"case: {n} chunks in {parts} parts, {looks} looks, {ctx.plan_info()}")
            side = torch.cuda.Stream()
            with torch.cuda.stream(side):
                ctx.attn_mixed(d.q, d.k_cache, d.v_cache, *meta, out)
                side.synchronize()
                graph = torch.cuda.CUDAGraph()
                with torch.cuda.graph(graph, stream=side):
                    ctx.attn_mixed(d.q, d.k_cache, d.v_cache, *meta, out)
            for _ in range(4):
                out.zero_()
                torch.cuda.synchronize()
                graph.replay()
                torch.cuda.synchronize()
                assert_parity(out.view(torch.int16).cpu().numpy().view(np.uint16), want, "replay")
