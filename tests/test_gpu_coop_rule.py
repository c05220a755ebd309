"""Which decode batches take cooperative workgroups: on both sides of each line of the rule the kernels that a default context
launches, and the outputs against the float64 oracle and single waves."""
import numpy as np
import pytest

from oracle import ref_c
from paper_2511_21862_amd import binding as B
from paper_2511_21862_amd import workloads as W

pytestmark = pytest.mark.gpu


def spread(n, lo, hi):                      # lengths of lo .. hi, unequal
    return [int(x) for x in np.linspace(lo, hi, n).round()]


# heads, decode lengths, chunk (rows, cached tokens) or none, whether cooperative
CASES = [
    # up to two beginnings per run of unequal lengths (512/Hkv sequences), half a one of lengths that differ by an eighth or less
    ((64, 8, 128), spread(64, 400, 1000), None, True), ((64, 8, 128), spread(65, 400, 1000), None, False),
    ((28, 4, 128), spread(128, 300, 900), None, True), ((28, 4, 128), spread(129, 300, 900), None, False),
    ((32, 8, 128), [900] * 16, None, True), ((32, 8, 128), [900] * 17, None, False),
    ((32, 8, 128), [900] * 17 + [1300] * 8, None, True),
    ((8, 2, 64), spread(256, 800, 1700), None, True), ((8, 2, 64), spread(257, 800, 1700), None, False),
    # beside a prefill part one per run
    ((32, 8, 128), spread(32, 500, 1500), (900, 40), True), ((32, 8, 128), spread(33, 500, 1500), (900, 40), False),
    # larger batches, up to 70,000 tiles, however many sequences; of head_dim 64 unequal ones
    ((64, 16, 128), spread(40, 1000, 2450), None, True), ((64, 16, 128), [1730] * 40, None, True),
    ((64, 16, 128), spread(40, 1000, 2580), None, False),
    ((32, 16, 64), spread(90, 900, 2100), None, True), ((32, 16, 64), [1500] * 90, None, False),
]


@pytest.mark.parametrize("heads,lens,chunk,coop", CASES, ids=lambda x: "-".join(map(str, x)) if isinstance(x, tuple) else None)
def test_rule_and_outputs(heads, lens, chunk, coop):
    from gpu_util import assert_parity, run_gpu, say
    q, c = [1] * len(lens), [n - 1 for n in lens]
    if chunk:
        q.append(chunk[0])
        c.append(chunk[1])
    blocks = sum((a + b + 15) // 16 for a, b in zip(q, c))
    b = W.build_batch(Hq=heads[0], Hkv=heads[1], hd=heads[2], q_lens=q, ctx_lens=c, num_blocks=blocks + 5, seed=33)
    with B.Context(*heads, 16, b.num_blocks, b.max_blocks_per_seq) as ctx:
        ctx.plan(b.seq_lens, b.query_start_loc, b.ctx_lens)
        kernel = ctx.plan_kernels()[0]
    say(f"case: {heads} {len(lens)} decodes {chunk} {kernel}")
    assert ("coop" in kernel or "true" in kernel) == coop, kernel
    want = ref_c.attn_mixed(b.q, b.k_cache, b.v_cache, b.block_tables, b.seq_lens, b.query_start_loc, b.ctx_lens)
    for opts in ({}, {"decode_coop": 0 if coop else 2}):
        assert_parity(run_gpu(b, options=opts), want, str(opts))
