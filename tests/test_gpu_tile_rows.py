"""The tile list by rows of the grid: where it just fits beside the decode runs and where it does not, a plan too long for the
kernel arguments, tiles of fewer key blocks than a workgroup asks for before it knows their number, every group size."""
import numpy as np
import pytest

from oracle import ref_c
from paper_2511_21862_amd import binding as B
from paper_2511_21862_amd import workloads as W

pytestmark = pytest.mark.gpu


def batch(heads, q_lens, ctx_lens, seed=71):
    seq = np.asarray(q_lens) + np.asarray(ctx_lens)
    return W.build_batch(Hq=heads[0], Hkv=heads[1], hd=heads[2], q_lens=q_lens, ctx_lens=ctx_lens,
                         num_blocks=int(((seq + 15) // 16).sum()) + 5, seed=seed, poison=True)


def agree(heads, b, variants):
    from gpu_util import assert_parity, run_gpu, say
    want = ref_c.attn_mixed(b.q, b.k_cache, b.v_cache, b.block_tables, b.seq_lens, b.query_start_loc, b.ctx_lens)
    for opts in variants:
        say(f"case: {heads} {b.num_seqs} sequences {opts}")
        assert_parity(run_gpu(b, options=opts), want, str(opts))


# a decode workgroup for each of the 256 sequences, a word for each and one more, and 448 or 449 tiles of 8 rows: 961 words
# of the argument block's 961, and 962
@pytest.mark.parametrize("tiles", [448, 449])
def test_step_at_the_edge_of_the_argument_block(tiles):
    heads = (16, 1, 128)
    b = batch(heads, [1] * 255 + [8 * tiles - 3], [59] * 255 + [1])
    with B.Context(*heads, 16, b.num_blocks, b.max_blocks_per_seq) as ctx:
        ctx.plan(b.seq_lens, b.query_start_loc, b.ctx_lens)
        kernels = ctx.plan_kernels()
    assert kernels == ["step_kernel<128, 2, true>"], kernels
    agree(heads, b, [{}, {"mixed_step": 0}])


@pytest.mark.parametrize("n", [958, 959, 960, 970])       # the last whose plan travels with the call, and beyond
def test_plans_on_both_sides_of_the_argument_block(n):
    rng = np.random.default_rng(n)
    q = [1] * n
    q[0], q[n // 2], q[-1] = 5, 70, 2                     # the first and the last sequence among the chunks
    b = batch((4, 1, 64), q, rng.integers(0, 90, size=n).tolist())
    agree((4, 1, 64), b, [{}, {"overlap": 0}, {"overlap": 2}, {"prefill_sorted": 0}])


@pytest.mark.parametrize("hd", [64, 128])
@pytest.mark.parametrize("g", range(1, 17))
def test_every_group_size(g, hd):
    # tiles of one block, of 4 and of 12 and one more (what is asked for ahead), table rows no longer than that
    for q, c in (([2, 16 // g + 2], [0, 3]), ([64 // g + 1, 3, 128 // g + 2], [60, 64, 190]), ([7], [240]), ([2, 130 // g + 2], [1, 700])):
        b = batch((2 * g, 2, hd), q, c, seed=72 + g)
        agree((2 * g, 2, hd), b, [{"prefill_groups": 1}, {"prefill_groups": 4}, {"prefill_sorted": 0}])
