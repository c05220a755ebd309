"""Prefill output rows, which leave through LDS: every row of ragged tiles and nothing beside them, whole tiles and merged ones, and
an output that is not aligned to the width of the stores."""
import numpy as np
import pytest
import torch

from oracle import ref_c
from paper_2511_21862_amd import binding as B
from paper_2511_21862_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("opts", [{"prefill_groups": 1}, {"prefill_groups": 1, "prefill_split": 2}, {"prefill_groups": 1, "prefill_split": 5},
                                  {"prefill_groups": 4}, {"prefill_groups": 4, "prefill_split": 3}, {"prefill_waves": 8}, {"mixed_lean": 2}], ids=str)
@pytest.mark.parametrize("heads", [(32, 8, 128), (14, 2, 128), (3, 3, 128), (16, 1, 64), (6, 2, 64)], ids=str)
def test_rows_land_where_they_belong(heads, opts):
    from gpu_util import device_meta, errors, say, REL_L2
    Hq, Hkv, hd = heads
    q, c = [2, 131, 1, 19], [700, 40, 90, 333]
    b = W.build_batch(Hq=Hq, Hkv=Hkv, hd=hd, q_lens=q, ctx_lens=c, num_blocks=90, seed=17, poison=True)
    want = ref_c.attn_mixed(b.q, b.k_cache, b.v_cache, b.block_tables, b.seq_lens, b.query_start_loc, b.ctx_lens)
    d, meta = W.to_device(b), device_meta(b)
    n, guard = b.total_q * Hq * hd, 512
    got = []
    for shift in (0, 4, 1):             # elements: 0, 8 and 2 bytes past a 16-byte boundary
        buf = torch.full((n + 2 * guard,), 7.0, dtype=torch.bfloat16, device="cuda")
        out = buf[guard + shift: guard + shift + n].view(b.total_q, Hq, hd)
        with B.Context(Hq, Hkv, hd, 16, b.num_blocks, b.max_blocks_per_seq) as ctx:
            for k, v in opts.items():
                ctx.set_option(k, v)
            ctx.plan(b.seq_lens, b.query_start_loc, b.ctx_lens)
            ctx.attn_mixed(d.q, d.k_cache, d.v_cache, *meta, out)
            torch.cuda.synchronize()
        assert (buf[:guard + shift] == 7).all() and (buf[guard + shift + n:] == 7).all()
        got.append(out.cpu().view(torch.int16).numpy().view(np.uint16))
    e = errors(got[0], want)
    say(f"  {heads} {opts}: {e}")
    assert e["finite"] and e["rel_l2"] <= REL_L2
    assert np.array_equal(got[0], got[1]) and np.array_equal(got[0], got[2])
