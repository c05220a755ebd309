"""Block copies ordered by destination region: every pair arrives, at the sizes where the ordering kernel changes its passes
or gives way to the radix sort; captured copies are not ordered."""
import ctypes

import pytest
import torch

from paper_2511_21862_amd import binding as B

from gpu_util import say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("pool", [1 << 15, 40000, 16500])
@pytest.mark.parametrize("n", [1, 63, 1023, 1024, 1025, 16383, 16384, 16385])
def test_ordered_copies_move_every_block(n, pool):
    say(f"case: {n} pairs, pool of {pool} blocks")
    g = torch.Generator(device="cuda").manual_seed(n)
    elems = 2 * 64 * 16
    src = [torch.randint(-32768, 32767, (pool, elems), dtype=torch.int16, device="cuda", generator=g).view(torch.bfloat16) for _ in range(2)]
    # destinations all over the pool, in its upper end only (one bucket or few), and descending
    spread = torch.randperm(pool, generator=g, device="cuda")[:n]
    for dst_ids in (spread, torch.arange(pool - n, pool, device="cuda"), torch.arange(n - 1, -1, -1, device="cuda")):
        src_ids = torch.randperm(pool, generator=g, device="cuda")[:n].contiguous()
        dst_ids = dst_ids.contiguous()
        dst = [torch.zeros((pool, elems), dtype=torch.bfloat16, device="cuda") for _ in range(2)]
        want = [torch.zeros_like(d) for d in dst]
        for w, s in zip(want, src):
            w[dst_ids] = s[src_ids]
        with B.Context(8, 2, 64, 16, pool, 8) as ctx:
            ctx.set_option("copy_sort", 2)
            ids = src_ids.clone(), dst_ids.clone()
            ctx.kv_block_copy(src[0], src[1], dst[0], dst[1], src_ids, dst_ids)
            torch.cuda.synchronize()
            assert torch.equal(ids[0], src_ids) and torch.equal(ids[1], dst_ids)
        for w, d in zip(want, dst):
            assert torch.equal(w.view(torch.int16), d.view(torch.int16))


def test_a_captured_copy_does_not_use_the_buffer_of_ordered_copies():
    # a context whose earlier copies were ordered holds a buffer for the ordered lists, and a later, larger copy frees it:
    # a copy captured in between is one kernel on the caller's own lists, and its replays stay right
    pool, n, elems = 40000, 2000, 2 * 64 * 16
    say(f"case: captured copy of {n} pairs on a context with an ordering buffer")
    g = torch.Generator(device="cuda").manual_seed(5)
    src = [torch.randint(-32768, 32767, (pool, elems), dtype=torch.int16, device="cuda", generator=g).view(torch.bfloat16) for _ in range(2)]
    dst = [torch.zeros_like(s) for s in src]
    ids = lambda m: torch.randperm(pool, generator=g, device="cuda")[:m].contiguous()
    src_ids, dst_ids = ids(n), ids(n)
    want = [torch.zeros_like(s) for s in src]
    for w, s in zip(want, src):
        w[dst_ids] = s[src_ids]
    with B.Context(8, 2, 64, 16, pool, 8) as ctx:
        ctx.set_option("copy_sort", 2)
        side = torch.cuda.Stream()
        graph = torch.cuda.CUDAGraph(keep_graph=True)
        side.wait_stream(torch.cuda.current_stream())
        with torch.cuda.stream(side):
            ctx.kv_block_copy(src[0], src[1], dst[0], dst[1], src_ids, dst_ids)      # ordered: the buffer is there now
            side.synchronize()
            with torch.cuda.graph(graph, stream=side):
                ctx.kv_block_copy(src[0], src[1], dst[0], dst[1], src_ids, dst_ids)
        nodes = ctypes.c_size_t()
        assert B._lib.hipGraphGetNodes(ctypes.c_void_p(graph.raw_cuda_graph()), None, ctypes.byref(nodes)) == 0
        assert nodes.value == 1, "the captured copy is one kernel: no ordering, whose buffer the graph would keep"
        graph.instantiate()
        more_src, more_dst = ids(20000), ids(20000)
        other = [torch.zeros_like(s) for s in src]
        for rep in range(3):
            # larger copies through the same context, each with another buffer size, and their allocations
            m = 17000 + 1500 * rep
            ctx.kv_block_copy(src[0], src[1], other[0], other[1], more_src[:m].contiguous(), more_dst[:m].contiguous())
            for d in dst:
                d.zero_()
            torch.cuda.synchronize()
            graph.replay()
            torch.cuda.synchronize()
            for w, d in zip(want, dst):
                assert torch.equal(w.view(torch.int16), d.view(torch.int16)), f"replay {rep}"


@pytest.mark.parametrize("n,ordered", [(2047, False), (2048, True)])
def test_copies_of_few_large_blocks_keep_the_callers_order(n, ordered):
    # (an ordered copy allocates the context's buffer: seen here over many contexts)
    say(f"case: {n} pairs of 128 KiB")
    pool = 2048
    src = [torch.zeros((pool, 32 * 128 * 16), dtype=torch.bfloat16, device="cuda") for _ in range(2)]
    dst = [torch.empty_like(s) for s in src]
    ids = torch.arange(n, dtype=torch.int64, device="cuda")
    ctxs = [B.Context(32, 32, 128, 16, pool, 8, workspace_bytes=1 << 20) for _ in range(40)]
    torch.cuda.synchronize()
    before = torch.cuda.mem_get_info()[0]
    for c in ctxs:
        c.kv_block_copy(src[0], src[1], dst[0], dst[1], ids, ids)
    torch.cuda.synchronize()
    used = before - torch.cuda.mem_get_info()[0]
    for c in ctxs:
        c.close()
    assert (used >= 40 * 16384 * 16) == ordered, used
