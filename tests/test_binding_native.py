"""The native argument marshalling takes the plain form of the per-step calls and leaves everything else to the general
way; both ways give the same results, statuses and messages."""
import ctypes

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2511_21862_amd import binding as B
from paper_2511_21862_amd import workloads as W

N = B._native


def test_the_native_module_is_there():
    assert N is not None


def test_a_module_for_another_torch_is_not_used(tmp_path):
    """... and is built again: it reads torch's objects directly."""
    import os
    import shutil
    import subprocess
    import sys

    from paper_2511_21862_amd import build
    stamp = build.built_for(torch)
    assert N.BUILT_FOR == stamp and torch.__version__ in stamp and build.has_stamp(build.MARSHAL, stamp)
    other = tmp_path / "_binding.so"
    code = open(build.MARSHAL, "rb").read()
    other.write_bytes(code.replace(stamp.encode(), stamp.replace("torch " + torch.__version__[0], "torch 9").encode()))
    assert not build.has_stamp(str(other), stamp)
    # a copy of the package with that module: the general way, and a warning that says why
    pkg = tmp_path / "paper_2511_21862_amd"
    pkg.mkdir()
    for f in os.listdir(build.HERE):
        if f.endswith((".py", ".so")):
            shutil.copy(os.path.join(build.HERE, f), pkg / f)
    shutil.copy(other, pkg / "_binding.so")
    res = subprocess.run([sys.executable, "-c", "from paper_2511_21862_amd import binding as B; assert B._native is None; "
                          "assert B._plan_fast is B._not_native"], cwd=tmp_path, capture_output=True, text=True)
    assert res.returncode == 0 and "torch 9" in res.stderr, res.stderr


@pytest.mark.parametrize("seq", [[3, 5], np.array([3, 5], np.int64), np.array([3, 5, 7, 9], np.int32)[::2], np.array([3, 5], ">i4"),
                                 None, np.array([3, 5], np.uint32), torch.tensor([3, 5], dtype=torch.int32)])
def test_other_length_arrays_are_left_to_the_general_way(seq):
    plain = np.array([1, 2], np.int32)
    assert N.plan(ctypes.c_void_p(0), 2, seq, plain, plain) is NotImplemented
    assert N.plan(ctypes.c_void_p(0), 2, plain, plain, seq) is NotImplemented


@pytest.mark.parametrize("ctx,n", [(0, 2), (None, 2), (b"12345678", 2), (ctypes.c_uint64(0), 2), (ctypes.c_void_p(0), None),
                                   (ctypes.c_void_p(0), True), (ctypes.c_void_p(0), 1 << 31), (ctypes.c_void_p(0), 2.0)])
def test_other_handles_and_sizes_are_left_to_the_general_way(ctx, n):
    plain = np.array([1, 2], np.int32)
    assert N.plan(ctx, n, plain, plain, plain) is NotImplemented


def test_a_plain_call_reaches_the_library():
    plain = np.array([1, 2], np.int32)
    plain.flags.writeable = False
    assert N.plan(ctypes.c_void_p(0), 2, plain, plain, plain) == B.OOCO_EINVAL     # (no context)
    with pytest.raises(B.OocoError) as e:
        B.ooco_plan(ctypes.c_void_p(0), 2, plain, plain, plain)
    assert e.value.status == B.OOCO_EINVAL


def test_tensors_on_the_host_and_wrong_counts_are_left_to_the_general_way():
    h, t = ctypes.c_void_p(0), torch.zeros(4, dtype=torch.int32)
    assert N.attn_mixed(h, *[t] * 8, 1, 1, 0) is NotImplemented
    assert N.kv_append(h, *[t] * 7, 1, 1, 0) is NotImplemented
    assert N.kv_block_copy(h, *[t] * 6, 1, 0) is NotImplemented
    assert N.attn_mixed(h) is NotImplemented and N.plan() is NotImplemented


@pytest.fixture
def general(monkeypatch):
    """Switches the binding to its general way."""
    def switch():
        for name in ("_plan_fast", "_attn_fast", "_static_fast", "_append_fast", "_copy_fast"):
            monkeypatch.setattr(B, name, B._not_native)
    return switch


@pytest.mark.gpu
def test_plain_calls_are_taken():
    """Every native function accepts its plain form (else both ways below would be the general one), with sizes given and read
    off the tensors, on the current stream and on one given by its handle."""
    b = W.config1(poison=True)
    d = W.to_device(b, "cuda:0")
    t = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    tabs = [t(x) for x in (b.block_tables, b.seq_lens, b.query_start_loc, b.ctx_lens)]
    n, host = len(b.seq_lens), (b.seq_lens, b.query_start_loc, b.ctx_lens)
    kn = torch.randn(b.total_q, b.Hkv, b.hd, device="cuda").bfloat16()
    ids, dst = torch.tensor([1, 2, 3], device="cuda"), torch.tensor([2, 0, 1], device="cuda")
    kd, vd = torch.zeros_like(d.k_cache[:4]), torch.zeros_like(d.v_cache[:4])
    out = torch.zeros((b.total_q, b.Hq, b.hd), dtype=torch.bfloat16, device="cuda")
    with B.Context(b.Hq, b.Hkv, b.hd, b.BS, b.num_blocks, b.max_blocks_per_seq) as ctx:
        for stream in (None, torch.cuda.current_stream().cuda_stream):
            for sizes in ((n, b.total_q), (N.OF_TENSOR, N.OF_TENSOR)):
                assert N.kv_append(ctx.h, kn, kn, d.k_cache, d.v_cache, tabs[0], tabs[2], tabs[3], *sizes, stream) == B.OOCO_OK
                assert N.plan(ctx.h, n, *host) == B.OOCO_OK
                assert N.attn_mixed(ctx.h, d.q, d.k_cache, d.v_cache, *tabs, out, *sizes, stream) == B.OOCO_OK
            for pairs in (3, N.OF_TENSOR):
                assert N.kv_block_copy(ctx.h, d.k_cache, d.v_cache, kd, vd, ids, dst, pairs, stream) == B.OOCO_OK
            assert N.attn_mixed_static(b.Hq, b.Hkv, b.hd, b.BS, b.max_blocks_per_seq, 0.0, *host, d.q, d.k_cache, d.v_cache, *tabs,
                                       torch.zeros_like(out), n, b.total_q, stream) == B.OOCO_OK
        torch.cuda.synchronize()


@pytest.mark.gpu
def test_both_ways_agree(general):
    b = W.config1(poison=True)
    d = W.to_device(b, "cuda:0")
    t = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    tabs = [t(x) for x in (b.block_tables, b.seq_lens, b.query_start_loc, b.ctx_lens)]
    kn = torch.randn(b.total_q, b.Hkv, b.hd, device="cuda").bfloat16()
    ids, dst = torch.tensor([1, 2, 3], device="cuda"), torch.tensor([2, 0, 1], device="cuda")

    def everything():
        k, v = d.k_cache.clone(), d.v_cache.clone()
        kd, vd = torch.zeros_like(k[:4]), torch.zeros_like(v[:4])
        out = torch.zeros((3, b.total_q, b.Hq, b.hd), dtype=torch.bfloat16, device="cuda")
        side = torch.cuda.Stream()
        with B.Context(b.Hq, b.Hkv, b.hd, b.BS, b.num_blocks, b.max_blocks_per_seq) as ctx:
            ctx.kv_append(kn, kn, k, v, tabs[0], tabs[2], tabs[3])
            ctx.plan(b.seq_lens, b.query_start_loc, b.ctx_lens)
            ctx.attn_mixed(d.q, k, v, *tabs, out[0])
            torch.cuda.synchronize()
            for s, o in ((side, out[1]), (side.cuda_stream, out[2])):    # a stream, its handle; lengths as lists
                ctx.plan(list(b.seq_lens), list(b.query_start_loc), list(b.ctx_lens))
                ctx.attn_mixed(d.q, k, v, *tabs, o, stream=s)
            ctx.kv_block_copy(k, v, kd, vd, ids, dst)
            torch.cuda.synchronize()
            errors = []
            for f in (lambda: ctx.plan(b.seq_lens, b.query_start_loc[::-1].copy(), b.ctx_lens),
                      lambda: B.ooco_attn_mixed(ctx.h, d.q, k, v, *tabs, out[0], -1, b.total_q),
                      lambda: ctx.attn_mixed(d.q.transpose(0, 1), k, v, *tabs, out[0]),
                      lambda: B.ooco_attn_mixed(ctx.h, d.q, k, v, *tabs, None, len(b.seq_lens), b.total_q),
                      lambda: B.ooco_attn_mixed(ctx.h, d.q, k, v, *tabs, out[0], None, b.total_q),
                      lambda: B.ooco_attn_mixed_static(b.Hq, b.Hkv, 96, b.BS, b.max_blocks_per_seq, 0.0, b.seq_lens, b.query_start_loc,
                                                       b.ctx_lens, d.q, k, v, *tabs, out[0], len(b.seq_lens), b.total_q)):
                with pytest.raises(Exception) as e:
                    f()
                errors.append((type(e.value), str(e.value)))
        B.ooco_attn_mixed_static(b.Hq, b.Hkv, b.hd, b.BS, b.max_blocks_per_seq, 0.0, b.seq_lens, b.query_start_loc, b.ctx_lens, d.q, k, v,
                                 *tabs, static := torch.zeros_like(out[0]), len(b.seq_lens), b.total_q)
        torch.cuda.synchronize()
        bits = lambda x: x.view(torch.int16).cpu()
        return [bits(x) for x in (out, static, k, v, kd, vd)], errors

    native, native_errors = everything()
    general()
    other, other_errors = everything()
    assert native_errors == other_errors
    for x, y in zip(native, other):
        assert torch.equal(x, y)
    assert torch.equal(native[0][0], native[0][1]) and torch.equal(native[0][0], native[0][2])
