"""ooco_plan_kernels names the kernels as a profiler shows them: every name is a kernel of the library, and it follows the
conditions by which the launches choose (dynamic tail, XCD weights, plans in device memory, key groups, forced steps)."""
import re
import subprocess

import numpy as np
import pytest

from paper_2511_21862_amd import binding as B

pytestmark = pytest.mark.gpu


def kernels_of_the_library():
    out = subprocess.run(["nm", "-C", "--defined-only", B.LIB_PATH], capture_output=True, text=True, check=True).stdout
    return {m.group(1) for m in re.finditer(r"ooco::(\w+<[^>]*>)\(ooco::KernArgs\)", out) if not m.group(1).startswith("__device_stub__")}


WEIGHTS = 0x0807060505060708
MIXED = [1] * 12 + [64], [3000 + 31 * i for i in range(12)] + [10]
LONG = [1] * 64, [3000] * 64
SMALL = [1, 1, 40], [500, 70, 1000]
MANY = [1] * 1000, [40] * 1000            # (a plan that does not fit the kernel arguments)
LEAN = [1] * 128 + [512] * 8, [2100] * 128 + [1000] * 8
CASES = [
    ((32, 8, 128), [64], [10], {}, "prefill_kernel<128, 4>"),
    ((32, 4, 64), [64], [10], {}, "prefill_kernel<64, 4>"),
    ((32, 8, 128), [64], [10], {"prefill_waves": 8}, "prefill_kernel<128, 8>"),
    ((32, 8, 128), [40], [1000], {}, "prefill_kernel_groups<128>"),
    ((32, 8, 128), [40], [1000], {"prefill_sorted": 0}, "prefill_kernel<128, 4>"),
    ((32, 8, 128), [40], [1000], {"prefill_sorted": 0, "prefill_groups": 4}, "prefill_kernel_groups<128>"),
    ((32, 8, 128), *SMALL, {}, "step_kernel_groups<128, 2>"),
    ((32, 8, 128), *SMALL, {"overlap": 0}, "decode_coop_kernel_groups<128, 2>;prefill_kernel_groups<128>"),
    ((32, 4, 64), *SMALL, {"overlap": 0, "prefill_groups": 4}, "decode_coop_kernel_groups<64, 4>;prefill_kernel_groups<64>"),
    ((32, 8, 128), *SMALL, {"prefill_groups": 1}, "step_kernel<128, 2, true>"),
    ((32, 8, 128), [1] * 3, [500] * 3, {}, "decode_coop_kernel<128, 2>"),
    ((32, 8, 128), *MANY, {"decode_coop": 2}, "decode_coop_kernel_general<128, 2>"),
    ((32, 4, 64), *MANY, {"decode_coop": 2}, "decode_coop_kernel_general<64, 4>"),
    ((32, 8, 128), *LONG, {}, "decode_kernel<128, 1>"),
    ((32, 8, 128), *LONG, {"decode_nbi": 4}, "decode_kernel<128, 4>"),
    ((32, 8, 128), *LONG, {"decode_nbi": 3}, "decode_kernel<128, 1>"),
    ((32, 8, 128), *LONG, {"decode_tail_pct": 20}, "decode_kernel_general<128, 1>"),
    ((32, 8, 128), *LONG, {"xcd_weights": WEIGHTS}, "decode_kernel_general<128, 1>"),
    ((32, 8, 128), *MANY, {"decode_coop": 0}, "decode_kernel_general<128, 1>"),
    ((32, 8, 128), *MIXED, {"decode_tail_pct": 30, "decode_tail_blocks": 2}, "decode_kernel_general<128, 2>;prefill_kernel<128, 4>"),
    ((32, 8, 128), *LEAN, {}, "step_kernel_lean<128>"),
    ((32, 8, 128), *LEAN, {"overlap": 2}, "decode_kernel_lean<128>;prefill_kernel_lean<128>"),
    ((32, 8, 128), *LEAN, {"xcd_weights": WEIGHTS}, "decode_kernel_lean_general<128>;prefill_kernel_lean<128>"),
    ((32, 8, 128), *MIXED, {"mixed_fused": 1}, "mixed_kernel<128>"),
]


def test_names_follow_the_launches():
    known = kernels_of_the_library()
    wrong = []
    for heads, q, c, opts, want in CASES:
        q, c = np.asarray(q, np.int32), np.asarray(c, np.int32)
        with B.Context(*heads, 16, 64, 512) as ctx:
            for k, v in opts.items():
                ctx.set_option(k, v)
            ctx.plan(q + c, np.r_[0, np.cumsum(q)].astype(np.int32), c)
            names = ctx.plan_kernels()
        if ";".join(names) != want or not set(names) <= known:
            wrong.append((heads, opts, names, want))
    assert not wrong, wrong
