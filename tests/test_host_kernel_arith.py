"""The kernels' arithmetic of csrc/ooco_arith.h, compiled for the CPU as it is: the run bounds' quotient against whole-number
division, and every order of events at the arrival counter of a shared merge."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2511_21862_amd", "csrc")
SHIM = r"""
#include "ooco_arith.h"
using ooco::MergeWord;
extern "C" {
int64_t wrong_quotients(const int *a, const int *b, const int *n, int c, int ulps, int64_t count)
{
    int64_t wrong = 0;
    for (int64_t i = 0; i < count; ++i) {
        union { double d; int64_t bits; } inv = {1.0 / n[i]};
        inv.bits += ulps;
        wrong += ooco::quotient_by_reciprocal(a[i], b[i], c, n[i], inv.d) != (int)(((int64_t)a[i] * b[i] - c) / n[i]);
    }
    return wrong;
}
int slices() { return MergeWord::kSlices; }
int arrive() { return MergeWord::kArrive; }
int draw() { return MergeWord::kDraw; }
int leave() { return MergeWord::kLeave; }
int arrivals(int w) { return MergeWord::arrivals(w); }
int arrived_last(int w, int nparts) { return MergeWord::arrived_last(w, nparts); }
int slice(int w) { return MergeWord::slice(w); }
int last_event(int w, int nparts) { return MergeWord::last_event(w, nparts); }
int past_caches(int total_q, int num_seqs, int64_t bytes) { return ooco::append_past_caches(total_q, num_seqs, bytes); }
int by_rows(int total_q, int num_seqs, int64_t workgroups, int num_cus) { return ooco::append_by_rows(total_q, num_seqs, workgroups, num_cus); }
}
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("arith")
    (d / "shim.cpp").write_text(SHIM)
    out = str(d / "shim.so")
    subprocess.run([os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-shared", "-fPIC", "-Wall", "-Werror", "-I", CSRC, "-o", out,
                    str(d / "shim.cpp")], check=True)
    r = ctypes.CDLL(out)
    r.wrong_quotients.restype = ctypes.c_int64
    r.wrong_quotients.argtypes = [ctypes.c_void_p] * 3 + [ctypes.c_int, ctypes.c_int, ctypes.c_int64]
    return r


def test_run_bounds_by_reciprocal_equal_the_divisions(lib):
    # the device's reciprocal is within two units in the last place; runs * blocks of up to 2^30 each, quotients below 2^30
    rng = np.random.default_rng(8)
    n = np.concatenate([np.arange(1, 400), np.exp(rng.uniform(0, np.log(2 ** 30), size=200000)).astype(np.int64)])
    a = np.minimum(np.exp(rng.uniform(0, np.log(2 ** 30), size=len(n))).astype(np.int64) + 1, 2 ** 30)
    for b in (np.minimum(n, a), n, np.maximum(1, (n * rng.random(len(n))).astype(np.int64)), np.ones_like(n)):
        x, y, z = (np.ascontiguousarray(v, np.int32) for v in (a, b, n))
        ok = (a * b) // n < 2 ** 30
        x, y, z = (np.ascontiguousarray(v[ok]) for v in (x, y, z))
        assert len(x) > 1000
        for c in (0, 1):
            for ulps in (-2, -1, 0, 1, 2):
                assert lib.wrong_quotients(x.ctypes.data, y.ctypes.data, z.ctypes.data, c, ulps, len(x)) == 0


# (sequences, rows, parts, compute units, a workgroup per row)
@pytest.mark.parametrize("n, rows, parts, cus, want", [(64, 64, 2, 256, True), (63, 63, 2, 256, True), (62, 62, 2, 256, False), (64, 64, 1, 256, False),
                                                       (16, 16, 2, 64, True), (15, 15, 2, 64, False), (62, 62, 2, 128, True), (300, 300, 2, 304, True),
                                                       (70, 70, 2, 304, False), (64, 80, 2, 256, True), (64, 81, 2, 256, False), (8, 512, 8, 64, False)])
def test_append_takes_a_workgroup_per_row_past_one_per_compute_unit(lib, n, rows, parts, cus, want):
    lib.by_rows.argtypes = [ctypes.c_int, ctypes.c_int, ctypes.c_int64, ctypes.c_int]
    assert bool(lib.by_rows(rows, n, (rows // 16 + 2 * n + 1) * parts, cus)) == want


# (sequences, rows, bytes of K and V per row, past the caches)
@pytest.mark.parametrize("n, rows, row, want", [(4, 8, 4096, False), (1, 1000, 4096, False), (9, 1008, 4096, False), (17, 1016, 4096, True), (16, 16, 1024, True),
                                                (15, 15, 4096, False), (16, 1600, 4096, False), (16, 1599, 4096, True), (1, 2048, 4096, False),
                                                (1, 2049, 4096, True), (8, 4096, 4096, True), (136, 4224, 4096, True), (1 << 20, 1 << 26, 1, True)])
def test_append_goes_past_the_caches_by_size(lib, n, rows, row, want):
    lib.past_caches.argtypes = [ctypes.c_int, ctypes.c_int, ctypes.c_int64]
    assert bool(lib.past_caches(rows, n, rows * row)) == want


# A part: "work" before it arrives, "wait" while it looks at the counter, "merge" while it holds a slice, "gone".  An atomic is
# one step; what a waiting part's look finds may be old news by the time it acts, so giving up is possible at any time, and
# so is drawing once all have arrived.
@pytest.mark.parametrize("nparts", [2, 4, 5, 7, 16])
def test_every_order_of_arrivals_draws_and_leaves(lib, nparts):
    S = lib.slices()
    start = (0, (nparts, 0, 0), 0, False)        # word, parts in (work, wait, merge), slices taken (bits), reset
    seen, stack = {start}, [start]
    ends = 0

    def event(w, what):
        return (0, True) if lib.last_event(w, nparts) else (w + what, False)

    while stack:
        w, (work, wait, merge), taken, reset = stack.pop()
        nxt = []
        if work + wait + merge == 0:
            assert reset and w == 0 and taken == (1 << S) - 1
            ends += 1
            continue
        assert not reset                         # nobody has an event left after the reset
        if work:
            if lib.arrived_last(w, nparts):
                assert work == 1 and not taken & 1
                nxt.append((w + lib.arrive(), (0, wait, merge + 1), taken | 1, False))
            else:
                nxt.append((w + lib.arrive(), (work - 1, wait + 1, merge), taken, False))
        if wait:
            v, r = event(w, lib.leave())
            nxt.append((v, (work, wait - 1, merge), taken, r))
        for frm in ([1] if wait and lib.arrivals(w) == nparts else []) + ([2] if merge else []):
            s, (v, r) = lib.slice(w), event(w, lib.draw())
            parts = [work, wait, merge]
            parts[frm] -= 1
            if s >= 0:
                assert 1 <= s < S and not taken >> s & 1 and not r
                parts[2] += 1
                taken_now = taken | 1 << s
            else:
                taken_now = taken
            nxt.append((v, tuple(parts), taken_now, r))
        for x in nxt:
            assert 0 <= x[0] < 1 << 24
            if x not in seen:
                seen.add(x)
                stack.append(x)
    assert ends == 1
