"""Prefill softmax: weights are computed against the reference of the steps before, which moves when a half step's sum shows that it
was too low.  Scores that rise within and across half steps, fall, jump past the range of fp32 exponentials, or rise for some
columns only, on tiles of every workgroup shape, whole and in parts, against the float64 oracle."""
import numpy as np
import pytest

from oracle import ref_c
from paper_2511_21862_amd import workloads as W

pytestmark = pytest.mark.gpu

# score of token j of n, in units of the natural exponent
PROFILES = {
    "rise": lambda j, n: 50.0 * j / n,
    "steep": lambda j, n: 0.7 * j,
    "fall": lambda j, n: 50.0 * (n - j) / n,
    "saw": lambda j, n: 9.0 * ((j // 32) % 3),
    "jump": lambda j, n: np.where(j < n // 3, 0.0, 300.0) + 0.01 * j,
    "last": lambda j, n: np.where(j < n - 3, 0.0, 40.0),
}
# (the four-wave workgroups, whole and in parts; eight waves; key groups; without the tile list)
OPTS = [{"prefill_groups": 1, "prefill_split": 1}, {"prefill_groups": 1, "prefill_split": 3}, {"prefill_groups": 1, "prefill_waves": 8},
        {"prefill_groups": 4, "prefill_split": 1}, {"prefill_groups": 4, "prefill_split": 2}, {"prefill_sorted": 0}]


def batch(heads, profile, seed):
    """Chunks whose rows all look along one direction u per kv head, and keys that lie along it by the profile."""
    Hq, Hkv, hd = heads
    q_lens, ctx_lens = [70, 33, 2], [0, 700, 165]
    b = W.build_batch(Hq=Hq, Hkv=Hkv, hd=hd, q_lens=q_lens, ctx_lens=ctx_lens, num_blocks=80, seed=seed, poison=True)
    rng = np.random.default_rng(seed)
    u = rng.choice([-1.0, 1.0], size=(Hkv, hd))
    for i in range(b.num_seqs):
        k, v = W.gather_logical(b, i)
        n = k.shape[0]
        s = np.asarray(PROFILES[profile](np.arange(n), n), np.float64)
        s = s[:, None] * np.where(np.arange(Hkv) % 2 == 0, 1.0, 0.5)          # some kv heads rise less than others
        keys = u * s[:, :, None] + 0.2 * rng.standard_normal((n, Hkv, hd))
        W.scatter_logical(b, i, W.f32_to_bf16_bits(keys.astype(np.float32)), v)
    q = np.repeat(u, Hq // Hkv, axis=0) / np.sqrt(hd) * rng.uniform(0.2, 1.0, size=(b.total_q, Hq, 1))   # and some columns
    b.q[:] = W.f32_to_bf16_bits(q.astype(np.float32)).reshape(b.q.shape)
    return b


@pytest.mark.parametrize("profile", PROFILES)
@pytest.mark.parametrize("heads", [(16, 4, 128), (14, 2, 128), (16, 2, 64)], ids=str)
def test_scores_that_outgrow_the_reference(heads, profile):
    from gpu_util import assert_parity, run_gpu, say
    b = batch(heads, profile, 91)
    want = ref_c.attn_mixed(b.q, b.k_cache, b.v_cache, b.block_tables, b.seq_lens, b.query_start_loc, b.ctx_lens)
    for opts in OPTS:
        say(f"case: {heads} {profile} {opts}")
        assert_parity(run_gpu(b, options=opts), want, f"{profile} {opts}")
