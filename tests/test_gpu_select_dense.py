"""The select's form for denser rows (k above 58 of 4096) and for every block of
up to 2048 elements, where it can go wrong: the smallest and largest k of its range, tie
groups across the threshold, a zero bound and overflowing candidates (both
fall back to the search over all elements), ragged tails with few entries, and
the error-feedback formats.  State bit for bit against the oracle."""
import pytest
import torch

from gpu_harness import GpuOracleRun

pytestmark = pytest.mark.gpu
bf16, f32 = torch.bfloat16, torch.float32
BF = dict(param_dtype=bf16, grad_dtype=bf16, grad_scale=1e-3)

CASES = {
    "smallest_k59": dict(density=59 / 4096, **BF),
    "k205_student_t": dict(density=0.05, grad_dist="student_t4", **BF),
    "k205_f32": dict(density=0.05),
    "k205_f32_values": dict(density=0.05, value_f32=True),
    "largest_k384": dict(density=384 / 4096),
    "above_k385": dict(density=385 / 4096),
    "overflowing_candidates": dict(density=0.09, grad_dist="signs", degenerate=True),
    "ties_k205": dict(density=0.05, grad_dist="student_t2_snapped64", **BF),
    "ties_k205_f32_values": dict(density=0.05, grad_dist="student_t2_snapped64", value_f32=True),
    "zero_bound": dict(density=0.05, grad_dist="sparse_spikes", degenerate=True),
    "block2048_k65": dict(block=2048, density=65 / 2048, **BF),
    "block2048_k103_ties": dict(block=2048, density=0.05, grad_dist="student_t2_snapped64", **BF),
    "block2048_k256": dict(block=2048, density=0.125, window=2),
    "block2048_k257": dict(block=2048, density=257 / 2048, window=2),
    "block2048_f32_values": dict(block=2048, density=0.1, value_f32=True),
    "block1024_k128": dict(block=1024, density=0.125, window=2, **BF),
    "block1024_k129": dict(block=1024, density=129 / 1024, window=2, **BF),
    "block1024_ties": dict(block=1024, density=0.05, grad_dist="student_t2_snapped64", value_f32=True),
    "block512_signs": dict(block=512, density=0.02, grad_dist="signs", degenerate=True),
    "block3008_bucket16": dict(block=3008, bucket=16, density=0.04),
    "ef8": dict(density=0.03, ef_bits=8, **BF),
    "randomized": dict(density=0.03, ef_rounding=1, ef_seed=11, **BF),
    "spanning_buckets": dict(density=0.05, bucket=10000, **BF),
}


@pytest.mark.parametrize("name", CASES)
def test_select_dense(name):
    kw = dict(dict(window=3), **CASES[name])
    print(f"[select dense] {name} {kw}", flush=True)
    block = kw.get("block", 4096)
    run = GpuOracleRun([3 * block + 1000, block, 77], **kw)
    for _ in range(5):
        run.step(check_moments=False)
    run.opt.close()
