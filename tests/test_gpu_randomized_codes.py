"""Randomized rounding where its bracketed form hands over to the exact one:
quantization steps near and below the smallest that the reciprocal serves,
constant residuals (step 0), values on the quantization grid (gradients of few
magnitudes), and all select kernels.  Codes bit for bit against the oracle."""
import pytest
import torch

from gpu_harness import GpuOracleRun

pytestmark = pytest.mark.gpu
bf16 = torch.bfloat16

CASES = {
    "tiny_steps": dict(grad_scale=2e-37, degenerate=True),  # (too small to move a parameter)
    "below_smallest_step": dict(grad_scale=2e-38, degenerate=True),
    "large_steps": dict(grad_scale=1e17),
    "constant": dict(grad_dist="constant", grad_scale=0.25, degenerate=True),
    "signs": dict(grad_dist="signs", grad_scale=1e-2, degenerate=True),
    "few_magnitudes": dict(grad_dist="student_t2_snapped64", grad_scale=1e-3, grad_dtype=bf16, param_dtype=bf16),
    "normal": dict(),
}


@pytest.mark.parametrize("bits", [4, 8])
@pytest.mark.parametrize("block", [1024, 4096, 16384])
@pytest.mark.parametrize("name", CASES)
def test_randomized_codes(name, block, bits):
    kw = dict(CASES[name])
    print(f"[randomized] {name} block {block} bits {bits} {kw}", flush=True)
    run = GpuOracleRun([6 * 4096 + 700, 99], block=block, window=2, ef_bits=bits, ef_rounding=1, ef_seed=17, **kw)
    for _ in range(3):
        run.step(check_moments=False)
    run.opt.close()
