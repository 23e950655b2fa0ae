"""Buckets that end inside an 8-element vector, where the two buckets' ranges
differ: the elements before the bucket's end then quantize far outside the next
bucket's scale, and must not reach its codes.  Gradients fall by a factor of 64
from one bucket to the next and rise again (so residuals leave both scales), and
short last buckets hold 1 to 5 elements.  State bit for bit against the oracle."""
import pytest
import torch

from gpu_harness import GpuOracleRun

pytestmark = pytest.mark.gpu
bf16, f32 = torch.bfloat16, torch.float32


class SteppedScales(GpuOracleRun):
    """Every other bucket's gradients divided by 64 (exact in both types)."""

    def grads(self, t):
        out = []
        for g in super().grads(t):
            odd = (torch.arange(g.numel(), device=g.device) // self.bucket) % 2 == 1
            out.append(torch.where(odd, g / 64, g))
        return out


@pytest.mark.parametrize("grad", ["bf16", "f32"])
@pytest.mark.parametrize("bits,rounding", [(4, 0), (4, 1), (8, 0), (8, 1)],
                         ids=["near4", "rand4", "near8", "rand8"])
@pytest.mark.parametrize("block,bucket", [(1024, 1027), (1024, 1110), (4096, 4097), (4096, 5004), (4096, 5007),
                                          (8192, 8197), (12304, 12310)])
def test_bucket_ends_inside_a_vector(block, bucket, bits, rounding, grad):
    kw = dict(param_dtype=bf16, grad_dtype=bf16, grad_scale=1e-3) if grad == "bf16" else {}
    # whole and short last buckets: 1 to 5 elements past a bucket's end
    numels = [q * bucket + r for q, r in ((1, 1), (2, 2), (3, 3), (1, 4), (5, 5), (6, 0))] + [40]
    print(f"[straddle] block {block} bucket {bucket} bits {bits} rounding {rounding} {grad}", flush=True)
    run = SteppedScales(numels, block=block, bucket=bucket, density=0.01, window=2, ef_bits=bits, ef_rounding=rounding,
                        ef_seed=21, **kw)
    for _ in range(4):
        run.step(check_moments=False)
    run.opt.close()
