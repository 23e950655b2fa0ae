"""Buckets spanning Top-K blocks where a lane's run of 64 elements holds a
bucket's end (odd bucket sizes put it inside an 8-element vector), in every
error-feedback format and gradient type, and the bucket reduction with one,
several and more than 64 blocks per bucket; binary32 gradients of whole
4096-element blocks with 8-bit codes.  State bit for bit against the oracle."""
import pytest
import torch

from gpu_harness import GpuOracleRun

pytestmark = pytest.mark.gpu
bf16, f32 = torch.bfloat16, torch.float32
BF = dict(param_dtype=bf16, grad_dtype=bf16, grad_scale=1e-3)

CASES = {
    "bucket5003_bf16": dict(bucket=5003, **BF),
    "bucket5003_f32": dict(bucket=5003),
    "bucket4099_f32_ef8": dict(bucket=4099, ef_bits=8),
    "bucket4099_bf16_ef8": dict(bucket=4099, ef_bits=8, **BF),
    "bucket10007_bf16_randomized": dict(bucket=10007, ef_rounding=1, ef_seed=5, **BF),
    "bucket10007_f32_randomized8": dict(bucket=10007, ef_bits=8, ef_rounding=1, ef_seed=6),
    "bucket4096_one_block": dict(bucket=4096, **BF),
    "bucket300000_many_blocks": dict(bucket=300000, **BF),
    "block1024_bucket1111": dict(block=1024, bucket=1111, **BF),
    "block1024_bucket90000": dict(block=1024, bucket=90000),
    "block8192_bucket8195_bf16": dict(block=8192, bucket=8195, **BF),
    "block8192_bucket20011_f32": dict(block=8192, bucket=20011),
    "block12304_bucket15001": dict(block=12304, bucket=15001, **BF),
    "bf16_bucket32_inside": dict(bucket=32, **BF),
    "bf16_bucket8_randomized": dict(bucket=8, ef_rounding=1, ef_seed=3, **BF),
    "f32_ef8_inside": dict(ef_bits=8),
    "f32_ef8_bucket8": dict(ef_bits=8, bucket=8),
    "f32_randomized_bucket32": dict(ef_rounding=1, ef_seed=9, bucket=32),
}


@pytest.mark.parametrize("name", CASES)
def test_span_edges(name):
    kw = dict(dict(window=3, density=0.01), **CASES[name])
    print(f"[span edges] {name} {kw}", flush=True)
    block = kw.get("block", 4096)
    n = 330000 if kw.get("bucket", 0) >= 90000 else 5 * block + 1237
    run = GpuOracleRun([n, block, 501], **kw)
    for _ in range(4):
        run.step(check_moments=False)
    run.opt.close()


# binary32 gradients with 8-bit codes: the forms that load each lane's run
# directly (buckets below 64, buckets spanning blocks), at sparse and dense rows
@pytest.mark.parametrize("kw", [
    dict(bucket=8, density=0.05),
    dict(bucket=16, density=0.05, value_f32=True),
    dict(bucket=32, ef_rounding=1, ef_seed=12),
    dict(bucket=32, density=0.05, ef_rounding=1, ef_seed=13),
    dict(bucket=4099, density=0.05),
    dict(bucket=5003, value_f32=True),
], ids=str)
def test_f32_ef8_direct(kw):
    test_args = dict(dict(window=3, density=0.01, ef_bits=8), **kw)
    print(f"[f32 ef8 direct] {test_args}", flush=True)
    run = GpuOracleRun([5 * 4096 + 1237, 4096, 501], **test_args)
    for _ in range(4):
        run.step(check_moments=False)
    run.opt.close()
