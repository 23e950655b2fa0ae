"""The staged update (blocks of up to 4096 elements) at the edges of its
dispatch: entries per thread at and around each instantiation, rows of one,
two and more 64-entry chunks, the largest stage and the row-by-row form above
it, and decrements outside the range of the fast root and quotient.  Each
against the oracle, with the harness's tolerances."""
import pytest
import torch

from gpu_harness import GpuOracleRun

pytestmark = pytest.mark.gpu
bf16, f32 = torch.bfloat16, torch.float32

CASES = {
    # B_d = 4096, 256 threads: k, m -> entries of the live rows
    "two_per_thread": dict(density=256 / 4096, window=2),                 # 512
    "above_two_per_thread": dict(density=57 / 4096, window=9),            # 513, one chunk per row
    "chunk_64": dict(density=64 / 4096, window=16),                       # 1024
    "chunk_65": dict(density=65 / 4096, window=16, grad_dtype=bf16, param_dtype=bf16, grad_scale=1e-3),  # 1040
    "chunk_128": dict(density=128 / 4096, window=16),                     # 2048
    "chunk_129": dict(density=129 / 4096, window=16),                     # 2064
    "row_of_seven_chunks": dict(density=0.1, window=3, grad_dtype=bf16, param_dtype=bf16, grad_scale=1e-3),
    "largest_stage": dict(density=0.25, window=6, param_dtype=bf16),      # 6144
    "above_largest_stage": dict(density=0.25, window=7, param_dtype=bf16, weight_decay=0.1),  # 7168: row by row
    "largest_stage_f32_values": dict(density=0.2495, window=6, value_f32=True),    # 6132 of 8 bytes
    "above_largest_f32_values": dict(density=0.25, window=6, value_f32=True),
    # B_d = 1024, 64 threads
    "block1024_k52_window20": dict(block=1024, density=0.05, window=20),  # 1040
    "block1024_largest_stage": dict(block=1024, density=0.074, window=20, param_dtype=bf16),  # 1520
    "block1024_above": dict(block=1024, density=0.075, window=20),        # 1540
    # B_d = 2048, 128 threads
    "block2048_window20": dict(block=2048, density=0.01, window=20, param_dtype=bf16),  # 420
    "block1040_four_per_thread": dict(block=1040, bucket=16, density=0.05, window=9),  # 468
    "block2048_largest_stage": dict(block=2048, density=0.0745, window=20),  # 3060
    "block2048_above": dict(block=2048, density=0.075, window=20, param_dtype=bf16, grad_dtype=bf16, grad_scale=1e-3),
    # sqrt and division outside [2^-100, 2^100], eps outside it
    "small_moments": dict(window=3, grad_scale=1e-16, eps=1e-20),
    "large_moments": dict(window=3, grad_scale=1e18),
    "small_eps": dict(window=3, eps=1e-32),
}


@pytest.mark.parametrize("name", CASES)
def test_update_stage(name):
    kw = dict(CASES[name])
    print(f"[update stage] {name} {kw}", flush=True)
    run = GpuOracleRun([2 * kw.get("block", 4096) + 700, 33], **kw)
    for _ in range(kw["window"] + 2):
        run.step(check_moments=run.t % 7 == 0)
    run.opt.close()


# blocks of one wave with rows of 25 to 64 entries, held in registers: the rule's
# edges in k, live rows (4, 7, 10 and 13 at most) and types, and both sides of it
HELD = {
    "k24_window4": dict(density=24 / 1024, window=4),
    "k25_window4": dict(density=25 / 1024, window=4),
    "k64_window5": dict(density=64 / 1024, window=5, param_dtype=bf16),
    "k64_window7_f32_values": dict(density=64 / 1024, window=7, value_f32=True),
    "k65_window7": dict(density=65 / 1024, window=7),
    "k41_window8": dict(density=41 / 1024, window=8),
    "k52_window10": dict(density=0.05, window=10),
    "k52_window11_f32": dict(density=0.05, window=11),
    "k52_window11_bf16": dict(density=0.05, window=11, param_dtype=bf16),
    "k52_window13_f32_values": dict(density=0.05, window=13, param_dtype=bf16, value_f32=True),
    "k52_window14": dict(density=0.05, window=14, param_dtype=bf16),
    "ties": dict(density=0.05, window=6, grad_dist="signs", grad_scale=1e-2, degenerate=True),
    "zero_values": dict(density=0.05, window=3, grad_dist="sparse_spikes", degenerate=True),
    "outside_the_range": dict(density=0.05, window=3, grad_scale=1e-16, eps=1e-20),
    "block512_k26_window10": dict(block=512, density=0.05, window=10, param_dtype=bf16, weight_decay=0.1),
    "block1008_bucket16": dict(block=1008, bucket=16, density=0.04, window=9),
}


@pytest.mark.parametrize("name", HELD)
def test_update_held(name):
    kw = dict(dict(block=1024), **HELD[name])
    print(f"[update held] {name} {kw}", flush=True)
    run = GpuOracleRun([5 * kw["block"] + 700, 33, kw["block"]], **kw)
    for _ in range(kw["window"] + 2):
        run.step(check_moments=False)
    run.opt.close()


def test_update_many_blocks_f32():
    """Binary32 parameters in 8192 and 8193 blocks, the two sides of the rule."""
    for blocks in (8192, 8193):
        print(f"[update held] {blocks} blocks", flush=True)
        run = GpuOracleRun([512 * blocks - 12], block=512, density=26 / 512, window=3,
                           sample=lambda j, nb: (0, 1, nb // 2, nb - 1))
        for _ in range(4):
            run.step(check_moments=False)
        run.opt.close()
