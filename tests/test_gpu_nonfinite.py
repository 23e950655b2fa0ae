"""Non-finite gradients: NaN and +-inf in some Top-K blocks of one tensor.

The method leaves them undefined (every step of Algorithm 1 assumes finite
values), so the library promises only this: a block whose gradient holds a
NaN or an infinity gets unspecified parameters and state, and every other
block, of that tensor or of another, is computed exactly as if the
non-finite values were not there.  Blocks are independent in the step (with
buckets inside blocks), so each clean block and the second tensor must match,
bit for bit, a run on the same inputs with the non-finite values replaced by
zeros.  Both select kernels are covered: B_d = 4096 and B_d = 65536."""
import pytest

import paper_2405_15593_amd as ma

pytestmark = pytest.mark.gpu


def _run(numels, block, density, window, grads, steps, bucket):
    import torch
    dev = torch.device("cuda:0")
    gen = torch.Generator(device="cpu").manual_seed(5)
    params = [(torch.randn(n, generator=gen) * 0.02).to(dev, torch.bfloat16) for n in numels]
    cfg = ma.make_config(density=density, window=window, ef_bucket=bucket, topk_block=block, lr=1e-3)
    opt = ma.MicroAdam(params, cfg)
    for t in range(steps):
        opt.step([g[t % len(g)] for g in grads])
    torch.cuda.synchronize()
    moments = [opt.debug_moments(j) for j in range(len(numels))]
    out = [p.clone() for p in params], moments
    opt.close()
    return out


@pytest.mark.parametrize("block,bucket,density,window", [(4096, 64, 0.01, 3), (65536, 128, 0.05, 4)],
                         ids=["block4096", "block65536"])
def test_nonfinite_blocks_are_isolated(block, bucket, density, window):
    import torch
    dev = torch.device("cuda:0")
    na = block * 5 + 1000          # five full blocks and a ragged one
    nb = block + 333
    gen = torch.Generator(device="cpu").manual_seed(11)
    bad_blocks = [1, 3]            # blocks of tensor A that get NaN / inf
    ga, ga_clean, gb = [], [], []
    for s in range(2):
        a = torch.randn(na, generator=gen) * 1e-3
        clean = a.clone()
        # block 1: NaNs, one of them the largest-index element; block 3: +-inf
        a[block + 7] = float("nan")
        a[2 * block - 1] = float("nan")
        a[3 * block + 100] = float("inf")
        a[3 * block + 101] = float("-inf")
        clean[block + 7] = clean[2 * block - 1] = clean[3 * block + 100] = clean[3 * block + 101] = 0.0
        ga.append(a.to(dev, torch.bfloat16))
        ga_clean.append(clean.to(dev, torch.bfloat16))
        gb.append((torch.randn(nb, generator=gen) * 1e-3).to(dev, torch.bfloat16))
    print(f"[nonfinite] block={block} numels={[na, nb]} bad blocks {bad_blocks}", flush=True)
    steps = window + 2
    (p_bad, m_bad) = _run([na, nb], block, density, window, [ga, gb], steps, bucket)
    print("[nonfinite] run with NaN/inf done", flush=True)
    (p_ok, m_ok) = _run([na, nb], block, density, window, [ga_clean, gb], steps, bucket)
    print("[nonfinite] clean run done", flush=True)
    # the second tensor: bit-identical parameters and moments
    assert torch.equal(p_bad[1].view(torch.int16), p_ok[1].view(torch.int16))
    for x, y in zip(m_bad[1], m_ok[1]):
        assert torch.equal(x.view(torch.int32), y.view(torch.int32))
    # tensor A: every block other than the bad ones bit-identical
    good = torch.ones(na, dtype=torch.bool, device=dev)
    for q in bad_blocks:
        good[q * block:(q + 1) * block] = False
    assert torch.equal(p_bad[0][good].view(torch.int16), p_ok[0][good].view(torch.int16))
    for x, y in zip(m_bad[0], m_ok[0]):
        assert torch.equal(x[good].view(torch.int32), y[good].view(torch.int32))


# the forms that the cases above do not reach: dense rows (k above 58) and blocks
# of up to 2048 elements (vector maxima, the short blocks' updates), binary32
# gradients (their exchange and direct loads), 8-bit and randomized codes
FORMS = {
    "k205": dict(density=0.05),
    "k205_f32": dict(density=0.05, grad="f32"),
    "k385_all_elements": dict(density=385 / 4096),
    "f32": dict(grad="f32"),
    "f32_ef8": dict(grad="f32", ef_bits=8),
    "f32_ef8_bucket16": dict(grad="f32", ef_bits=8, ef_bucket=16),
    "f32_values": dict(density=0.05, grad="f32", value_f32=True),
    "ef8": dict(ef_bits=8),
    "randomized": dict(ef_rounding=1),
    "randomized8_f32": dict(grad="f32", ef_rounding=1, ef_bits=8),
    "block1024": dict(topk_block=1024),
    "block1024_k52": dict(topk_block=1024, density=0.05),
    "block1024_k52_f32_randomized": dict(topk_block=1024, density=0.05, grad="f32", ef_rounding=1),
    "block2048_k103": dict(topk_block=2048, density=0.05),
    "block512": dict(topk_block=512, ef_bucket=8),
}


@pytest.mark.parametrize("name", FORMS)
def test_nonfinite_forms(name):
    import torch
    dev = torch.device("cuda:0")
    kw = dict(FORMS[name])
    gdt = torch.float32 if kw.pop("grad", "bf16") == "f32" else torch.bfloat16
    if kw.pop("value_f32", False):
        kw["window_value_dtype"] = ma.MICROADAM_F32
    block, window, steps = kw.get("topk_block", 4096), 4, 6
    numels = [block * 7 + 1000 % block, block + 33]
    bad = {1: ["nan"], 3: ["inf", "-inf"], 5: ["nan"] * (block - 3), 7: ["nan"]}  # block 5: 3 finite values left
    gen = torch.Generator(device="cpu").manual_seed(23)
    grads = {"bad": [], "clean": []}
    for _ in range(steps):
        a, b = (torch.randn(n, generator=gen) * 1e-3 for n in numels)
        clean = a.clone()
        for q, values in bad.items():
            at = slice(q * block + 2, q * block + 2 + len(values))
            a[at] = torch.tensor([float(v) for v in values])
            clean[at] = 0.0
        for key, x in (("bad", a), ("clean", clean)):
            grads[key].append([x.to(dev, gdt), b.to(dev, gdt)])

    def run(gs):
        pg = torch.Generator(device="cpu").manual_seed(5)
        params = [(torch.randn(n, generator=pg) * 0.02).to(dev, torch.bfloat16) for n in numels]
        opt = ma.MicroAdam(params, ma.make_config(**dict(dict(window=window, lr=1e-3, seed=9), **kw)))
        for g in gs:
            opt.step(g)
        torch.cuda.synchronize()
        moments = [opt.debug_moments(j) for j in range(2)]
        opt.close()
        return params, moments

    print(f"[nonfinite forms] {name} {kw} {gdt}", flush=True)
    p_bad, m_bad = run(grads["bad"])
    p_ok, m_ok = run(grads["clean"])
    good = [torch.ones(n, dtype=torch.bool, device=dev) for n in numels]
    for q in bad:
        good[0][q * block:(q + 1) * block] = False
    for j in range(2):
        assert torch.equal(p_bad[j][good[j]], p_ok[j][good[j]])
        for x, y in zip(m_bad[j], m_ok[j]):
            assert torch.equal(x[good[j]].view(torch.int32), y[good[j]].view(torch.int32))
