"""What the framework is timed on: one MicroAdam step over a parameter list,
mid-training (the window full), through the package's public classes.

Every case is a step of ``MicroAdam.step(grads)`` (or, for one case, of the
``torch.optim`` front-end ``MicroAdamW``) on parameters, gradients and
optimizer state resident in device memory.  The gradients of successive steps
are four windows of one random buffer, each shifted against the last, so that
an element sees other values from step to step as it does in training.
"""
from __future__ import annotations

import math
import random

import torch

from paper_2405_15593_amd import MICROADAM_ROUND_NEAREST, MICROADAM_ROUND_RANDOMIZED, MicroAdam, make_config
from paper_2405_15593_amd.optim import MicroAdamW
from paper_2405_15593_amd.workloads import bert_base_shapes, llama2_shapes

RING = 4            # gradient windows that successive steps take in turn
SHIFT = 8 * 1013    # elements between two windows: a multiple of 16 bytes, of no block or bucket
LR = 1e-4
BETA1, BETA2, EPS = 0.9, 0.999, 1e-8
DTYPES = {"bf16": torch.bfloat16, "f32": torch.float32}


def _case(name, shapes, **kw):
    c = {"name": name, "list": shapes, "d": 0, "tensors": 1, "layers": 0, "param": "bf16", "grad": "bf16",
         "dist": "student_t4", "scale": 1e-3, "block": 4096, "density": 0.01, "window": 10, "bucket": 64,
         "bits": 4, "randomized": False, "weight_decay": 0.0, "front": "engine"}
    c.update(kw)
    return c


def listed():
    return [
        # the smallest call: one flat fp32 tensor of 2^20 elements, normal
        # gradients (a fused small model, or one rank's shard of one)
        _case("flat1m_f32", "flat", d=1 << 20, param="f32", grad="f32", dist="normal", scale=1.0),
        # a small model trained in fp32 through torch.optim: the 4-layer,
        # 256-wide transformer of the package's training loop, 53 tensors of
        # 256 to 262,144 elements, so most blocks are ragged
        _case("tinylm_f32_optim", "tinylm", param="f32", grad="f32", front="optim"),
        # fine-tuning BERT-base in bf16: 196 tensors, 109 M parameters
        _case("bert_base_bf16", "bert", dist="normal"),
        # the same in fp32 storage, with decoupled weight decay
        _case("bert_base_f32", "bert", param="f32", grad="f32", dist="normal", weight_decay=0.01),
        # fine-tuning Llama-2-7B: the headline list, 291 tensors, 6.74e9 parameters
        _case("llama2_7b_bf16", "llama2_7b", layers=32),
        # the longer window, m = 20, that the paper also trains Llama-2-7B
        # with; two decoder layers, as one rank of a sharded run holds them
        _case("llama_layers_window20", "llama_layers", layers=2, window=20),
        # 8-bit error-feedback codes
        _case("llama_layers_ef8", "llama_layers", layers=2, bits=8),
        # the unbiased randomized quantizer of the convergence analysis
        _case("llama_layers_randomized", "llama_layers", layers=2, randomized=True),
        # quantization buckets of 100,000 elements, spanning Top-K blocks
        _case("llama_layers_bucket100k", "llama_layers", layers=2, bucket=100_000),
        # short Top-K blocks of 1024 elements
        _case("bert_base_block1024", "bert", block=1024, dist="normal"),
        # a dense selection, 5% of each 4096-element block (k = 205), over
        # tensors of odd sizes
        _case("odd_density5", "split", d=120_000_007, tensors=41, density=0.05),
        # one flat tensor of 1.5e9 with Top-K blocks of 65536, 5%, a window
        # of 20 and gradients full of exact ties
        _case("flat1p5b_ties_bf16", "flat", d=1_500_000_000, dist="student_t2_snapped64", block=65536, density=0.05,
              window=20, bucket=128),
    ]


def draw(rng: random.Random):
    """One more case of these ranges: 2^18 to 2^30 parameters in 1 to 64
    tensors of any size, the storage types, blocks, densities, windows and
    error-feedback formats above and what lies between them."""
    param, grad = rng.choice([("bf16", "bf16")] * 4 + [("f32", "f32")] * 3 + [("bf16", "f32")])
    block = rng.choice([1024, 2048, 4096, 4096, 4096, 4096, 16384, 65536])
    dist = rng.choice(["normal", "student_t4", "student_t4"] + (["student_t2_snapped64"] if block > 4096 else []))
    bucket = rng.choice([32, 64, 64, 64, 128, 256] + ([100_000] if block == 4096 else []))
    d = int(2.0 ** rng.uniform(18.0, 30.0)) + rng.randrange(1000)
    kw = dict(d=d, tensors=int(2.0 ** rng.uniform(0.0, 6.0)), param=param, grad=grad, dist=dist, block=block,
              density=rng.choice([0.01, 0.01, 0.01, round(math.exp(rng.uniform(math.log(0.005), math.log(0.05))), 4)]),
              window=rng.choice([10, 10, 10, 20, 20, rng.randint(5, 20)]), bucket=bucket,
              bits=rng.choice([4, 4, 4, 8]), randomized=rng.random() < 0.2,
              weight_decay=rng.choice([0.0, 0.0, 0.01]))
    c = _case("", "flat" if kw["tensors"] == 1 else "split", **kw)
    del c["name"]
    return c


# ---------------------------------------------------------------- shapes
def _tinylm_numels(vocab=1024, dim=256, layers=4, seq=128):
    block = [dim, dim, 3 * dim * dim, 3 * dim, dim * dim, dim, dim, dim, 4 * dim * dim, 4 * dim, 4 * dim * dim, dim]
    return [vocab * dim, seq * dim] + block * layers + [dim, dim, vocab * dim]


def _split_numels(d, n):
    """n sizes that sum to d, spread over a factor of about a thousand."""
    r = random.Random(d)
    w = [math.exp(r.uniform(0.0, 7.0)) for _ in range(n)]
    sizes = [max(1, int(d * x / sum(w))) for x in w[:-1]]
    return sizes + [max(1, d - sum(sizes))]


def numels_of(case):
    kind = case["list"]
    if kind == "flat":
        return [case["d"]]
    if kind == "split":
        return _split_numels(case["d"], case["tensors"])
    if kind == "tinylm":
        return _tinylm_numels()
    if kind == "bert":
        shapes = bert_base_shapes()
    elif kind == "llama2_7b":
        shapes = llama2_shapes(4096, 11008, case["layers"])
    else:  # decoder layers without the embedding, the final norm and the head
        shapes = llama2_shapes(4096, 11008, case["layers"])[1:-2]
    return [math.prod(s) for s in shapes]


def _offsets(numels):
    """Places of the tensors in one flat buffer, each on a multiple of 8
    elements (16 bytes), and the buffer's length."""
    offs, at = [], 0
    for n in numels:
        offs.append(at)
        at += (n + 7) // 8 * 8
    return offs, at


# ---------------------------------------------------------------- inputs
def _fill(out, dist, scale, gen):
    """Fills a flat tensor with scale times the named distribution."""
    step = 1 << 26
    for lo in range(0, out.numel(), step):
        part = out[lo:lo + step]
        new = lambda: torch.empty(part.numel(), dtype=torch.float32, device=out.device)  # noqa: E731
        z = new().normal_(generator=gen)
        if dist != "normal":
            # Student-t: a normal over the root of chi2/df, where a chi2 of 2
            # degrees is -2 ln U
            e = new().exponential_(generator=gen)
            if dist == "student_t4":
                e.add_(new().exponential_(generator=gen)).mul_(0.5)
            z.div_(e.clamp_min_(1e-12).sqrt_())
        if dist == "student_t2_snapped64":
            j = (torch.log2(z.abs().clamp_min_(1e-30)) * 4 + 40).round_().clamp_(0, 63)
            z = torch.where(z < 0, -1.0, 1.0) * torch.exp2((j - 40) / 4)
        part.copy_(z.mul_(scale))


def _inputs(case, seed):
    """(flat parameters, flat gradient buffer) of a case, from the seed alone."""
    _, length = _offsets(numels_of(case))
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    flat = torch.empty(length, dtype=DTYPES[case["param"]], device="cuda")
    _fill(flat, "normal", 0.02, gen)
    gbuf = torch.empty(length + (RING - 1) * SHIFT, dtype=DTYPES[case["grad"]], device="cuda")
    _fill(gbuf, case["dist"], case["scale"], gen)
    return flat, gbuf


def prepare(case, seed):
    numels = numels_of(case)
    offs, _ = _offsets(numels)
    flat, gbuf = _inputs(case, seed)
    params = [flat[o:o + n] for o, n in zip(offs, numels)]
    grads = [[gbuf[r * SHIFT + o:r * SHIFT + o + n] for o, n in zip(offs, numels)] for r in range(RING)]
    state = {"flat": flat, "grads": grads, "turn": 0}
    if case["front"] == "optim":
        state["params"] = [torch.nn.Parameter(p) for p in params]
        state["optim"] = MicroAdamW(state["params"], lr=LR, betas=(BETA1, BETA2), eps=EPS,
                                    weight_decay=case["weight_decay"], density=case["density"],
                                    window=case["window"], ef_bucket=case["bucket"], topk_block=case["block"])
        state["out"] = {"params": flat}
    else:
        cfg = make_config(density=case["density"], beta1=BETA1, beta2=BETA2, eps=EPS, lr=LR,
                          weight_decay=case["weight_decay"], window=case["window"], ef_bits=case["bits"],
                          ef_bucket=case["bucket"], topk_block=case["block"], seed=seed,
                          ef_rounding=MICROADAM_ROUND_RANDOMIZED if case["randomized"] else MICROADAM_ROUND_NEAREST)
        state["engine"] = MicroAdam(params, cfg)
    for _ in range(case["window"]):  # the window is full from here on
        _step(state)
    if case["front"] == "engine":
        opt = state["engine"]
        lay = opt.layout(0)
        pairs = lay.stats_plane + 2 * lay.bucket_table_bytes if lay.bucket_table_bytes else lay.window_plane
        state["out"] = {"params": flat, "codes": opt.state_view[:lay.stats_plane],
                        "pairs": opt.state_view[lay.stats_plane:pairs],
                        "window": opt.state_view[lay.window_plane:]}
    return state


def _step(state):
    grads = state["grads"][state["turn"]]
    state["turn"] = (state["turn"] + 1) % RING
    if "optim" in state:
        for p, g in zip(state["params"], grads):
            p.grad = g
        state["optim"].step()
    else:
        state["engine"].step(grads)


def run(state):
    """One optimizer step; the updated parameters and optimizer state."""
    _step(state)
    return state["out"]


# ---------------------------------------------------------------- measures
def _block_k(s, density):
    return min(s, max(1, math.ceil(density * s - 1e-9)))


def work(case):
    """Parameters read and written, gradients read, codes and bucket pairs
    read and written, one window row written and the others read."""
    size = {"bf16": 2, "f32": 4}
    total = flops = 0.0
    for n in numels_of(case):
        full, tail = divmod(n, case["block"])
        k = full * _block_k(case["block"], case["density"]) + (_block_k(tail, case["density"]) if tail else 0)
        total += n * (2 * size[case["param"]] + size[case["grad"]] + 2 * case["bits"] / 8)
        total += 2 * 8 * math.ceil(n / case["bucket"]) + 4 * k * case["window"]
        # decode and add 3, compare 1, zero 1, min/max 2, quantize 4, update 1;
        # per window entry: two weighted sums 5, the decrement 6
        flops += 12 * n + 11 * k * case["window"]
    return {"bytes": total, "flops": flops}


def tolerance(case):
    """Codes, bucket pairs and window rows are fixed bit for bit by the method
    (they do not depend on the parameters); parameters differ where the
    binary32 rebuild rounds another way."""
    # binary32 storage: 3.9e-7 and 1.3e-6 from the 64-bit result with weight
    # decay (its factor is rounded to binary32), 8e-9 and 1.9e-7 without
    if case["param"] == "f32":
        return {"rel": 1.5e-6, "max": 5e-6}
    # bf16 storage: about one parameter in 1e7 lies near enough to a rounding
    # boundary to move by an ulp (rel 2e-7 from the 64-bit result rounded to
    # bf16); an ulp is at most 2^-7 of the value, and two steps may add up.
    # Other roundings of the decrement (a few binary32 ulps) move some tens of
    # times as many.
    return {"rel": 1e-5, "max": 0.016}


# ---------------------------------------------------------------- in 64 bits
def _philox_w24(n, j, t, seed, device):
    """The 24-bit integers of the randomized rounding's stream for elements
    [0, n) of tensor j at step t: Philox4x32-10 (Salmon et al., SC 2011)."""
    quads = (n + 3) // 4
    i = torch.arange(quads, dtype=torch.int64, device=device)
    m32 = 0xFFFFFFFF
    c = [i & m32, i >> 32, torch.full_like(i, j), torch.full_like(i, t)]
    k0, k1 = seed & m32, (seed >> 32) & m32

    def mul(a, x):  # high and low word of a 32 x 32-bit product
        lo, hi = a * (x & 0xFFFF), a * (x >> 16)      # below 2^48
        s = lo + ((hi & 0xFFFF) << 16)                # below 2^49
        return (hi >> 16) + (s >> 32), s & m32

    for r in range(10):
        h0, l0 = mul(0xD2511F53, c[0])
        h1, l1 = mul(0xCD9E8D57, c[2])
        c = [h1 ^ c[1] ^ k0, l1, h0 ^ c[3] ^ k1, l0]
        k0, k1 = (k0 + 0x9E3779B9) & m32, (k1 + 0xBB67AE85) & m32
    return (torch.stack(c, 1).reshape(-1)[:n] >> 8).to(torch.float64)


def _exact_tensor(case, j, theta, grad_of, steps, seed):
    """theta after `steps` steps on one tensor.  What the method holds in
    binary32 (the accumulator, the bucket pairs) is computed in binary32, the
    moments and the update in binary64; parameters are rounded to their
    storage type between steps."""
    n, block, bucket, m = theta.numel(), case["block"], case["bucket"], case["window"]
    dev = theta.device
    # as a tensor: torch divides by a Python number through its reciprocal
    levels = torch.full((1,), 255.0 if case["bits"] == 8 else 15.0, device=dev)
    nbk = -(-n // bucket)
    bk = torch.arange(n, device=dev) // bucket
    code = torch.zeros(n, dtype=torch.float32, device=dev)
    lo, hi = (torch.zeros(nbk, dtype=torch.float32, device=dev) for _ in range(2))
    nfull = n // block
    parts = [(0, nfull, block)] if nfull else []
    if n % block:
        parts.append((nfull * block, 1, n % block))
    rows = []
    store = theta.dtype
    x = theta.double()
    for t in range(1, steps + 1):
        a = grad_of(t).float() + (code * ((hi - lo) / levels)[bk] + lo[bk])
        idx = []
        for at, nb, s in parts:
            part = a[at:at + nb * s].view(nb, s)
            # |a| as bits, the lower index first among equals: no two keys alike
            key = (part.abs().view(torch.int32).long() << 16) + (65535 - torch.arange(s, device=dev))
            top = key.topk(_block_k(s, case["density"]), dim=1, sorted=False).indices
            idx.append((top + torch.arange(nb, device=dev)[:, None] * s).reshape(-1) + at)
            del key, top
        idx = torch.cat(idx)
        rows = (rows + [(idx, a[idx].bfloat16().double())])[-m:]
        a[idx] = 0.0
        pad = torch.cat([a, a[-1:].expand(nbk * bucket - n)]).view(nbk, bucket)
        lo, hi = pad.amin(1), pad.amax(1)
        del pad
        u = ((hi - lo) / levels)[bk]
        y = (a - lo[bk]) / u
        if case["randomized"]:
            fl = y.floor()
            carry = _philox_w24(n, j, t, seed, dev) + ((y - fl) * 16777216.0).floor().double() >= 16777216.0
            y = fl + carry.float()
        else:
            y = y.round()
        code = torch.where(u == 0, torch.zeros_like(y), y.clamp(0.0, 255.0 if case["bits"] == 8 else 15.0))
        del y, u
        z1, z2 = (torch.zeros(n, dtype=torch.float64, device=dev) for _ in range(2))
        for r, (i, v) in enumerate(reversed(rows)):
            z1[i] += BETA1 ** r * v
            z2[i] += BETA2 ** r * v * v
        z1 *= (1 - BETA1) / (1 - BETA1 ** t)
        z2 *= (1 - BETA2) / (1 - BETA2 ** t)
        x = x * (1 - LR * case["weight_decay"]) - LR * z1 / (EPS + z2.sqrt())
        if t < steps:
            x = x.to(store).double()
    return x


def exact(case, seed):
    numels = numels_of(case)
    if sum(numels) > 450_000_000 or (case["randomized"] and max(numels) > 100_000_000):
        return None
    offs, length = _offsets(numels)
    flat, gbuf = _inputs(case, seed)
    out = flat.double()
    for j, (o, n) in enumerate(zip(offs, numels)):
        grad_of = lambda t, o=o, n=n: gbuf[(t - 1) % RING * SHIFT + o:(t - 1) % RING * SHIFT + o + n]  # noqa: E731
        out[o:o + n] = _exact_tensor(case, j, flat[o:o + n], grad_of, case["window"] + 1, seed)
    if case["front"] == "optim":
        return {"params": out}
    return {"params": out, "codes": None, "pairs": None, "window": None}
