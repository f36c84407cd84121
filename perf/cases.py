"""The work that is timed: what a user of this package has it do, through its public calls.

A flow is sampled (the inverse pass, with a per-block choice of the sequential or the Jacobi inverse), a single
block is inverted one way or the other, or data is mapped forward to a latent with its log-determinant.  The listed
cases run over the range of such calls: one image and whole batches, widths 128 to 1024, 49 to 1024 tokens, round and
ragged sizes, IEEE half, bfloat16 and float32 flows.  Weights are drawn as in ``workloads`` (matrices and positions
N(0, 0.02^2), the head N(0, 0.01^2), biases and LayerNorm parameters perturbed), latents are N(0, 1).
"""
import math

import torch

import paper_2505_24791_amd as sjd
from workloads import FlowConfig, block_tensors, blob_floats, block_floats

_DTYPES = {"f32": sjd.DTYPE_F32, "bf16": sjd.DTYPE_BF16, "f16": sjd.DTYPE_F16}

# Jacobi passes of one block that the thresholds in use take on these flows (the mean over samples, 8 to 12 at
# tau = 1e-3 and 10 to 12 at 1e-4): the work of a block is that many whole-sequence passes
_PASSES = {1e-2: 7, 1e-3: 9, 1e-4: 11}

_DEFAULT = {"dtype": "f16", "jacobi_mask": 0, "tau": 1e-3, "refine_below": 0.0}


def _case(name, call, batch, tokens, dim, blocks, layers, width, heads, **kw):
    c = {"name": name, "call": call, "batch": batch, "tokens": tokens, "dim": dim, "blocks": blocks, "layers": layers,
         "width": width, "heads": heads}
    c.update(_DEFAULT)
    c.update(kw)
    return c


def listed():
    return [
        # a small float32 flow on 28x28 images in patches of 4: the correctness configuration, and what a call costs
        # when there is hardly any work in it
        _case("small float32 flow", "sample", 4, 49, 16, 4, 2, 128, 4, dtype="f32", jacobi_mask=0b1110),
        # one image at a time from a 32x32 flow: the latency of an interactive request
        _case("one image", "sample", 1, 256, 12, 4, 4, 512, 8, jacobi_mask=0b1110),
        # the same flow, an ordinary batch
        _case("batch of 64", "sample", 64, 256, 12, 4, 4, 512, 8, jacobi_mask=0b1110),
        # a narrow six-block flow, a batch and a token count that no tile divides
        _case("narrow ragged batch", "sample", 37, 225, 12, 6, 6, 256, 4, jacobi_mask=0b111110),
        # a wide batch of 32x32 images on an eight-block flow
        _case("batch of 256", "sample", 256, 256, 12, 8, 8, 768, 12, jacobi_mask=0b11111110),
        # 128x128 images: long sequences at the largest width, the benchmark's own step
        _case("long sequences", "sample", 32, 1024, 48, 8, 8, 1024, 16, jacobi_mask=0b11111110),
        # every block by Jacobi decoding (the ablation), 64x64 images, the flow cut to four blocks
        _case("every block Jacobi", "sample", 128, 256, 48, 4, 8, 1024, 16, jacobi_mask=0b1111),
        # data to latent with the log-determinant: density evaluation of a batch of 64x64 images, the flow cut to four blocks
        _case("forward", "forward", 128, 256, 48, 4, 8, 1024, 16),
        # density evaluation in float32
        _case("forward float32", "forward", 16, 256, 12, 2, 4, 512, 8, dtype="f32"),
        # one block token by token against the key/value cache, ragged sizes, long enough for per-step launches
        _case("sequential block", "sequential", 19, 777, 48, 1, 8, 1024, 16),
        # a threshold under the rounding floor of half operands: a sample's last passes run in float32
        _case("refined block", "jacobi", 32, 256, 12, 1, 4, 512, 8, tau=1e-4, refine_below=1e-3),
        # shift and scale of every token of a few ragged sequences, bfloat16 operands
        _case("conditioner bfloat16", "conditioner", 3, 1000, 48, 1, 8, 768, 12, dtype="bf16"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _seconds(case):
    """A rough duration, to keep drawn cases below the largest listed one."""
    rate = 5e13 if case["dtype"] == "f32" else 4e14
    n_seq = _n_sequential(case)
    jacobi_f32 = 0.0
    if case["refine_below"] > 0:
        jacobi_f32 = 3 * _pass_flops(case) / 5e13
    launch = 12e-6 * 7 if case["dtype"] == "f32" else 6e-6 * 7
    return (work(case)["flops"] / rate + jacobi_f32 + n_seq * case["tokens"] * case["layers"] * launch
            * (1 + case["batch"] / 32.0))


def draw(rng):
    while True:
        call = rng.choice(["sample", "sample", "sample", "sequential", "jacobi", "forward", "conditioner"])
        dtype = rng.choice(["f16", "f16", "f16", "f32"] if call in ("sample", "jacobi") else ["f16", "f16", "bf16", "f32"])
        width = rng.choice([128, 256, 512] if dtype == "f32" else [256, 512, 768, 1024])
        heads = 4 if width == 128 else width // 64
        tokens = _log_int(rng, 16, 1024)
        batch = _log_int(rng, 1, 256)
        if batch * tokens > 65536:
            continue
        blocks = rng.randint(2, 8) if call in ("sample", "forward") else 1
        full = (1 << blocks) - 1
        kw = {"dtype": dtype}
        if call == "sample":
            kw["jacobi_mask"] = rng.choice([full & ~1, full & ~1, full])
            kw["tau"] = rng.choice([1e-2, 1e-3, 1e-3])
        if call == "jacobi":
            kw["tau"] = rng.choice([1e-2, 1e-3])
            if dtype == "f16" and rng.random() < 0.5:
                kw.update(tau=1e-4, refine_below=1e-3)
        c = _case("", call, batch, tokens, rng.randint(3, 48), blocks, rng.randint(1, 8), width, heads, **kw)
        del c["name"]
        if _seconds(c) <= 0.5 and blob_floats(_config(c)) <= 250_000_000:
            return c


def _config(case):
    return FlowConfig("perf", n_blocks=case["blocks"], n_layers=case["layers"], width=case["width"],
                      n_heads=case["heads"], seq_len=case["tokens"], token_dim=case["dim"], batch=case["batch"],
                      bf16=case["dtype"] != "f32", tau=case["tau"])


def _draw_weights(cfg, gen):
    """The weight blob of ``workloads.make_weights(perturb_affine=True)``'s recipe, drawn on the GPU, as a host array."""
    blob = torch.empty(blob_floats(cfg), dtype=torch.float32, device="cuda")
    blob.normal_(generator=gen)
    off = 0
    for _ in range(cfg.n_blocks):
        for name, shape in block_tensors(cfg):
            n = math.prod(shape)
            part = blob[off:off + n]
            base = name.split(".")[-1]
            if base.endswith("_g"):
                part.mul_(0.1).add_(1.0)
            else:
                part.mul_(0.01 if base == "w_head" else 0.02)
            off += n
    if cfg.bf16:                     # 16-bit flows come with bfloat16 weights
        for a in range(0, blob.numel(), 1 << 26):
            part = blob[a:a + (1 << 26)]
            part.copy_(part.bfloat16())
    return blob.cpu().numpy()


def prepare(case, seed):
    cfg = _config(case)
    gen = torch.Generator(device="cuda").manual_seed(seed)
    flow = sjd.Flow(cfg, dtype=_DTYPES[case["dtype"]])
    flow.load_weights(_draw_weights(cfg, gen))
    z = torch.randn((cfg.batch, cfg.seq_len, cfg.token_dim), dtype=torch.float32, device="cuda", generator=gen)
    return {"case": case, "flow": flow, "z": z,
            "opts": sjd.JacobiOpts(tau=case["tau"], refine_below=case["refine_below"])}


def run(state):
    # The pass counts that come with a sample are left out of the outputs: a sample whose difference norm passes the
    # threshold narrowly takes one pass more or less in another order of sums (1 in 140 of half-precision samples, 1
    # in 9 of refined ones), and the iterate it ends with is the same to within the tolerance.
    case, flow, z = state["case"], state["flow"], state["z"]
    call = case["call"]
    if call == "sample":
        return flow.sample(z, case["jacobi_mask"], state["opts"])[0]
    if call == "jacobi":
        return flow.jacobi_inverse_block(0, z, state["opts"])[0]
    if call == "sequential":
        return flow.sequential_inverse_block(0, z)
    if call == "forward":
        latent, logdet = flow.forward(z)
        return {"z": latent, "logdet": logdet}
    mu, alpha = flow.conditioner(0, z)
    return {"mu": mu, "alpha": alpha}


def _pass_flops(case):
    """One whole-sequence pass of one block's conditioner (causal attention counted on the lower triangle)."""
    b, t, w, d, n = case["batch"], case["tokens"], case["width"], case["dim"], case["layers"]
    return 2.0 * b * t * (n * 12 * w * w + 3 * d * w) + 2.0 * b * t * (t + 1) * w * n


def _n_sequential(case):
    if case["call"] == "sequential":
        return 1
    return case["blocks"] - bin(case["jacobi_mask"]).count("1") if case["call"] == "sample" else 0


def work(case):
    n_seq = _n_sequential(case)
    if case["call"] in ("sample", "jacobi"):
        passes = (case["blocks"] - n_seq) * _PASSES[case["tau"]] + n_seq
    else:
        passes = case["blocks"]                          # a sequential block is one pass in flops, token by token
    cfg = _config(case)
    weights = case["blocks"] * block_floats(cfg) * (4 if case["dtype"] == "f32" else 2)
    state = case["batch"] * case["tokens"] * case["dim"] * 4
    return {"bytes": float(weights + 2 * state), "flops": passes * _pass_flops(case)}


def tolerance(case):
    # Measured by running each case again on latents that differ by 1e-6 (every 16-bit rounding then falls anew), and
    # against a float32 flow of the same weights; stated at about four times the largest seen.
    if case["dtype"] == "f32":
        return {"rel": 5e-6, "max": 3e-5}        # seen: 1.1e-6, 6.4e-6
    if case["dtype"] == "bf16":
        return {"rel": 1.5e-2, "max": 0.1}       # seen: 4.3e-3, 2.3e-2
    if case["refine_below"] > 0:
        return {"rel": 2e-4, "max": 2e-3}        # seen: 5.1e-5, 4.2e-4
    return {"rel": 3e-3, "max": 3e-2}            # seen: 7.8e-4, 6.9e-3
