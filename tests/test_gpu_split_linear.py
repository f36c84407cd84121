"""Float32 passes on split operands, where they can go wrong: tile edges of every size, widths whose LayerNorm and attention are the general
kernels, weights of very different scales, weights whose bounds the scales do not cover.  Needs an MI355X."""
import numpy as np
import pytest

import workloads as wl

pytestmark = pytest.mark.gpu


def _flow(cfg, blob):
    import paper_2505_24791_amd as sjd
    f = sjd.Flow(cfg)
    f.load_weights(blob)
    return f


def _tensors(cfg, blob):
    out, off = {}, 0
    for name, shape in wl.block_tensors(cfg):
        n = int(np.prod(shape))
        out[name] = blob[off:off + n].reshape(shape)
        off += n
    return out


# Every operand is hi + lo to 2^-23, a sum of K products then to about 2^-23 sqrt(K) of its terms' size, as with float32 products; two layers of
# some six such roundings each, relative to the result: 4e-6 (seen: 1.1e-6 at eight layers).
@pytest.mark.parametrize("W,H,T,D,B", [
    (512, 8, 129, 12, 3),           # 387 rows: 64x64 tiles, the last of three rows
    (96, 8, 50, 5, 50),             # heads of 12, LayerNorm of any width
    (128, 4, 49, 16, 33),           # heads of 32
    (256, 4, 225, 12, 37),          # 8325 rows
    (512, 8, 256, 33, 32),          # 128x128 and 128x64 tiles
    (768, 12, 193, 3, 5),
    (256, 4, 2, 12, 450),           # attention over two tokens, and over a last query tile of one row
    (256, 4, 769, 7, 2),
], ids=lambda v: str(v))
def test_split_conditioner_against_64_bits(orc64, W, H, T, D, B):
    import torch
    cfg = wl.FlowConfig("split", n_blocks=1, n_layers=2, width=W, n_heads=H, seq_len=T, token_dim=D, batch=B, bf16=False)
    print(cfg, flush=True)
    blob = wl.make_weights(cfg, perturb_affine=True)
    x = wl.make_latent(cfg, seed=31)
    f = _flow(cfg, blob)
    mu, al = f.conditioner(0, torch.from_numpy(x).cuda())
    one = f.conditioner(0, torch.from_numpy(x[-1:].copy()).cuda())                    # same bits in any tile size
    assert torch.equal(one[0][0], mu[-1]) and torch.equal(one[1][0], al[-1])
    for b in (0, B - 1):
        for got, ref in zip((mu, al), orc64.cond(cfg, blob, 0, x[b])):
            err = np.linalg.norm(got[b].cpu().numpy().astype(np.float64) - ref) / np.linalg.norm(ref)
            assert err <= 4e-6
    f.close()


def test_powers_of_two_in_the_weights_change_nothing():
    """LayerNorm's gains and shifts, the queries', the keys' and the values' columns times powers of two that the next matrix (or the keys) takes back:
    the scales follow them, and the results are the same bits."""
    import torch
    cfg = wl.FlowConfig("split", n_blocks=1, n_layers=1, width=256, n_heads=4, seq_len=100, token_dim=6, batch=9, bf16=False)
    print(cfg, flush=True)
    W = cfg.width
    blob = wl.make_weights(cfg, perturb_affine=True)
    x = torch.from_numpy(wl.make_latent(cfg, seed=37)).cuda()
    rng = np.random.default_rng(5)
    two = lambda n: np.ldexp(np.float32(1), rng.integers(-12, 13, n)).astype(np.float32)
    scaled = blob.copy()
    t = _tensors(cfg, scaled)
    for ln, nxt in (("l0.ln1", "l0.w_qkv"), ("l0.ln2", "l0.w_fc1"), ("lnf", "w_head")):
        p = two(W)
        t[ln + "_g"] *= p
        t[ln + "_b"] *= p
        t[nxt] /= p[:, None]
    p = two(W)
    t["l0.w_qkv"][:, :W] *= p
    t["l0.b_qkv"][:W] *= p
    t["l0.w_qkv"][:, W:2 * W] /= p
    t["l0.b_qkv"][W:2 * W] /= p
    p = two(W)
    t["l0.w_qkv"][:, 2 * W:] *= p
    t["l0.b_qkv"][2 * W:] *= p
    t["l0.w_o"] /= p[:, None]
    f, g = _flow(cfg, blob), _flow(cfg, scaled)
    for a, b in zip(f.conditioner(0, x), g.conditioner(0, x)):
        assert torch.equal(a, b)
    f.close()
    g.close()


# Channels that are zero for every input, among live ones whose queries are `spread` powers of two apart: the scales of the live ones are the smallest and
# largest that a head has.  The values weigh so much that the attention's rounding is the result's; bound as above.
@pytest.mark.parametrize("dead", ["query and key", "query", "key", "value", "hidden", "gain"])
@pytest.mark.parametrize("std,spread", [(0.02, 0), (0.002, 0), (0.02, 12)])
def test_dead_channels_take_no_bits_from_the_others(orc64, dead, std, spread):
    import torch
    cfg = wl.FlowConfig("split", n_blocks=1, n_layers=1, width=256, n_heads=4, seq_len=100, token_dim=6, batch=9, bf16=False)
    print(cfg, dead, std, spread, flush=True)
    W = cfg.width
    blob = wl.make_weights(cfg, perturb_affine=True)
    x = wl.make_latent(cfg, seed=43)
    t = _tensors(cfg, blob)
    rng = np.random.default_rng(11)
    for name in ("l0.w_qkv", "l0.w_fc1", "l0.b_qkv", "l0.b_fc1"):
        t[name][...] *= np.float32(std / 0.02)
    t["l0.w_qkv"][:, :W] *= np.float32(0.02 / std * 4)                     # scores of some size all the same
    t["l0.w_o"][...] *= np.float32(0.02 / std * 50)
    if spread:
        p = np.ldexp(np.float32(1), -rng.integers(0, spread + 1, W)).astype(np.float32)
        t["l0.w_qkv"][:, :W] *= p
        t["l0.b_qkv"][:W] *= p
    off = np.concatenate([h * 64 + rng.choice(64, 5, replace=False) for h in range(4)])
    cols = {"query and key": [off, W + off], "query": [off], "key": [W + off], "value": [2 * W + off]}.get(dead, [])
    for c in cols:
        t["l0.w_qkv"][:, c] = 0
        t["l0.b_qkv"][c] = 0
    if dead == "hidden":
        t["l0.w_fc1"][:, off] = 0
        t["l0.b_fc1"][off] = 0
        t["l0.w_fc1"][...] *= np.float32(2.0 ** -10)                       # the live ones' scales far above 1
        t["l0.b_fc1"][...] *= np.float32(2.0 ** -10)
        t["l0.w_fc2"][...] *= np.float32(2.0 ** 12)
    if dead == "gain":
        for ln, nxt in (("l0.ln1", "l0.w_qkv"), ("l0.ln2", "l0.w_fc1"), ("lnf", "w_head")):
            for part in ("_g", "_b"):
                t[ln + part][...] *= np.float32(2.0 ** -20)
                t[ln + part][off] = 0
            t[nxt][...] *= np.float32(2.0 ** 20)
    f = _flow(cfg, blob)
    mu, al = f.conditioner(0, torch.from_numpy(x).cuda())
    for b in (0, 8):
        for got, ref in zip((mu, al), orc64.cond(cfg, blob, 0, x[b])):
            err = np.linalg.norm(got[b].cpu().numpy().astype(np.float64) - ref) / np.linalg.norm(ref)
            assert err <= 4e-6
    f.close()


@pytest.mark.parametrize("kept", [64, 8, 1])
def test_scales_of_a_head_far_apart(orc64, kept):
    """All but `kept` channels of a head have queries and keys of 2^-20 to 1 of the others', each by itself: a score is what the large ones make it, and
    the common scale of the products must leave those their bits.  Bound as above."""
    import torch
    cfg = wl.FlowConfig("split", n_blocks=1, n_layers=1, width=256, n_heads=4, seq_len=100, token_dim=6, batch=9, bf16=False)
    print(cfg, kept, flush=True)
    W = cfg.width
    blob = wl.make_weights(cfg, perturb_affine=True)
    x = wl.make_latent(cfg, seed=47)
    t = _tensors(cfg, blob)
    rng = np.random.default_rng(13)
    p = np.ldexp(np.float32(1), -rng.integers(0, 21, 2 * W)).astype(np.float32)
    large = np.concatenate([h * 64 + rng.choice(64, kept, replace=False) for h in range(4)])
    p[large], p[W + large] = 8, 2
    t["l0.w_qkv"][:, :2 * W] *= p
    t["l0.b_qkv"][:2 * W] *= p
    t["l0.w_o"][...] *= np.float32(50)
    f = _flow(cfg, blob)
    mu, al = f.conditioner(0, torch.from_numpy(x).cuda())
    for b in (0, 8):
        for got, ref in zip((mu, al), orc64.cond(cfg, blob, 0, x[b])):
            err = np.linalg.norm(got[b].cpu().numpy().astype(np.float64) - ref) / np.linalg.norm(ref)
            print(f"{err:.1e}", flush=True)
            assert err <= 4e-6
    f.close()


def _out_of_range(kind, t, W):
    """Weights with a bound outside 2^-40 .. 2^60 on which split operands would go wrong."""
    if kind == "tiny value":      # a value column far below the others that the output projection brings back: its scale would leave it a few bits
        t["l0.w_qkv"][:, 2 * W + 5] *= np.float32(2.0 ** -75)
        t["l0.b_qkv"][2 * W + 5] *= np.float32(2.0 ** -75)
        t["l0.w_o"][5] *= np.float32(2.0 ** 81)
    elif kind == "tiny column":   # an output column of 2^-77
        t["w_head"][:, 3] *= np.float32(2.0 ** -75)
        t["b_head"][3] = 0
    elif kind == "huge":          # a query and a key channel, both exactly zero as sums of 2^90 and -2^90: no float32 scale takes their bound out of a score
        t["l0.ln1_g"][:2] = 0
        t["l0.ln1_b"][:2] = 1
        for c in (7, W + 7):
            t["l0.w_qkv"][:, c] = 0
            t["l0.b_qkv"][c] = 0
            t["l0.w_qkv"][0, c], t["l0.w_qkv"][1, c] = 2.0 ** 90, -2.0 ** 90
    else:                         # an output column that is infinite, which two halves cannot say (the lower one would be infinity less infinity)
        t["w_head"][5, 3] = np.inf


@pytest.mark.parametrize("kind", ["tiny value", "tiny column", "huge", "infinite"])
def test_bounds_out_of_range_keep_the_float32_instruction(orc64, kind):
    """Every output column by itself to float32's own error (the oracle in float32: up to 1.4e-6 here)."""
    import torch
    cfg = wl.FlowConfig("split", n_blocks=1, n_layers=1, width=256, n_heads=4, seq_len=60, token_dim=6, batch=16, bf16=False)
    print(cfg, kind, flush=True)
    blob = wl.make_weights(cfg, perturb_affine=True)
    _out_of_range(kind, _tensors(cfg, blob), cfg.width)
    x = wl.make_latent(cfg, seed=41)
    f = _flow(cfg, blob)
    mu, al = f.conditioner(0, torch.from_numpy(x).cuda())
    for got, ref in zip((mu, al), orc64.cond(cfg, blob, 0, x[3])):
        got = got[3].cpu().numpy().astype(np.float64)
        for d in range(cfg.token_dim):
            if np.isfinite(ref[:, d]).all():
                assert np.linalg.norm(got[:, d] - ref[:, d]) <= 6e-6 * np.linalg.norm(ref[:, d]), d
            else:
                assert kind == "infinite" and d == 3 and np.array_equal(got[1:, d], ref[1:, d])
    f.close()
