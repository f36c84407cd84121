"""The MLP-input projection with two workgroups per CU, inside a conditioner pass: the same bits as the tile kernels (which the other
tests hold against the oracle), for launches of one tile per CU and of those that the 256x256 kernel does not finish in one round, a last
row tile of one row and of all but one, row panels that the XCDs share unevenly, the shortest k, a width that is no multiple of
256, and launches past the rule.  Needs an MI355X."""
import pytest

import workloads as wl

pytestmark = pytest.mark.gpu

CASES = [
    # width, tokens, batch, layers, taken (rows = tokens * batch; a tile is 128 rows x 256 of the 4 * width columns)
    (1024, 113, 17, 1, True),      # 1921 rows: 16 row tiles, the last with one row, 256 tiles
    (1024, 97, 31, 1, False),      # 3007: one round of the 256x256 kernel
    (1024, 97, 43, 1, True),       # 4171: 33 row tiles, the last with 75
    (768, 255, 18, 2, True),       # 4590: 36, uneven over eight XCDs
    (512, 271, 17, 2, False),      # 4607: one round
    (512, 271, 33, 2, True),       # 8943: 70, the last with all but 17 rows
    (512, 1189, 7, 2, True),       # 8323: 66, the last with three
    (512, 256, 61, 1, True),       # 15616: several tiles per workgroup
    (256, 237, 35, 1, False),      # 8295: one round
    (256, 251, 67, 1, True),       # 16817: k of four k-tiles, the last row tile with 49 rows
    (640, 300, 12, 1, False),      # 3600: one round
    (640, 293, 23, 1, True),       # 6739: ten column tiles
    (768, 127, 65, 1, True),       # 8255: the last row tile with 63
    (1024, 256, 40, 1, True),      # 10240: the workgroups take two to three tiles each
    (320, 300, 64, 1, False),      # k = 320 is not covered: the same kernels on both sides
]


@pytest.mark.parametrize("width,tokens,batch,layers,taken", CASES, ids=[f"w{c[0]}_rows{c[1] * c[2]}" for c in CASES])
@pytest.mark.parametrize("dtype_name", ["f16", "bf16"])
def test_large_passes_give_the_bits_of_the_tile_kernels(launch_rules, width, tokens, batch, layers, taken, dtype_name):
    import torch
    import paper_2505_24791_amd as sjd
    assert bool(launch_rules.duo(tokens * batch, 4 * width, width)) == taken
    print(f"W {width} T {tokens} B {batch} {dtype_name}", flush=True)
    cfg = wl.FlowConfig("duo", n_blocks=1, n_layers=layers, width=width, n_heads=width // 64, seq_len=tokens, token_dim=12, batch=batch, bf16=True)
    f = sjd.Flow(cfg, dtype=sjd.DTYPE_F16 if dtype_name == "f16" else sjd.DTYPE_BF16)
    f.load_weights(wl.make_weights(cfg, perturb_affine=True))
    x = torch.from_numpy(wl.make_latent(cfg, seed=31)).cuda()
    mu, al = f.conditioner(0, x)
    again = f.conditioner(0, x)
    assert torch.isfinite(mu).all() and torch.equal(mu, again[0]) and torch.equal(al, again[1])
    f.set_projection_path(1)
    tmu, tal = f.conditioner(0, x)
    assert torch.equal(mu, tmu) and torch.equal(al, tal)
    f.close()
