"""Float32 projections of whole-sequence passes through the conditioner, against the CPU oracle: row counts that give
every tile size of the matrix kernel and its edges, token sizes that pad the head matrix, a width off the matrix kernel.
Needs an MI355X.  Tolerance: 1e-4 (the float32 bound; values are of order 0.1 to 1)."""
import numpy as np
import pytest

import workloads as wl

pytestmark = pytest.mark.gpu

CASES = [
    # width, heads, tokens, token size, batch: rows 1, 63, 65, 1000, 8192, 9000
    (128, 4, 1, 3, 1),
    (128, 4, 63, 5, 1),
    (256, 4, 13, 16, 5),
    (64, 2, 100, 7, 10),
    (128, 2, 256, 12, 32),
    (512, 8, 250, 33, 36),
    (72, 2, 50, 4, 3),             # 72 = 8 mod 16: the plain kernel
]


@pytest.mark.parametrize("W,H,T,D,B", CASES, ids=[f"w{c[0]}_rows{c[2] * c[4]}_d{c[3]}" for c in CASES])
def test_float32_conditioner_matches_oracle(orc32, W, H, T, D, B):
    import torch
    import paper_2505_24791_amd as sjd
    cfg = wl.FlowConfig("lin_f32", n_blocks=2, n_layers=1, width=W, n_heads=H, seq_len=T, token_dim=D, batch=B, bf16=False)
    print(cfg, flush=True)
    blob = wl.make_weights(cfg, perturb_affine=True)
    x = wl.make_latent(cfg, seed=23)
    f = sjd.Flow(cfg)
    f.load_weights(blob)
    for j in range(2):
        mu, al = f.conditioner(j, torch.from_numpy(x).cuda())
        one_mu, one_al = f.conditioner(j, torch.from_numpy(x[-1:].copy()).cuda())     # same bits in any tile size
        assert torch.equal(one_mu[0], mu[-1]) and torch.equal(one_al[0], al[-1])
        for b in sorted({0, B // 2, B - 1}):
            rmu, ral = orc32.cond(cfg, blob, j, x[b][::-1] if j else x[b])             # the oracle works in processing order
            if j:
                rmu, ral = rmu[::-1], ral[::-1]
            assert np.abs(mu[b].cpu().numpy() - rmu).max() <= 1e-4
            assert np.abs(al[b].cpu().numpy() - ral).max() <= 1e-4
    f.close()


@pytest.mark.parametrize("W,H,T,D,B", [
    (128, 4, 96, 16, 16),          # rows * width on the line below which the step kernels take a pass
    (128, 4, 97, 16, 16),          # and past it
    (256, 4, 15, 5, 3),            # 45 rows, the last block of sixteen with thirteen
    (768, 12, 17, 33, 1),
    (1024, 16, 24, 48, 8),
], ids=lambda v: str(v))
def test_passes_of_few_rows_match_oracle(orc32, W, H, T, D, B):
    import torch
    import paper_2505_24791_amd as sjd
    cfg = wl.FlowConfig("few_f32", n_blocks=2, n_layers=2, width=W, n_heads=H, seq_len=T, token_dim=D, batch=B, bf16=False)
    print(cfg, flush=True)
    blob = wl.make_weights(cfg, perturb_affine=True)
    x = wl.make_latent(cfg, seed=29)
    f = sjd.Flow(cfg)
    f.load_weights(blob)
    f.profile_enable(range(sjd.PROF_FAMILIES))
    mu, al = f.conditioner(1, torch.from_numpy(x).cuda())
    prof = f.profile_read()
    f.profile_enable([])
    few = B * T * W <= 192 * 1024
    assert prof["other"]["launches"] == (1 if few else 6)          # the embedding, and LayerNorm where it is a launch of its own
    one_mu, one_al = f.conditioner(1, torch.from_numpy(x[-1:].copy()).cuda())         # one row block or two: the same bits
    assert torch.equal(one_mu[0], mu[-1]) and torch.equal(one_al[0], al[-1])
    for b in (0, B - 1):
        rmu, ral = orc32.cond(cfg, blob, 1, x[b][::-1])
        assert np.abs(mu[b].cpu().numpy() - rmu[::-1]).max() <= 1e-4
        assert np.abs(al[b].cpu().numpy() - ral[::-1]).max() <= 1e-4
    f.close()


@pytest.mark.parametrize("W,H,T,B", [(64, 16, 1, 2), (64, 16, 130, 2), (64, 8, 65, 3), (64, 4, 33, 2), (128, 4, 17, 2), (128, 4, 150, 2), (96, 8, 70, 2)],
                         ids=lambda v: str(v))
def test_rowwise_attention_of_small_heads(orc32, W, H, T, B):
    """Heads of 4 to 32 (the wave splits into groups of keys) and of 12 (it does not), keys below, at and past the groups' eight rows."""
    import torch
    import paper_2505_24791_amd as sjd
    cfg = wl.FlowConfig("att_f32", n_blocks=1, n_layers=2, width=W, n_heads=H, seq_len=T, token_dim=5, batch=B, bf16=False)
    print(cfg, flush=True)
    blob = wl.make_weights(cfg, perturb_affine=True)
    x = wl.make_latent(cfg, seed=37)
    f = sjd.Flow(cfg)
    f.load_weights(blob)
    mu, al = f.conditioner(0, torch.from_numpy(x).cuda())
    for b in range(B):
        rmu, ral = orc32.cond(cfg, blob, 0, x[b])
        assert np.abs(mu[b].cpu().numpy() - rmu).max() <= 1e-4
        assert np.abs(al[b].cpu().numpy() - ral).max() <= 1e-4
    f.close()
