"""Single-token steps of float32 flows against the CPU oracle: every width whose LayerNorm is part of a projection and
one whose is not, every head size of the attention kernel below and above the keys it walks at a time, row counts around
the 16-row blocks, head columns that no tile divides; flows made for so many samples that the whole-sequence projections
take the steps.  Needs an MI355X.  Tolerance: 1e-4 on the block's output (the float32 bound)."""
import numpy as np
import pytest

import workloads as wl

pytestmark = pytest.mark.gpu

CASES = [
    # width, heads, layers, tokens, token size, batch
    (64, 2, 2, 12, 3, 6),          # LayerNorm as a launch of its own
    (128, 4, 2, 49, 16, 1),
    (128, 8, 1, 35, 5, 17),        # head size 16, second row block with one row
    (256, 4, 2, 70, 7, 16),
    (512, 4, 1, 20, 12, 33),       # head size 128
    (768, 12, 1, 9, 11, 40),
    (1024, 16, 1, 7, 48, 3),
    (128, 4, 1, 1, 5, 3),          # one token: copied
    # past the keys that the attention kernel walks at a time (256, 128, 64 and 32 at head sizes 16 to 128), with a remainder
    (64, 4, 1, 270, 4, 2),
    (64, 2, 1, 140, 3, 3),
    (128, 2, 1, 133, 5, 2),
    (256, 2, 1, 70, 4, 2),
    (48, 4, 1, 10, 4, 5),          # head size 12: the plain path
    (256, 4, 1, 6, 5, 3073),       # max_batch * width above 768 K: whole-sequence projections, token size that pads the head matrix
    (1024, 16, 1, 5, 8, 769),
]


@pytest.mark.parametrize("W,H,N,T,D,B", CASES, ids=[f"w{c[0]}_dh{c[0] // c[1]}_t{c[3]}_b{c[5]}" for c in CASES])
def test_float32_steps_match_oracle(orc32, W, H, N, T, D, B):
    import torch
    import paper_2505_24791_amd as sjd
    cfg = wl.FlowConfig("seq_f32", n_blocks=2, n_layers=N, width=W, n_heads=H, seq_len=T, token_dim=D, batch=B, bf16=False)
    print(cfg, flush=True)
    blob = wl.make_weights(cfg, perturb_affine=True)
    z = wl.make_latent(cfg, seed=17)
    zd = torch.from_numpy(z).cuda()
    f = sjd.Flow(cfg)
    f.load_weights(blob)
    for j in range(2):                                     # block 1 works on the reversed token order
        x = f.sequential_inverse_block(j, zd)
        assert torch.equal(f.sequential_inverse_block(j, zd), x)
        one = f.sequential_inverse_block(j, zd[-1:].contiguous())       # a row does not depend on the rows beside it
        assert torch.equal(one[0], x[-1])
        pick = sorted({0, B // 2, B - 1})
        ref = np.stack([orc32.sequential_inverse_block(cfg, blob, j, z[b]) for b in pick])
        assert np.abs(x.cpu().numpy()[pick] - ref).max() <= 1e-4
    f.close()


@pytest.mark.parametrize("W,H,N,T,D,B", [
    (64, 4, 3, 70, 3, 2),          # more keys than are walked at a time (64), head size 16
    (64, 1, 1, 257, 5, 2),         # several batches of cached keys, head size 64
    (128, 8, 2, 130, 16, 5),       # the same at 32 keys at a time
    (128, 1, 1, 34, 2, 3),         # head size 128
    (128, 4, 1, 3, 1024, 2),       # the largest token size
    (128, 2, 1, 4, 511, 2),        # an odd one: the head matrix is padded
    (128, 4, 2, 9, 16, 300),       # more samples than CUs
])
def test_narrow_block_in_one_launch(orc32, W, H, N, T, D, B):
    """Widths 64 and 128: the whole block in one launch and, on request, per-step launches."""
    import torch
    import paper_2505_24791_amd as sjd
    cfg = wl.FlowConfig("seq_f32", n_blocks=2, n_layers=N, width=W, n_heads=H, seq_len=T, token_dim=D, batch=B, bf16=False)
    print(cfg, flush=True)
    blob = wl.make_weights(cfg, perturb_affine=True)
    z = wl.make_latent(cfg, seed=19)
    zd = torch.from_numpy(z).cuda()
    f = sjd.Flow(cfg)
    f.load_weights(blob)
    for j in range(2):
        f.set_sequential_path(0)
        f.profile_enable(range(sjd.PROF_FAMILIES))
        x = f.sequential_inverse_block(j, zd)
        prof = f.profile_read()
        f.profile_enable([])
        assert prof["decode_fused"]["launches"] == 1 and prof["decode_gemm"]["launches"] == 0
        assert torch.equal(f.sequential_inverse_block(j, zd), x)
        assert torch.equal(f.sequential_inverse_block(j, zd[-1:].contiguous())[0], x[-1])
        f.set_sequential_path(1)
        steps = f.sequential_inverse_block(j, zd)
        for b in (0, B - 1):
            ref = orc32.sequential_inverse_block(cfg, blob, j, z[b])
            assert np.abs(x[b].cpu().numpy() - ref).max() <= 1e-4
            assert np.abs(steps[b].cpu().numpy() - ref).max() <= 1e-4
    f.close()
