"""The matrix-core projection kernels one by one against the CPU oracle (its `linear` and `gelu`
primitives in float64 on the same 16-bit-rounded operands).  Needs an MI355X.

Shapes span several tiles of each kernel with ragged edges in M and N; the error bound is the one
float32 accumulation of 16-bit products allows plus, for 16-bit results, one output rounding."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

KERNELS = {1: "256x128x32 staged", 2: "256x256x64 LDS-direct", 3: "128x128x64", 0: "auto"}
# K values give the register-staged kernels 1..16 k-tiles: both main loops (two register sets from 4
# k-tiles on when the count is even, else one set) with zero, one and several steady-state iterations
SHAPES = [(300, 200, 128), (700, 1000, 64), (513, 257, 320), (1024, 768, 256), (400, 384, 512), (260, 130, 384)]


@pytest.fixture(scope="module")
def torch_cuda():
    import torch
    assert torch.cuda.is_available(), "these tests need the GPU"
    return torch


def _operands(torch, M, N, K, dtype, seed):
    g = np.random.default_rng(seed)
    a = torch.from_numpy(g.standard_normal((M, K)).astype(np.float32)).to(dtype)
    w = torch.from_numpy((g.standard_normal((K, N)) * 0.05).astype(np.float32)).to(dtype)
    bias = torch.from_numpy(g.standard_normal(N).astype(np.float32) * 0.1)
    n_pad = (N + 255) // 256 * 256
    wt = torch.zeros((n_pad, K), dtype=dtype)
    wt[:N] = w.T
    return a, w, wt, bias


@pytest.mark.parametrize("kernel", sorted(KERNELS), ids=[KERNELS[k].replace(" ", "_") for k in sorted(KERNELS)])
@pytest.mark.parametrize("dtype_name", ["float16", "bfloat16"])
def test_projection_kernels_match_oracle(torch_cuda, orc64, kernel, dtype_name):
    import paper_2505_24791_amd as sjd
    torch = torch_cuda
    dtype = getattr(torch, dtype_name)
    out_eps = 2.0 ** -11 if dtype_name == "float16" else 2.0 ** -8
    for si, (M, N, K) in enumerate(SHAPES):
        a, w, wt, bias = _operands(torch, M, N, K, dtype, seed=10 + si)
        ref = orc64.linear(a.float().numpy(), w.float().numpy(), bias.numpy())        # float64, same rounded operands
        scale = np.abs(ref).max()
        ad, wd, bd = a.cuda(), wt.cuda(), bias.cuda()
        c = sjd.op_linear_h16(ad, wd, bd, M, N, K, 0, kernel=kernel).float().cpu().numpy()
        assert np.abs(c - ref).max() <= out_eps * scale + 1e-3, (KERNELS[kernel], M, N, K)
        cg = sjd.op_linear_h16(ad, wd, bd, M, N, K, 1, kernel=kernel).float().cpu().numpy()
        refg = orc64.gelu(ref)
        assert np.abs(cg - refg).max() <= out_eps * scale + 1e-3, (KERNELS[kernel], M, N, K)
        r0 = np.random.default_rng(99).standard_normal((M, N)).astype(np.float32)
        rd = torch.from_numpy(r0.copy()).cuda()
        sjd.op_linear_h16(ad, wd, bd, M, N, K, 2, resid=rd, kernel=kernel)
        assert np.abs(rd.cpu().numpy() - (r0 + ref)).max() <= 2e-4 * scale + 1e-4, (KERNELS[kernel], M, N, K)


def test_projection_rows_do_not_depend_on_their_neighbours(torch_cuda):
    """A row's result is the same bits whether it is computed alone in a small problem or deep
    inside a large one (what lets converged samples leave the batch without changing anything)."""
    import paper_2505_24791_amd as sjd
    torch = torch_cuda
    M, N, K = 1024, 512, 256
    a, w, wt, bias = _operands(torch, M, N, K, torch.float16, seed=5)
    ad, wd, bd = a.cuda(), wt.cuda(), bias.cuda()
    for kernel in (1, 2, 3):
        full = sjd.op_linear_h16(ad, wd, bd, M, N, K, 0, kernel=kernel)
        part = sjd.op_linear_h16(ad[300:556].contiguous(), wd, bd, 256, N, K, 0, kernel=kernel)
        assert torch.equal(full[300:556], part)


def _tiles(M, N, bm, bn):
    return -(-M // bm) * -(-N // bn)


@pytest.mark.parametrize("M,N,K,tile", [
    # 64x64 ring: one k-tile, fewer k-tiles than stages, edges, long k, an odd number of k-tiles
    (1, 24, 64, "64x64"), (49, 96, 128, "64x64"), (64, 64, 192, "64x64"), (65, 65, 256, "64x64"),
    (257, 500, 2048, "64x64"), (700, 1000, 320, "64x64"),
    # 64x128 ring of three stages: fewer k-tiles than stages, edges on both sides, one 96-column tile (a head), two tiles per CU and more
    (4000, 1024, 256, "64x128"), (1990, 1900, 64, "64x128"), (1990, 1900, 128, "64x128"), (32700, 96, 1024, "64x128"),
    (3001, 1900, 320, "64x128"), (900, 4000, 1024, "64x128"),
    # more tiles than that, or a second round too short for it, or a weight too large
    (3001, 2300, 128, "128x128"), (3001, 1900, 192, "128x128"), (500, 5000, 576, "128x128"), (700, 3800, 1280, "128x128"),
])
def test_small_launches_give_the_tile_kernels_bits(torch_cuda, M, N, K, tile):
    """The automatic choice for launches that do not fill the chip walks k in the same order as the 128x128 kernel: same bits."""
    import paper_2505_24791_amd as sjd
    torch = torch_cuda
    # the choice, restated
    t6 = _tiles(M, N, 64, 128)
    assert _tiles(M, N, 128, 128) <= 512
    small = t6 <= (768 if K >= 256 else 512) and (N <= 2560 or N * K <= (4 << 20 if N <= 4096 else 5 << 19))
    assert tile == ("64x64" if _tiles(M, N, 64, 64) <= 512 else "64x128" if small else "128x128")
    for dtype in (torch.float16, torch.bfloat16):
        a, _, wt, bias = _operands(torch, M, N, K, dtype, seed=M)
        ad, wd, bd = a.cuda(), wt.cuda(), bias.cuda()
        for epi in (0, 1):
            assert torch.equal(sjd.op_linear_h16(ad, wd, bd, M, N, K, epi), sjd.op_linear_h16(ad, wd, bd, M, N, K, epi, kernel=3)), epi
        r = [torch.arange(M * N, dtype=torch.float32).reshape(M, N).cuda() * 1e-3 for _ in range(2)]
        for rd, kernel in zip(r, (0, 3)):
            sjd.op_linear_h16(ad, wd, bd, M, N, K, 2, resid=rd, kernel=kernel)
        assert torch.equal(r[0], r[1])


@pytest.mark.parametrize("M,N,K,one_round", [
    (8690, 1024, 128, True), (4500, 3072, 128, False),      # 5 row panels x 4 column tiles on an XCD, 3 x 12
    (2049, 4096, 192, True), (2049, 4352, 192, False),      # 2 x 16: exactly a round of 32 CUs, 2 x 17: one tile more
])
def test_middling_launches_give_the_tile_kernels_bits(torch_cuda, M, N, K, one_round):
    """More than two 128x128 tiles per CU, but no 256x256 tile for every CU: the persistent kernel where no XCD gets more tiles than it
    has CUs, else 128x128 tiles.  Same bits on both sides."""
    import paper_2505_24791_amd as sjd
    torch = torch_cuda
    assert _tiles(M, N, 128, 128) > 512 and _tiles(M, N, 256, 256) < 256
    assert (-(-_tiles(M, 1, 256, 1) // 8) * (N // 256) <= 32) == one_round
    a, _, wt, bias = _operands(torch, M, N, K, torch.float16, seed=N)
    ad, wd, bd = a.cuda(), wt.cuda(), bias.cuda()
    for epi in (0, 1):
        assert torch.equal(sjd.op_linear_h16(ad, wd, bd, M, N, K, epi), sjd.op_linear_h16(ad, wd, bd, M, N, K, epi, kernel=3)), epi
    r = [torch.zeros((M, N)).cuda() for _ in range(2)]
    for rd, kernel in zip(r, (0, 3)):
        sjd.op_linear_h16(ad, wd, bd, M, N, K, 2, resid=rd, kernel=kernel)
    assert torch.equal(r[0], r[1])


@pytest.mark.parametrize("T", [1, 17, 32, 33, 96, 225, 256])
def test_short_attention_matches_oracle_and_the_long_kernel(torch_cuda, orc64, T):
    """Up to 256 tokens and 2048 (sample, head) pairs one workgroup takes a whole pair; with more pairs the kernel with passing key
    tiles does, with the same bits."""
    import paper_2505_24791_amd as sjd
    torch = torch_cuda
    H, W, many = 3, 192, 700
    for dtype, eps in ((torch.float16, 2.0 ** -11), (torch.bfloat16, 2.0 ** -8)):
        g = torch.Generator().manual_seed(T)
        qkv = torch.randn((many * T, 3 * W), generator=g).to(dtype)
        few = sjd.op_attention_h16(qkv[:2 * T].cuda(), 2, T, H)
        assert torch.equal(sjd.op_attention_h16(qkv.cuda(), many, T, H)[:2 * T], few)
        q = qkv[T:2 * T].float().numpy()
        ref = orc64.causal_attention(q[:, :W], q[:, W:2 * W], q[:, 2 * W:], H)
        # probabilities are rounded to 16 bits before the second product: relative eps per term
        assert np.abs(few[T:].float().cpu().numpy() - ref).max() <= 4 * eps * np.abs(q[:, 2 * W:]).max()


@pytest.mark.parametrize("dtype_name", ["float16", "bfloat16"])
def test_gelu_epilogue_of_values_that_are_not_finite(torch_cuda, dtype_name):
    """GELU in its erf form, 0.5 v (1 + erf(v / sqrt 2)): +inf stays +inf, -inf and NaN give NaN, large finite values stay
    themselves.  The values come in through the bias (the product is zero) and, in bfloat16, through a sum that overflows
    float32."""
    import paper_2505_24791_amd as sjd
    torch = torch_cuda
    dtype = getattr(torch, dtype_name)
    inf, nan, N = float("inf"), float("nan"), 512
    special = torch.tensor([inf, -inf, nan, 3.0e38, -3.0e38, 6.0e4, -6.0e4, 15.5, 16.5, -16.5, 0.0, 1.0])
    bias = torch.cat([special, torch.linspace(-8, 8, N - len(special))])
    ref = 0.5 * bias.double() * (1 + torch.erf(bias.double() / 2 ** 0.5))
    eps = 2.0 ** -11 if dtype_name == "float16" else 2.0 ** -8
    runs = []
    for M, K in ((70, 128), (4200, 512), (70, 512)):
        a, wt = torch.zeros((M, K), dtype=dtype).cuda(), torch.zeros((N, K), dtype=dtype).cuda()
        runs += [(f"kernel {k}, {M} rows", sjd.op_linear_h16(a, wt, bias.cuda(), M, N, K, 1, kernel=k)) for k in range(5)]
        if K == 512:
            one = torch.ones(K).cuda()
            runs.append((f"panel, {M} rows", sjd.op_panel_linear_h16(a.float(), wt, bias.cuda(), M, N, 1, ln_g=one, ln_b=one)))
    for what, c in runs:
        c = c.cpu().double()
        for i, v in enumerate(special):
            want = ref[i].to(dtype).double()         # 3e38 is past the largest half
            assert torch.equal(torch.isnan(c[:, i]), torch.isnan(want).expand(len(c))), (what, v)
            if not torch.isnan(want):
                got = c[:, i]
                assert (got == want).all() or ((got - want).abs() <= eps * abs(want) + 1e-7).all(), (what, v, want, got[0])
        rest = slice(len(special), None)
        assert (c[:, rest] - ref[rest]).abs().max() <= eps * 8 + 1e-6, what
    if dtype_name == "bfloat16":
        a, wt = torch.full((70, 128), 3.0e38, dtype=dtype).cuda(), torch.ones((N, 128), dtype=dtype).cuda()
        for k in range(5):
            c = sjd.op_linear_h16(a, wt, torch.zeros(N).cuda(), 70, N, 128, 1, kernel=k)
            assert torch.isinf(c).all() and (c > 0).all(), k


def _moved(torch, t, elements):
    """A contiguous copy of t that starts `elements` past a 16-byte boundary."""
    buf = torch.empty(t.numel() + 8, dtype=t.dtype, device=t.device)
    assert buf.data_ptr() % 16 == 0
    v = buf[elements:elements + t.numel()].view(t.shape)
    v.copy_(t)
    return v


@pytest.mark.parametrize("M,N,K", [
    (70, 256, 128), (3001, 1900, 128),          # the shapes of the two rings
    (5000, 2048, 256),                           # of the persistent kernel with less than a tile per CU
    (16640, 1024, 128), (16640, 1000, 3072),     # of the persistent and the 256x256 kernel
])
def test_operands_off_16_byte_boundaries(torch_cuda, M, N, K):
    """Operands may start anywhere: the kernels whose loads want 16-byte boundaries leave them to those that do not, also when
    they are asked for by number.  Same bits as from aligned operands."""
    import paper_2505_24791_amd as sjd
    torch = torch_cuda
    a, _, wt, bias = _operands(torch, M, N, K, torch.float16, seed=N)
    ad, wd, bd = a.cuda(), wt.cuda(), bias.cuda()
    ref = sjd.op_linear_h16(ad, wd, bd, M, N, K, 0, kernel=3)
    for ea, ew in ((4, 0), (0, 4), (2, 6)):
        am, wm = _moved(torch, ad, ea), _moved(torch, wd, ew)
        assert (am.data_ptr() | wm.data_ptr()) % 16 != 0
        for kernel in range(5):
            assert torch.equal(sjd.op_linear_h16(am, wm, bd, M, N, K, 0, kernel=kernel), ref), (ea, ew, kernel)


@pytest.mark.parametrize("T", [40, 256, 300])
def test_attention_input_off_16_byte_boundaries(torch_cuda, T):
    import paper_2505_24791_amd as sjd
    torch = torch_cuda
    qkv = torch.randn((2 * T, 3 * 128), generator=torch.Generator().manual_seed(T)).half().cuda()
    ref = sjd.op_attention_h16(qkv, 2, T, 2)
    assert torch.equal(sjd.op_attention_h16(_moved(torch, qkv, 4), 2, T, 2), ref)


@pytest.mark.parametrize("M,N,K", [
    (1, 10, 64), (130, 200, 192), (2100, 960, 256),        # 64x64, four stages: fewer k-tiles than stages, an odd number, two tiles to a CU
    (33, 64, 1024), (1217, 960, 2112),                     # 64x64, five stages, and with a few tiles more than CUs 128x64
    (1400, 768, 768), (1345, 1000, 576),                   # 128x64, four stages
    (5000, 520, 64), (2945, 770, 512),                     # 128x64, three stages
    (1500, 2300, 768), (1409, 2817, 1088),                 # 128x128, three stages
    (2945, 770, 2048),                                     # 128x128, four stages
    (4576, 3072, 1024), (2829, 4600, 128),                 # 128x128, two stages, more than two tiles to a CU
    (5429, 766, 128), (1050, 3800, 1024),                  # 64x128, three stages: one more row block of 128 than one a CU
    (8100, 1930, 3072),                                    # deep, a 256x256 tile for every CU
])
@pytest.mark.parametrize("dtype_name", ["float16", "bfloat16"])
def test_every_ring_gives_the_tile_kernels_bits(torch_cuda, M, N, K, dtype_name):
    import paper_2505_24791_amd as sjd
    torch = torch_cuda
    print(M, N, K, dtype_name, flush=True)
    a, _, wt, bias = _operands(torch, M, N, K, getattr(torch, dtype_name), seed=83)
    ad, wd, bd = a.cuda(), wt.cuda(), bias.cuda()
    for epi in (0, 1):
        assert torch.equal(sjd.op_linear_h16(ad, wd, bd, M, N, K, epi), sjd.op_linear_h16(ad, wd, bd, M, N, K, epi, kernel=3))
    r = torch.from_numpy(np.random.default_rng(7).standard_normal((M, N)).astype(np.float32)).cuda()
    r0, r3 = r.clone(), r.clone()
    sjd.op_linear_h16(ad, wd, bd, M, N, K, 2, resid=r0)
    sjd.op_linear_h16(ad, wd, bd, M, N, K, 2, resid=r3, kernel=3)
    assert torch.equal(r0, r3)
