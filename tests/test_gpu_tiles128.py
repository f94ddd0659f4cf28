"""The 128 x 128 GEMM kernel (tiled fp8 between decode and the 256 x 256 grid, bf16 above 64
tokens) as the planner chooses it: bit for bit the row-split kernel's results on exact-integer data (their
sums are exact in any order), and repeatable on random data."""
import sys

import numpy as np
import pytest
import torch

import gen

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def S():
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_2606_10445_amd as S
    return S


# (axis, M, N, K, dense_begin): 144 to 256 tiles without K slices, ragged rows, tokens and
# columns, partial last steps of both kinds, all-2:4 and all-dense; then K slices (fewer
# tiles, K from 28 chunks of 512), which may end on either side of the boundary.
CASES = [(1, 257, 6500, 2080, 1056), (0, 385, 5000, 2048, 3000), (1, 513, 4608, 2048, 2048), (0, 300, 6528, 2048, 0),
         (1, 640, 5120, 2112, 32), (0, 256, 11300, 2048, 8432), (1, 1537, 1250, 2304, 1728),
         (1, 100, 2412, 14368, 10016), (1, 250, 1100, 14336, 14336), (0, 70, 2304, 14336, 1200), (1, 90, 2435, 15000, 96)]
CASES = [(a, M, N, K // 32 * 32, db, gen.FP8) for a, M, N, K, db in CASES]
# K slices and a dense region that starts off multiples of 4 (its partial sums are not in whole quads)
CASES += [(0, 70, 2304, 14336, 1202, gen.FP8)]
# bf16, row-major: several rounds, partial steps (boundary and K off multiples of 64), rows off
# multiples of 16, all-2:4, all-dense, K slices
CASES += [(1, 513, 5000, 4128, 2080, gen.BF16), (0, 513, 9001, 4096, 6001, gen.BF16), (1, 700, 4608, 4128, 4128, gen.BF16),
          (0, 300, 8192, 4128, 0, gen.BF16), (1, 200, 2600, 16416, 12320, gen.BF16), (0, 65, 25600, 2080, 19200, gen.BF16)]
# bf16 on the 256 x 256 kernel: ragged rows and tokens, a boundary and K inside a step, all-2:4,
# all-dense, a row boundary off multiples of 16
CASES256 = [(0, 1030, 9000, 2080, 6001, gen.BF16), (1, 1300, 7003, 2112, 1056, gen.BF16),
            (1, 1100, 8200, 2080, 2080, gen.BF16), (0, 2049, 5000, 2048, 0, gen.BF16), (0, 1200, 9000, 2080, 6001, gen.BF16)]


@pytest.mark.parametrize("axis,M,N,K,db,dtype", CASES + CASES256)
def test_planned_tiles_exact(S, axis, M, N, K, db, dtype, capfd):
    print(f"[128x128] axis={axis} M={M} N={N} K={K} db={db} {dtype}", file=sys.stderr, flush=True)
    W, mask, X, sw, sx = gen.make_exact_int(41, M, M, N, K, gen.OUTPUT if axis == 0 else gen.INPUT, db, dtype)
    dev = lambda a: None if a is None else torch.from_numpy(a.view(np.int16) if a.dtype == np.uint16 else a).cuda()  # noqa: E731
    X, sw, sx = dev(X), dev(sw), dev(sx)
    pw = S.compress(dev(W), dev(mask), axis, db)
    pw = S.tile(pw) if dtype == gen.FP8 else pw
    ref = S.gemm(X, pw, sw, sx, out_f32=True, plan=S.plan_override(kernel=2, ksplit=1))
    prev = S.spense_set_log(1)
    capfd.readouterr()
    try:
        y = S.gemm(X, pw, sw, sx, out_f32=True)
        torch.cuda.synchronize()
    finally:
        S.spense_set_log(prev)
    log = capfd.readouterr().err.strip().splitlines()[-1]
    if (axis, M, N, K, db, dtype) in CASES256:
        assert "large-M 256x256" in log, log
    else:
        assert "large-M 128x128" in log, log
    assert torch.equal(y, ref)
    for pad in (8, 3):  # whole-row stores, scalar stores; the padding is untouched
        big = torch.full((M, N + pad), 7.0, dtype=torch.bfloat16, device="cuda")
        S.gemm(X, pw, sw, sx, out=big[:, :N])
        torch.cuda.synchronize()
        assert torch.equal(big[:, :N], ref.bfloat16()), pad
        assert torch.all(big[:, N:] == 7.0)


@pytest.mark.parametrize("axis,M,N,K,db", [CASES[0][:5], CASES[7][:5]])
def test_planned_tiles_repeatable(S, axis, M, N, K, db):
    """Random data: the same bits every time, and within the fp32 sums' reordering (K
    slices) of the row-split kernel: both are within 2^-12 of sum |x w| (the fp8
    instructions' ~13 fraction bits), checked on the norm."""
    g = torch.Generator(device="cuda").manual_seed(5)
    draw = lambda *s: (torch.randn(s, generator=g, device="cuda") * 8).to(torch.float8_e4m3fn).view(torch.uint8)  # noqa: E731
    W, X = draw(N, K), draw(M, K)
    mask = torch.from_numpy(gen.random_mask_24(np.random.default_rng(3), N, K, gen.OUTPUT if axis == 0 else gen.INPUT, db)).cuda()
    pw = S.tile(S.compress(W, mask, axis, db))
    ref = S.gemm(X, pw, out_f32=True, plan=S.plan_override(kernel=2, ksplit=1))
    first = S.gemm(X, pw, out_f32=True)
    for _ in range(5):
        assert torch.equal(S.gemm(X, pw, out_f32=True), first)
    assert (first - ref).norm() <= 2.0 ** -12 * ref.norm()


@pytest.mark.parametrize("M", [16, 64, 100])
def test_row_split_slices_off_quads(S, M):
    """The row-split kernels' partial sums where the dense region starts off multiples of 4."""
    N, K, db = 1024, 5120, 766
    print(f"[slices off quads] M={M}", file=sys.stderr, flush=True)
    W, mask, X, sw, sx = gen.make_exact_int(43, M, M, N, K, gen.OUTPUT, db, gen.FP8)
    W, mask, X, sw, sx = (torch.from_numpy(a).cuda() for a in (W, mask, X, sw, sx))
    pw = S.tile(S.compress(W, mask, 0, db))
    assert S.spense_gemm_workspace_size(M, pw.desc) > 0
    assert torch.equal(S.gemm(X, pw, sw, sx), S.gemm(X, pw, sw, sx, plan=S.plan_override(kernel=2, ksplit=1)))
