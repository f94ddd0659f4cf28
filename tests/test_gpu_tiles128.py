"""The 128 x 128 GEMM kernel (tiled fp8 between decode and the 256 x 256 grid, bf16 above 64
tokens) and the 256 x 256 one as the planner chooses them: bit for bit the row-split kernel's
results on exact-integer data (their sums are exact in any order), repeatable and within the
error bound on random data, infinities and NaN where the row-split kernel has them."""
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
# a K of fewer steps than the ring has stages
CASES += [(0, 1100, 27648, 128, 20736, gen.BF16)]
# bf16 on the 256 x 256 kernel: ragged rows and tokens, a boundary and K inside a step, all-2:4,
# all-dense, a row boundary off multiples of 16
CASES256 = [(0, 1030, 9000, 2080, 6001, gen.BF16), (1, 1300, 7003, 2112, 1056, gen.BF16),
            (1, 1100, 8200, 2080, 2080, gen.BF16), (0, 2049, 5000, 2048, 0, gen.BF16), (0, 1200, 9000, 2080, 6001, gen.BF16),
            (0, 2048, 27648, 128, 20736, gen.BF16), (0, 2048, 27648, 256, 20736, gen.BF16)]


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


# (axis, M, N, K, dense_begin, type, kernel, K slices): both types on either kernel, both regions,
# tiles of two, three and four token tiles a wave
RANDOM = [(0, 385, 5000, 2048, 3000, gen.FP8, "128x128", 1), (1, 250, 1100, 14336, 10016, gen.FP8, "128x128", 8),
          (0, 300, 8192, 4128, 6144, gen.BF16, "128x128", 1), (1, 200, 2600, 16416, 12320, gen.BF16, "128x128", 6),
          (0, 450, 20480, 1056, 15360, gen.FP8, "256x256", 1), (0, 300, 20480, 1056, 15360, gen.FP8, "256x256", 1),
          (1, 2040, 5632, 2080, 1536, gen.FP8, "256x256", 1), (0, 1030, 9000, 2080, 6001, gen.BF16, "256x256", 1),
          (1, 1200, 9000, 1056, 544, gen.BF16, "256x256", 1)]


def random_weight(S, g, axis, N, K, db, dtype):
    """Codes, the dense matrix in fp64 and the packed weight."""
    W = torch.randn((N, K), generator=g, device="cuda") * (8 if dtype == gen.FP8 else 1)
    W = W.to(torch.float8_e4m3fn) if dtype == gen.FP8 else W.bfloat16()
    mask = torch.from_numpy(gen.random_mask_24(np.random.default_rng(3), N, K, gen.OUTPUT if axis == 0 else gen.INPUT, db)).cuda()
    codes = W.view(torch.uint8) if dtype == gen.FP8 else W
    pw = S.compress(codes, mask, axis, db)
    return W.double() * mask, S.tile(pw) if dtype == gen.FP8 else pw


def logged(S, capfd, f):
    prev = S.spense_set_log(1)
    capfd.readouterr()
    try:
        y = f()
        torch.cuda.synchronize()
    finally:
        S.spense_set_log(prev)
    return y, capfd.readouterr().err.strip().splitlines()[-1]


@pytest.mark.parametrize("axis,M,N,K,db,dtype,kernel,slices", RANDOM)
def test_planned_tiles_repeatable_within_bound(S, axis, M, N, K, db, dtype, kernel, slices, capfd):
    """The same bits every time, and each element within the bound of its sum: (2^-12 of sum
    |x w| for the fp8 instructions' ~13 fraction bits) + 2 gamma_K.  A matrix-core result read
    before it is written shows up as run-to-run differences."""
    print(f"[random] axis={axis} M={M} N={N} K={K} db={db} {dtype}", file=sys.stderr, flush=True)
    g = torch.Generator(device="cuda").manual_seed(5)
    Wd, pw = random_weight(S, g, axis, N, K, db, dtype)
    X = torch.randn((M, K), generator=g, device="cuda") * (8 if dtype == gen.FP8 else 1)
    X = X.to(torch.float8_e4m3fn) if dtype == gen.FP8 else X.bfloat16()
    codes = X.view(torch.uint8) if dtype == gen.FP8 else X
    y, log = logged(S, capfd, lambda: S.gemm(codes, pw, out_f32=True))
    assert f"large-M {kernel} " in log and f"k_slices={slices} " in log, log
    for _ in range(4):
        assert torch.equal(S.gemm(codes, pw, out_f32=True), y)
    Xd, u = X.double(), 2.0 ** -24
    want, dot = Xd @ Wd.T, Xd.abs() @ Wd.abs().T
    gamma = K * u / (1 - K * u)
    bound = ((2.0 ** -12 if dtype == gen.FP8 else 0.0) + 2 * gamma) * dot + 4 * u * want.abs()
    assert bool(((y.double() - want).abs() <= bound).all())


@pytest.mark.parametrize("axis,M,N,K,db,dtype,kernel,slices", RANDOM)
def test_planned_tiles_nan_and_infinity(S, axis, M, N, K, db, dtype, kernel, slices, capfd):
    """Tokens with NaN (fp8 has no infinities) or infinities in the last columns of a region or of
    K give what the row-split kernel gives, and no other token changes."""
    print(f"[nan] axis={axis} M={M} N={N} K={K} db={db} {dtype}", file=sys.stderr, flush=True)
    W, mask, X, sw, sx = gen.make_exact_int(47, M, M, N, K, gen.OUTPUT if axis == 0 else gen.INPUT, db, dtype)
    dev = lambda a: None if a is None else torch.from_numpy(a.view(np.int16) if a.dtype == np.uint16 else a).cuda()  # noqa: E731
    pw = S.compress(dev(W), dev(mask), axis, db)
    pw = S.tile(pw) if dtype == gen.FP8 else pw
    clean, sw, sx = dev(X), dev(sw), dev(sx)
    edge = db if axis == 1 else K // 2
    cols = [0, edge - 1, min(edge, K - 1), K - 1]
    rows = [0, M // 2, M - 2, M - 1]
    X = clean.clone()
    for m, k in zip(rows, cols):
        X[m, k] = 0x7F if dtype == gen.FP8 else 0x7F80 if m % 2 else 0x7FC0
    y = S.gemm(X, pw, sw, sx, out_f32=True)
    ref = S.gemm(X, pw, sw, sx, out_f32=True, plan=S.plan_override(kernel=2, ksplit=1))
    assert torch.equal(y.isnan(), ref.isnan()) and torch.equal(y.nan_to_num(7.0), ref.nan_to_num(7.0))
    assert not bool(y[rows].isfinite().all())
    keep = torch.ones(M, dtype=torch.bool, device="cuda")
    keep[rows] = False
    assert torch.equal(y[keep], S.gemm(clean, pw, sw, sx, out_f32=True)[keep])


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
