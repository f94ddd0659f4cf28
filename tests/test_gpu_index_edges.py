"""Index selection and gathers at the edges of their variants' ranges, exact against numpy."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def S():
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_2606_10445_amd as S
    return S


@pytest.mark.parametrize("I", [1, 15, 1023, 1025, 10240, 10241, 15360, 15361, 16384, 24576, 24577, 25601, 32768, 32769])
def test_permutation_edges(S, I):
    """TopK with ties, NaN, infinities and signed zeros; ties keep the lower index, NaN last."""
    print(f"[perm] I={I}", flush=True)
    r = np.random.default_rng(I)
    t = np.round(r.standard_normal(I) * 8).astype(np.float32) / 8
    t[r.random(I) < 0.05] = np.nan
    t[r.random(I) < 0.05] = -0.0
    if I > 4:
        t[1], t[2] = np.inf, -np.inf
    key = np.where(np.isnan(t), -np.inf, t + 0.0)
    order = np.lexsort((np.arange(I), -key, np.isnan(t)))  # numbers before NaN, larger first, lower index first
    for n in sorted({0, 1, I // 4, I // 2, I - 1, I}):
        flags, perm = S.dense_permutation(torch.from_numpy(t).cuda(), n)
        want = np.zeros(I, np.uint8)
        want[order[:n]] = 1
        idx = np.arange(I, dtype=np.int32)
        assert np.array_equal(flags.cpu().numpy(), want), n
        assert np.array_equal(perm.cpu().numpy(), np.concatenate([idx[want == 0], idx[want == 1]])), n


@pytest.mark.parametrize("dtype", [torch.uint8, torch.bfloat16, torch.float32])
@pytest.mark.parametrize("rows,cols", [(1, 1), (3, 4097), (517, 1024), (130, 4099), (2049, 7), (2100, 67), (5000, 260)])
def test_gather_cols_edges(S, dtype, rows, cols):
    """Odd widths, rows that are not 4-byte aligned, a strided destination whose padding stays."""
    g = torch.Generator(device="cuda").manual_seed(cols)
    src = torch.randint(0, 200, (rows, cols), generator=g, device="cuda").to(dtype)
    perm = torch.randperm(cols, generator=g, device="cuda").to(torch.int32)
    want = src[:, perm.long()]
    assert torch.equal(S.gather_cols(src, perm), want)
    big = torch.full((rows, cols + 3), 7, device="cuda").to(dtype)
    S.gather_cols(src, perm, out=big[:, 1:cols + 1])
    assert torch.equal(big[:, 1:cols + 1], want) and (big[:, 0] == 7).all() and (big[:, cols + 1:] == 7).all()


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("I,D", [(5, 8), (130, 2056), (1028, 5120), (700, 8192)])
def test_scores_edges(S, dtype, I, D):
    """Each count of row pieces a score kernel is built for; sums of positive fp32 terms are
    within max(I, D) u of fp64."""
    g = torch.Generator(device="cuda").manual_seed(I)
    wg, wu, wd = (torch.randn(s, generator=g, device="cuda").to(dtype) for s in ((I, D), (I, D), (D, I)))
    hi, hm = torch.rand(D, generator=g, device="cuda"), torch.rand(I, generator=g, device="cuda")
    sc = S.index_scores(wg, wu, wd, hi, hm)
    tol = 2.0 ** -24 * (max(I, D) + 8)
    for name, ref in (("gate", wg.double().abs() @ hi.double().sqrt() / D), ("up", wu.double().abs() @ hi.double().sqrt() / D),
                      ("down", wd.double().abs().mean(0) * hm.double().sqrt())):
        assert ((sc[name].double() - ref).abs() <= tol * ref).all(), name
