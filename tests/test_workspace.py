"""Scratch of the calls that cut K into slices: who owns it, and for how long."""
import threading
import types

import numpy as np
import pytest
import torch

import gen


@pytest.fixture(scope="module")
def S():
    import paper_2606_10445_amd as S
    return S


def test_overlapping_calls_hold_their_own_scratch(S, monkeypatch):
    """Without a workspace, a call's scratch is its own while the call runs, whatever the
    stream or thread of the other call (the launches replaced, a call run inside a call)."""
    M, N, K = 256, 5120, 8192  # bf16, K slices
    L = S.spense_layout(N, K, S.SPENSE_BF16, S.SPENSE_SPLIT_INPUT, 6144)
    desc = S.spense_packed_t(S.SPENSE_BF16, S.SPENSE_SPLIT_INPUT, N, K, 6144, 4096, L.values_ld, 8192, L.meta_ld, 16384,
                             L.dense_ld, S.SPENSE_LAYOUT_ROWMAJOR)
    need = S.spense_gemm_workspace_size(M, desc)
    assert need > 0
    pw = types.SimpleNamespace(dtype=S.SPENSE_BF16, N=N, K=K, desc=desc)
    X = torch.empty((M, K), dtype=torch.bfloat16)
    held = []

    def launch(*args):
        held.append((args[9], args[9] + args[10]))
        if len(held) == 1:
            S.gemm(X, pw)
        elif len(held) == 2:
            t = threading.Thread(target=S.gemm, args=(X, pw))
            t.start()
            t.join()
        return S.SPENSE_OK

    monkeypatch.setattr(S, "spense_gemm", launch)
    monkeypatch.setattr(S, "_stream", lambda device: 0)
    S.gemm(X, pw)
    assert len(held) == 3 and all(b - a >= need for a, b in held)
    held.sort()
    assert all(held[i][1] <= held[i + 1][0] for i in range(2))


def _weight(S, g, dtype, N, K, axis, db):
    if dtype == "bf16":
        W = torch.randn((N, K), generator=g, device="cuda").bfloat16()
    else:
        W = torch.randn((N, K), generator=g, device="cuda").to(torch.float8_e4m3fn).view(torch.uint8)
    mask = torch.ones((N, K), dtype=torch.uint8, device="cuda")
    part = mask[:db] if axis == 0 else mask[:, :db]
    part.view(part.shape[0], -1, 4)[:, :, ::2] = 0
    pw = S.compress(W, mask, axis, db)
    return pw if dtype == "bf16" else S.tile(pw)


def _x(g, dtype, M, K):
    x = torch.randn((M, K), generator=g, device="cuda")
    return x.bfloat16() if dtype == "bf16" else x.to(torch.float8_e4m3fn).view(torch.uint8)


@pytest.mark.gpu
@pytest.mark.parametrize("dtype,M,N,K", [("bf16", 256, 5120, 8192), ("fp8", 200, 4096, 14336)])
def test_two_streams_without_a_workspace(S, dtype, M, N, K):
    """K-sliced calls on two streams, in flight together, give the serial results."""
    print(f"[two streams] {dtype} M={M} {N}x{K}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(1)
    pw = _weight(S, g, dtype, N, K, 1, K * 3 // 4)
    assert S.spense_gemm_workspace_size(M, pw.desc) > 0
    xs = [_x(g, dtype, M, K) for _ in range(2)]
    want = [S.gemm(x, pw, out_f32=True) for x in xs]
    torch.cuda.synchronize()
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    got = [[], []]
    for _ in range(6):
        for i, s in enumerate(streams):
            with torch.cuda.stream(s):
                got[i].append(S.gemm(xs[i], pw, out_f32=True))
    torch.cuda.synchronize()
    for i in range(2):
        assert all(torch.equal(y, want[i]) for y in got[i]), i


@pytest.mark.gpu
@pytest.mark.parametrize("own", [True, False])
def test_a_graph_keeps_its_scratch(S, own):
    """A graph of a K-sliced call, replayed after a larger call has grown the workspace and
    other tensors were made, touches none of them and repeats its result."""
    print(f"[graph scratch] workspace={own}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(2)
    M, N, K = 256, 5120, 8192
    pw = _weight(S, g, "bf16", N, K, 1, K * 3 // 4)
    x = _x(g, "bf16", M, K)
    ws = S.Workspace("cuda") if own else None
    need = S.spense_gemm_workspace_size(M, pw.desc)
    out = torch.empty((M, N), dtype=torch.float32, device="cuda")
    want = S.gemm(x, pw, out_f32=True, workspace=ws).clone()
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        S.gemm(x, pw, out=out, out_f32=True, workspace=ws)
    torch.cuda.current_stream().wait_stream(side)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        S.gemm(x, pw, out=out, out_f32=True, workspace=ws)
    if own:
        ws.get(4 * need)
    others = [torch.full((need,), 7, dtype=torch.uint8, device="cuda") for _ in range(3)]
    for _ in range(3):
        out.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, want)
        assert all(bool((t == 7).all()) for t in others)


@pytest.mark.gpu
@pytest.mark.parametrize("dtype,M,N,K", [("bf16", 256, 5120, 8192), ("fp8", 200, 4096, 14336)])
def test_c_call_without_a_workspace(S, dtype, M, N, K):
    """A call that is sliced only where it has the workspace: without one, the same values
    (whole numbers: any order of the sums) and every other result in place."""
    print(f"[no workspace] {dtype} M={M} {N}x{K}", flush=True)
    W, mask, X, sw, sx = gen.make_exact_int(51, 0, M, N, K, gen.INPUT, K * 3 // 4, gen.BF16 if dtype == "bf16" else gen.FP8)
    dev = lambda a: None if a is None else torch.from_numpy(a.view(np.int16) if a.dtype == np.uint16 else a).cuda()  # noqa: E731
    pw = S.compress(dev(W), dev(mask), 1, K * 3 // 4)
    pw = pw if dtype == "bf16" else S.tile(pw)
    X, sw, sx = dev(X), dev(sw), dev(sx)
    want = S.gemm(X, pw, sw, sx, out_f32=True)
    y = torch.full((M, N), 7.0, device="cuda")
    ptr = lambda t: None if t is None else t.data_ptr()  # noqa: E731
    rc = S.spense_gemm(X.data_ptr(), M, K, pw.desc, ptr(sw), ptr(sx), y.data_ptr(), N, S.SPENSE_OUT_F32, None, 0,
                       torch.cuda.current_stream().cuda_stream)
    assert rc == S.SPENSE_OK
    torch.cuda.synchronize()
    assert torch.equal(y, want)
