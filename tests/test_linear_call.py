"""qarvd_linear, the online pair in one call: argument checks (no GPU needed) and equality with the two calls it stands for."""
import pytest
import torch

import workloads as wl

q = pytest.importorskip("paper_2605_21072_amd")

OK, INVALID, UNSUPPORTED, WORKSPACE = 0, -1, -2, -3


def test_workspace_query_and_argument_checks():
    lib = q.load_library()
    M, K, N = 7, 1000, 64
    for K_o in (0, 7, 32, 1000):
        ld = q.packed_ld(K, K_o)
        assert lib.qarvd_linear_workspace(M, K, K_o) == M * ld + 4 * M and ld % 128 == 0
    assert lib.qarvd_linear_workspace(0, K, 0) == 0 and lib.qarvd_linear_workspace(M, K, K + 1) == 0
    assert lib.qarvd_linear_workspace(M, K, -1) == 0
    need = lib.qarvd_linear_workspace(M, K, 32)

    def call(M=M, bits=8, ws=0x1000, ws_bytes=need, xdt=0):      # addresses that are never reached
        return lib.qarvd_linear(0x1000, xdt, K, 0x1000, bits, 0x1000, 1152, 0x1000, 0x1000, None, M, N, K, 32, 0x1000, 1, N, ws,
                                ws_bytes, None)

    assert call(M=0) == INVALID and call(bits=5) == INVALID
    assert call(ws=None) == WORKSPACE and call(ws_bytes=need - 1) == WORKSPACE and call(ws=0x1010) == WORKSPACE
    assert call(xdt=7) == UNSUPPORTED


def bad_gemm_arguments(bits, kp, N):
    """(changed arguments, status) of calls whose activation half is in order and whose GEMM half is not."""
    row = kp * bits // 8
    for name in ("Wq", "s_n", "s_o", "Y"):
        yield {name: None}, INVALID
    yield dict(N=0), INVALID
    yield dict(ldwq=row - 16), INVALID
    yield dict(ldy=N - 1), INVALID
    yield dict(ldwq=row + 8), UNSUPPORTED
    yield dict(ydt=9), UNSUPPORTED
    yield dict(off_Wq=8), UNSUPPORTED
    yield dict(off_Y=1), UNSUPPORTED
    for name in ("off_s_n", "off_s_o", "off_bias"):
        yield {name: 2}, UNSUPPORTED


def call_linear(lib, bits, M, N, K, K_o, kp, ws, ws_bytes, at, kw={}):
    """qarvd_linear on the addresses `at`; kw: addresses that are None or moved by off_... bytes, other sizes."""
    a = {k: None if k in kw and kw[k] is None else at[k] + kw.get("off_" + k, 0) for k in ("Wq", "s_n", "s_o", "bias", "Y")}
    return lib.qarvd_linear(at["X"], 0, K, at["perm"], bits, a["Wq"], kw.get("ldwq", kp * bits // 8), a["s_n"], a["s_o"], a["bias"], M,
                            kw.get("N", N), K, K_o, a["Y"], kw.get("ydt", 1), kw.get("ldy", N), ws, ws_bytes, at.get("stream"))


@pytest.mark.parametrize("bits", [8, 4])
def test_nothing_is_launched_before_both_halves_are_checked(bits):
    """A GEMM argument that is refused is refused before the activation is quantized.  Where there is no GPU a launch
    would fail and answer with its own status; where there is one the next test looks at the workspace."""
    if torch.cuda.is_available():
        pytest.skip("addresses that are never reached: run where nothing can be launched")
    lib = q.load_library()
    M, N, K, K_o = 7, 64, 1000, 32
    kp = q.packed_k(K, K_o)
    need = lib.qarvd_linear_workspace(M, K, K_o)
    at = {k: 0x1000 for k in ("X", "perm", "Wq", "s_n", "s_o", "bias", "Y")}
    for kw, status in bad_gemm_arguments(bits, kp, N):
        assert call_linear(lib, bits, M, N, K, K_o, kp, 0x1000, need, at, kw) == status, kw


@pytest.mark.gpu
@pytest.mark.parametrize("bits", [8, 4])
def test_refused_calls_leave_the_workspace_alone(bits):
    lib = q.load_library()
    M, N, K, K_o = 7, 64, 1000, 32
    kp = q.packed_k(K, K_o)
    need = lib.qarvd_linear_workspace(M, K, K_o)
    X = torch.randn(M, K, device="cuda")
    perm = torch.arange(K, dtype=torch.int32, device="cuda")
    Wq = torch.zeros(N * kp * bits // 8 + 64, dtype=torch.uint8, device="cuda")
    s = torch.ones(N + 4, device="cuda")
    Y = torch.zeros(M * N + 8, dtype=torch.bfloat16, device="cuda")
    ws = torch.full((need,), 0x5A, dtype=torch.uint8, device="cuda")
    at = dict(X=X.data_ptr(), perm=perm.data_ptr(), Wq=Wq.data_ptr(), s_n=s.data_ptr(), s_o=s.data_ptr(), bias=s.data_ptr(),
              Y=Y.data_ptr(), stream=torch.cuda.current_stream().cuda_stream)
    for kw, status in bad_gemm_arguments(bits, kp, N):
        assert call_linear(lib, bits, M, N, K, K_o, kp, ws.data_ptr(), need, at, kw) == status, kw
    torch.cuda.synchronize()
    assert bool((ws == 0x5A).all())
    assert call_linear(lib, bits, M, N, K, K_o, kp, ws.data_ptr(), need, at) == OK
    torch.cuda.synchronize()
    assert not bool((ws == 0x5A).all())


@pytest.mark.gpu
@pytest.mark.parametrize("bits", [8, 4])
@pytest.mark.parametrize("M,N,K,c", [(33, 72, 256, 5), (200, 256, 1000, 0), (5, 40, 130, 3), (300, 1536, 1536, 8)])
def test_equals_the_pair(bits, M, N, K, c):
    L = wl.small_random_case(M + N + K, M, N, K, c)
    W, X, b = (torch.from_numpy(L[k]).cuda() for k in ("W", "X", "bias"))
    w = q.quantize_weight(W, bits=bits)
    assert (w.K_o > 0) == (c > 0)
    for Xd in (X, X.to(torch.bfloat16), torch.nn.functional.pad(X, (4, 4))[:, 4:-4]):
        Xq, s_x = q.quant_act(Xd, w.perm if w.K_o else None, w.K_o)
        for bias in (b, None):
            for dt in (torch.bfloat16, torch.float32):
                assert torch.equal(q.w8a8_linear(Xd, w, bias, dt), q.w8a8_dual_gemm(Xq, s_x, w, bias, M, dt))
    with pytest.raises(ValueError):
        q.w8a8_linear(X[:, :K - 1], w, b)
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        Y = q.w8a8_linear(X, w, b)
    stream.synchronize()
    assert torch.equal(Y, q.w8a8_linear(X, w, b))


@pytest.mark.gpu
@pytest.mark.parametrize("M,K,N,c,dtype", [(7500, 5120, 5120, 20, torch.float32), (4700, 8960, 256, 0, torch.float32), (25000, 1536, 4608, 9, torch.float32),
                                           (15100, 5120, 1536, 0, torch.bfloat16)])
def test_large_inputs_by_either_loads(M, K, N, c, dtype):
    """X of more than 144 MB: how it is loaded depends on what the call moves in all, so the linear and quant_act by itself may differ in that;
    the results do not."""
    gen = torch.Generator(device="cuda").manual_seed(M)
    W = torch.randn((N, K), generator=gen, device="cuda") * 0.02
    W[:, :c] *= 30
    w = q.quantize_weight(W)
    X = torch.randn((M, K), generator=gen, device="cuda").to(dtype)
    b = torch.randn(N, generator=gen, device="cuda")
    Xq, s_x = q.quant_act(X, w.perm if w.K_o else None, w.K_o)
    assert torch.equal(q.w8a8_linear(X, w, b), q.w8a8_dual_gemm(Xq, s_x, w, b, M))
