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
