"""The native marshalling of the online calls against the Python one, which calls with an explicit stream take: same results, same
buffers handed back, same errors."""
import pytest
import torch

q = pytest.importorskip("paper_2605_21072_amd")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,K,N,c,bits,dtype", [(1, 256, 8, 0, 8, torch.float32), (33, 512, 264, 7, 8, torch.bfloat16), (50, 512, 272, 7, 8, torch.bfloat16), (70, 1001, 130, 40, 4, torch.float32)])
def test_same_results_and_buffers(M, K, N, c, bits, dtype):
    gen = torch.Generator(device="cuda").manual_seed(M + K)
    W = torch.randn((N, K), generator=gen, device="cuda") * 0.02
    W[:, :c] *= 30
    X = torch.randn((M, K), generator=gen, device="cuda").to(dtype)
    w = q.quantize_weight(W, bits=bits)
    perm = w.perm if w.K_o else None
    kp = q.packed_k(K, w.K_o)
    for bias in (None, torch.randn(N, generator=gen, device="cuda")):
        for out in (torch.bfloat16, torch.float32):
            got = []
            for st in (None, torch.cuda.current_stream()):
                Xq, s_x = q.quant_act(X, perm, w.K_o, stream=st)
                static = q.quant_act_static(X, perm, w.K_o, 0.02, stream=st)
                Y = torch.empty((M, N), dtype=out, device="cuda")
                assert q.w8a8_dual_gemm(Xq, s_x, w, bias, M, Y=Y, stream=st) is Y
                given = q.quant_act(X, perm, w.K_o, Xq=Xq, s_x=s_x, stream=st)
                assert given[0] is Xq and given[1] is s_x and q.quant_act_static(X, perm, w.K_o, 0.02, Xq=static, stream=st) is static
                got.append([Xq[:, :kp], s_x, static[:, :kp], Y, q.w8a8_dual_gemm(Xq, s_x, w, bias, M, out, stream=st), q.w8a8_linear(X, w, bias, out, stream=st)])
                if bits == 8 and N % 16 == 0:
                    Y8 = torch.full((M, N + 16), 7, dtype=torch.int8, device="cuda")
                    assert q.w8a8_dual_gemm_q8(Xq, s_x, w, bias, M, 0.05, Y8=Y8, stream=st) is Y8
                    got[-1] += [Y8, q.w8a8_dual_gemm_q8(Xq, s_x, w, bias, M, 0.05, q.ACT_GELU_TANH, stream=st)]
            assert len(got[0]) == (8 if N == 272 else 6)
            for a, b in zip(*got):
                assert a.dtype == b.dtype and a.shape == b.shape and a.stride() == b.stride() and torch.equal(a, b)


def test_same_errors():
    W = torch.randn((16, 128), device="cuda")
    w = q.quantize_weight(W)
    X = torch.randn((4, 128), device="cuda")
    Xq, s_x = q.quant_act(X, None, 0)
    for st in (None, torch.cuda.current_stream()):
        for bad, error in ((X.half(), TypeError), (X.t(), ValueError), (X[0], ValueError), (X.cpu(), ValueError), (X[:, :64], ValueError)):
            with pytest.raises(error):
                q.w8a8_linear(bad, w, None, stream=st)
        with pytest.raises(TypeError, match="expected float32 or bfloat16, got torch.float16"):
            q.quant_act(X.half(), None, 0, stream=st)
        with pytest.raises(TypeError):
            q.w8a8_linear(X, w, None, torch.float16, stream=st)
        for y in (q.w8a8_linear(X, w, None, None, stream=st), q.w8a8_dual_gemm(Xq, s_x, w, None, 4, None, stream=st)):
            assert y.dtype == torch.get_default_dtype() == torch.float32
        Y = torch.empty((4, 16), dtype=torch.bfloat16, device="cuda")
        assert q.w8a8_dual_gemm(Xq, s_x, w, None, 4, None, Y=Y, stream=st) is Y
        with pytest.raises(q.QarvdError):
            q.w8a8_dual_gemm(Xq, None, w, None, 4, stream=st)
        for scale in (None, "0.03"):
            with pytest.raises(TypeError):
                q.quant_act_static(X, None, 0, scale, stream=st)
        for call in (lambda: q.w8a8_linear(X[:0], w, None, stream=st), lambda: q.quant_act(X, None, 32, stream=st),
                     lambda: q.quant_act_static(X, None, 0, -1.0, stream=st), lambda: q.w8a8_dual_gemm(Xq, s_x, w, None, 4, variant=999, stream=st),
                     lambda: q.w8a8_dual_gemm_q8(Xq, s_x, w, None, 4, 0.0, stream=st)):
            with pytest.raises(q.QarvdError):
                call()
