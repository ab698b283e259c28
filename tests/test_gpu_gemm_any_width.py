"""The general 128-byte-stage tiles (any outlier width, any N, any output alignment) and the rule that sends calls to them."""
import numpy as np
import pytest
import torch

import oracle
from tests.gpu_util import bf16_bits, dev

q = pytest.importorskip("paper_2605_21072_amd")
pytestmark = pytest.mark.gpu


def _named(part):
    return [v for v in range(1, q.gemm_num_variants() + 1) if part in q.gemm_variant_name(v)]


def _pack(a, K, K_o):
    n_off, kp = q.packed_normal_offset(K_o), q.packed_k(K, K_o)
    out = np.zeros((a.shape[0], kp), np.int8)
    out[:, :K_o] = a[:, :K_o]
    out[:, n_off:n_off + K - K_o] = a[:, K_o:]
    return out


# one element; tails of one column beside whole tiles; an outlier range that ends inside, at the end of and past the
# first stage, in the last stage and with the whole K; fewer K tiles than LDS stages; more tiles than workgroups; two shapes for which
# the cost model takes the 64x128 tile, odd columns and an outlier range beyond the first stage among them
@pytest.mark.parametrize("which", ["heuristic", "128x128", "64x128", "64x64"])
@pytest.mark.parametrize("M,N,K,K_o", [(1, 1, 1, 0), (1, 3, 1, 1), (16, 7, 77, 77), (65, 129, 130, 1), (127, 255, 640, 161), (128, 128, 512, 512),
                                       (129, 257, 700, 96), (64, 65, 1003, 128), (300, 1003, 1000, 129), (40, 64, 2048, 1900), (2300, 2305, 200, 33),
                                       (300, 3331, 200, 33), (600, 1603, 250, 140)])
def test_any_width(which, M, N, K, K_o):
    variant = 0 if which == "heuristic" else [v for v in _named("any width") if which in q.gemm_variant_name(v)][0]
    rng = np.random.default_rng(M * 7 + N * 5 + K * 3 + K_o)
    Xq = rng.integers(-127, 128, (M, K)).astype(np.int8)
    Wq = rng.integers(-127, 128, (N, K)).astype(np.int8)
    sx, sn, so = (rng.uniform(0.001, 0.1, n).astype(np.float32) for n in (M, N, N))
    b = rng.standard_normal(N).astype(np.float32)
    ref = oracle.dual_gemm(Xq, sx, Wq, sn, so, b, K_o)
    w = q.DualScaleWeight(dev(_pack(Wq, K, K_o)), dev(sn), dev(so), None, K_o, N, K)
    Xd, sxd, bd = dev(_pack(Xq, K, K_o)), dev(sx), dev(b)
    for dt in (torch.float32, torch.bfloat16):
        for pad, shift in ((0, 0), (3, 1), (8, 8)):      # row stride and first element off the 16-byte grid, and on it
            big = torch.full((M * (N + pad) + shift + 16,), -5.0, dtype=dt, device="cuda")
            Y = big[shift:shift + M * (N + pad)].view(M, N + pad)[:, :N]
            q.w8a8_dual_gemm(Xd, sxd, w, bd, M, Y=Y, variant=variant)
            # the arithmetic is defined operation by operation: bit-equal
            if dt == torch.float32:
                assert np.array_equal(Y.cpu().numpy(), ref["Y_f32"])
            else:
                assert np.array_equal(bf16_bits(Y.contiguous()), ref["Y_bf16"])
            Y.fill_(-5.0)
            assert bool((big == -5.0).all()), "bytes outside the output were written"
        Yd, an, ao = q.w8a8_dual_gemm(Xd, sxd, w, bd, M, dt, debug_acc=True, variant=variant)
        assert np.array_equal(an.cpu().numpy(), ref["acc_n"]) and np.array_equal(ao.cpu().numpy(), ref["acc_o"])


@pytest.mark.parametrize("M,N,K,K_o", [(1, 8, 100, 0), (65, 72, 640, 128), (129, 136, 1280, 96), (200, 392, 384, 0), (520, 1536, 8960, 32), (1560, 1536, 2048, 64)])
def test_small_tiles_on_whole_lines(M, N, K, K_o):
    """The aligned 128x128, 64x128 and 64x64 tiles against the general ones (which the oracle checks above)."""
    gen = torch.Generator(device="cuda").manual_seed(M + N)
    Xq = torch.randint(-127, 128, (M, q.packed_k(K, K_o)), generator=gen, device="cuda", dtype=torch.int8)
    Wq = torch.randint(-127, 128, (N, q.packed_k(K, K_o)), generator=gen, device="cuda", dtype=torch.int8)
    sx, sn, so, b = (torch.rand(n, generator=gen, device="cuda") * 0.1 for n in (M, N, N, N))
    w = q.DualScaleWeight(Wq, sn, so, None, K_o, N, K)
    kind = "dual" if K_o else "single"
    tiles = [[v for v in _named("128-byte stages %s " % size) if kind in q.gemm_variant_name(v)] for size in ("128x128", "64x128", "64x64")]
    assert [len(t) for t in tiles] == [1, 1, 1]
    for dt in (torch.float32, torch.bfloat16):
        want = q.w8a8_dual_gemm(Xq, sx, w, b, M, dt, variant=_named("any width")[0])
        for v, in tiles:
            assert torch.equal(q.w8a8_dual_gemm(Xq, sx, w, b, M, dt, variant=v), want), q.gemm_variant_name(v)


@pytest.mark.parametrize("M,N,K,K_o", [(1, 1, 1, 0), (1, 8, 100, 32), (65, 129, 130, 1), (127, 255, 640, 161), (129, 264, 1280, 96), (300, 1003, 1000, 129),
                                       (520, 1536, 2048, 32), (40, 64, 2048, 1900), (4400, 4352, 256, 0)])
def test_packed_int4_tiles(M, N, K, K_o):
    """Every INT4 tile that takes a shape, and the heuristic, against the register-staged one (pinned to the oracle elsewhere)."""
    gen = torch.Generator(device="cuda").manual_seed(M + N + K)
    kp = q.packed_k(K, K_o)
    Xq = torch.randint(-127, 128, (M, kp), generator=gen, device="cuda", dtype=torch.int8)
    lo, hi = (torch.randint(-7, 8, (N, kp // 2), generator=gen, device="cuda") for _ in range(2))
    Wq4 = ((hi & 15) << 4 | (lo & 15)).to(torch.uint8)
    sx, sn, so, b = (torch.rand(n, generator=gen, device="cuda") * 0.1 for n in (M, N, N, N))
    w = q.DualScaleWeight(Wq4, sn, so, None, K_o, N, K, bits=4)
    for dt in (torch.float32, torch.bfloat16):
        want, an, ao = q.w8a8_dual_gemm(Xq, sx, w, b, M, dt, debug_acc=True, variant=3)
        for v in [0] + list(range(4, q.load_library().qarvd_w4_gemm_num_variants() + 1)):
            try:
                got = q.w8a8_dual_gemm(Xq, sx, w, b, M, dt, debug_acc=True, variant=v)
            except q.QarvdError as e:
                assert e.status == -2 and 4 <= v <= 6 and (N % 8 or q.packed_normal_offset(K_o) > 128)
                continue
            assert torch.equal(got[0], want) and torch.equal(got[1], an) and torch.equal(got[2], ao), v
            assert torch.equal(q.w8a8_dual_gemm(Xq, sx, w, b, M, dt, variant=v), want), v
