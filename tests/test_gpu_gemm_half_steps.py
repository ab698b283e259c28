"""Outlier ranges of one to four 32-byte units beside K loops of every short length, on the 128-byte-stage tiles: the range may end in the
middle of a 64-byte MFMA step, be the whole K, and the loop may be shorter than the LDS ring."""
import numpy as np
import pytest
import torch

import oracle
from tests.gpu_util import bf16_bits, dev

q = pytest.importorskip("paper_2605_21072_amd")
pytestmark = pytest.mark.gpu


def _pack(a, K, K_o):
    n_off, kp = q.packed_normal_offset(K_o), q.packed_k(K, K_o)
    out = np.zeros((a.shape[0], kp), np.int8)
    out[:, :K_o] = a[:, :K_o]
    out[:, n_off:n_off + K - K_o] = a[:, K_o:]
    return out


@pytest.mark.parametrize("M,N", [(17, 24), (145, 280), (300, 272)])     # a few rows of a tile; ragged tiles of every size
@pytest.mark.parametrize("K,K_o", [(128, 0), (128, 32), (128, 64), (128, 96), (128, 128), (200, 90), (256, 32), (384, 96), (512, 33), (640, 128), (900, 1)])
def test_every_tile(M, N, K, K_o):
    rng = np.random.default_rng(M + N + K + K_o)
    Xq, Wq = (rng.integers(-127, 128, (r, K)).astype(np.int8) for r in (M, N))
    sx, sn, so = (rng.uniform(0.001, 0.1, n).astype(np.float32) for n in (M, N, N))
    b = rng.standard_normal(N).astype(np.float32)
    ref = oracle.dual_gemm(Xq, sx, Wq, sn, so, b, K_o)
    w = q.DualScaleWeight(dev(_pack(Wq, K, K_o)), dev(sn), dev(so), None, K_o, N, K)
    Xd, sxd, bd = dev(_pack(Xq, K, K_o)), dev(sx), dev(b)
    ran = 0
    for v in range(1, q.gemm_num_variants() + 1):
        if "128-byte stages" not in q.gemm_variant_name(v) or ("single" in q.gemm_variant_name(v) and K_o):
            continue
        Yf, an, ao = q.w8a8_dual_gemm(Xd, sxd, w, bd, M, torch.float32, debug_acc=True, variant=v)
        assert np.array_equal(an.cpu().numpy(), ref["acc_n"]) and np.array_equal(ao.cpu().numpy(), ref["acc_o"]), q.gemm_variant_name(v)
        # the epilogue is defined operation by operation: bit-equal, in the builds without the accumulator dump too
        assert np.array_equal(Yf.cpu().numpy(), ref["Y_f32"])
        assert np.array_equal(q.w8a8_dual_gemm(Xd, sxd, w, bd, M, torch.float32, variant=v).cpu().numpy(), ref["Y_f32"])
        assert np.array_equal(bf16_bits(q.w8a8_dual_gemm(Xd, sxd, w, bd, M, torch.bfloat16, variant=v)), ref["Y_bf16"])
        ran += 1
    assert ran >= 7


@pytest.mark.parametrize("M,N,K,K_o", [(1, 8, 100, 0), (65, 136, 640, 128), (129, 392, 1280, 96), (520, 1536, 8960, 32), (1560, 1536, 2048, 64), (2300, 2312, 200, 33)])
def test_aligned_tiles_against_the_general_one(M, N, K, K_o):
    """Every aligned 128-byte-stage tile on longer loops and on more tiles than workgroups, against the general tile (pinned to the oracle)."""
    gen = torch.Generator(device="cuda").manual_seed(M + N)
    Xq, Wq = (torch.randint(-127, 128, (r, q.packed_k(K, K_o)), generator=gen, device="cuda", dtype=torch.int8) for r in (M, N))
    sx, sn, so, b = (torch.rand(n, generator=gen, device="cuda") * 0.1 for n in (M, N, N, N))
    w = q.DualScaleWeight(Wq, sn, so, None, K_o, N, K)
    names = {v: q.gemm_variant_name(v) for v in range(1, q.gemm_num_variants() + 1)}
    general = [v for v in names if "any width" in names[v]]
    tiles = [v for v in names if "128-byte stages" in names[v] and ("dual" if K_o else "single") in names[v]]
    assert len(general) == 3 and len(tiles) == 6
    for dt in (torch.float32, torch.bfloat16):
        want = q.w8a8_dual_gemm(Xq, sx, w, b, M, dt, variant=general[0])
        for v in general[1:] + tiles:
            assert torch.equal(q.w8a8_dual_gemm(Xq, sx, w, b, M, dt, variant=v), want), names[v]


@pytest.mark.parametrize("dt,M,N", [(torch.bfloat16, 2709, 8008), (torch.float32, 1420, 7688), (torch.bfloat16, 2709, 8000)])
@pytest.mark.parametrize("K,K_o,bits", [(256, 0, 8), (384, 33, 8), (300, 130, 8), (384, 33, 4)])
def test_large_outputs_with_rows_inside_a_sector(dt, M, N, K, K_o, bits):
    """Outputs of more than 40 MB: rows that begin inside a 64-byte sector (8008 bf16 and 7688 fp32 columns, padded and shifted views) leave through
    plain stores, whole ones (8000 bf16) through write-through ones.  Every tile against the register-staged kernel, nothing outside."""
    gen = torch.Generator(device="cuda").manual_seed(K + N)
    kp = q.packed_k(K, K_o)
    Xq = torch.randint(-127, 128, (M, kp), generator=gen, device="cuda", dtype=torch.int8)
    Wq = torch.randint(-128, 128, (N, kp * bits // 8), generator=gen, device="cuda", dtype=torch.int8).clamp_(min=-127 if bits == 8 else -128)
    sx, sn, so, b = (torch.rand(n, generator=gen, device="cuda") * 0.1 for n in (M, N, N, N))
    w = q.DualScaleWeight(Wq if bits == 8 else Wq.view(torch.uint8), sn, so, None, K_o, N, K, bits=bits)
    want = q.w8a8_dual_gemm(Xq, sx, w, b, M, dt, variant=2 if bits == 8 else 3)
    if bits == 8:
        names = {v: q.gemm_variant_name(v) for v in range(1, q.gemm_num_variants() + 1)}
        tiles = [v for v in names if "128-byte stages" in names[v] and ("single" not in names[v] or not K_o)]
    else:
        tiles = range(4, q.load_library().qarvd_w4_gemm_num_variants() + 1)
    ran = 0
    for v in (0, *tiles):
        for pad, shift in ((0, 0), (16, 8)):
            big = torch.full((M + 1, N + pad), 7.0, dtype=dt, device="cuda")
            Y = big[:M, shift:shift + N]
            try:
                q.w8a8_dual_gemm(Xq, sx, w, b, M, Y=Y, variant=v)
            except q.QarvdError as e:
                assert e.status == -2 and K_o > 128
                continue
            assert torch.equal(Y, want), (v, pad)
            assert (big[M] == 7).all() and (big[:, :shift] == 7).all() and (big[:, shift + N:] == 7).all(), (v, pad)
            ran += 1
    assert ran >= 4
