"""Activation quantization where its kernels change shape: channel counts on both sides of every row width, with and
without a permutation, pads inside the packed row, element-wise loads, permutations in no order, more rows than fit at once,
and rows whose scale the exact quotient does not cover.  Codes and scales against the oracle, bit for bit."""
import numpy as np
import pytest
import torch

import oracle

pytestmark = pytest.mark.gpu

q = pytest.importorskip("paper_2605_21072_amd")
from gpu_util import dev, logical  # noqa: E402


def make(M, K, seed, dtype):
    rng = np.random.default_rng(seed)
    X = rng.standard_normal((M, K), dtype=np.float32)
    X[:, rng.integers(0, K, 3)] *= np.float32(15)
    Xd = dev(X).to(dtype)
    return Xd.float().cpu().numpy(), Xd, rng


def check(X, Xd, perm, K_o):
    K = X.shape[1]
    pd = None if perm is None else dev(perm)
    ref, sx = oracle.quant_act(X, perm)
    Xq, s = q.quant_act(Xd, pd, K_o)
    assert np.array_equal(s.cpu().numpy().view(np.uint32), sx.view(np.uint32))
    assert np.array_equal(logical(Xq, K, K_o), ref)
    scale = np.float32(np.abs(X).max() * 0.4 / 127)                     # clips the largest values
    if scale > 0:
        got = q.quant_act_static(Xd, pd, K_o, float(scale))
        assert np.array_equal(logical(got, K, K_o), oracle.quant_act_static(X, scale, perm))


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("K", [1, 3, 4, 5, 130, 256, 257, 512, 513, 1024, 1025, 1532, 1536, 1537, 1540, 2048, 2049, 3072, 3073, 3076,
                               4096, 4097, 4100, 5120, 5121, 6144, 6148, 10240, 10244, 12288, 12290, 14336, 14339, 16384, 16388, 18400, 18432,
                               18433, 18436, 20480, 20481, 20484])
def test_row_widths(K, dtype):
    X, Xd, rng = make(9, K, K, dtype)
    check(X, Xd, None, 0)
    for K_o in sorted({min(K, 32), min(K, 7), min(K, K // 2)}):
        sel = np.sort(rng.choice(K, K_o, replace=False))
        perm = np.concatenate([sel, np.setdiff1d(np.arange(K), sel)]).astype(np.int32)
        check(X, Xd, perm, K_o)
    check(X, Xd, rng.permutation(K).astype(np.int32), min(K, 32))


@pytest.mark.parametrize("M,K", [(9001, 1536), (9001, 200), (3100, 2048), (1700, 8960)])
def test_more_rows_than_fit_at_once(M, K):
    X, Xd, rng = make(M, K, M + K, torch.float32)
    check(X, Xd, rng.permutation(K).astype(np.int32), 32)
    check(X, Xd, None, 0)


def test_unaligned_rows_and_odd_strides():
    X, _, rng = make(33, 1001, 5, torch.float32)
    big = torch.zeros((33, 1005), device="cuda")
    big[:, 3:1004] = dev(X)
    check(X, big[:, 3:1004], rng.permutation(1001).astype(np.int32), 31)


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("K", [4, 259, 1000, 1536, 2362, 8960, 13825])
def test_rows_and_permutations_at_any_address(K, dtype):
    """X one to three elements off its alignment, strides that move it from row to row, perm off its own."""
    X, Xd, rng = make(11, K, 3 * K, dtype)
    for K_o in sorted({0, min(K, 32), min(K, 37), K}):
        sel = np.sort(rng.choice(K, K_o, replace=False))
        perm = np.concatenate([sel, np.setdiff1d(np.arange(K), sel)]).astype(np.int32)
        ref, sx = oracle.quant_act(X, perm)
        for off, pad in ((0, 1), (1, 0), (2, 3), (3, 2)):
            big = torch.full((11, K + off + pad), 1e6, dtype=dtype, device="cuda")
            big[:, off:off + K] = Xd
            pd = torch.zeros(K + 4, dtype=torch.int32, device="cuda")[off:off + K]
            pd.copy_(dev(perm))
            Xq, s = q.quant_act(big[:, off:off + K], pd, K_o)
            assert np.array_equal(s.cpu().numpy().view(np.uint32), sx.view(np.uint32))
            assert np.array_equal(logical(Xq, K, K_o), ref)
            if K_o == 0:                       # (the permutation is the identity)
                assert torch.equal(q.quant_act(big[:, off:off + K], None, 0)[0][:, :K], Xq[:, :K])


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("K", [261, 1536, 8960])
def test_scales_outside_the_exact_quotients_range(K, dtype):
    """Rows of every magnitude a type holds, down to its denormals, and static scales that such a row has next to one of
    ordinary size; rows with infinities."""
    X, _, rng = make(18, K, 7, torch.float32)
    powers = np.array([1, 1e-29, 1e-30, 1e-33, 1e-36, 1e-38, 1e-40, 1e-42, 1e-44, 1e29, 1e31, 1e33, 1e36, 1, 1, 1, 1, 1])
    X = (X.astype(np.float64) * powers[:, None]).astype(np.float32)
    X[13] = 0
    X[14, ::2] *= np.float32(1e-36)
    X[15, ::2] *= np.float32(1e34)
    X[16, 5] = np.inf
    X[17, 7], X[17, 9] = -np.inf, 1e-40
    Xd = dev(X).to(dtype)
    X = Xd.float().cpu().numpy()
    perm = rng.permutation(K).astype(np.int32)
    for p, K_o in ((perm, 64), (perm, 37), (None, 0)):
        pd = None if p is None else dev(p)
        with np.errstate(invalid="ignore"):
            ref, sx = oracle.quant_act(X, p)
        Xq, s = q.quant_act(Xd, pd, K_o)
        assert np.array_equal(s.cpu().numpy().view(np.uint32), sx.view(np.uint32))
        defined = np.isfinite(X if p is None else X[:, p])            # (an infinity over an infinite scale has no code)
        assert np.array_equal(logical(Xq, K, K_o)[defined], ref[defined])
        for scale in (np.float32(1e-45), np.float32(3e-39), np.float32(2e-31), np.float32(1e-30), np.float32(3e30), np.float32(3e38)):
            got = q.quant_act_static(Xd, pd, K_o, float(scale))
            assert np.array_equal(logical(got, K, K_o), oracle.quant_act_static(X, scale, p)), scale


@pytest.mark.parametrize("K,dtype", [(256, torch.float32), (1536, torch.bfloat16), (5120, torch.bfloat16), (8960, torch.float32), (16384, torch.float32)])
@pytest.mark.parametrize("K_o", [0, 32])
def test_inputs_larger_than_the_cache_rule_loads_plainly(K, dtype, K_o):
    """Inputs that are more than 265 MB together with their codes take kernels that load X with another cache hint; halves of them take the
    plain ones, which the tests above check against the oracle."""
    M = 240 * 2 ** 20 // (K * (4 if dtype == torch.float32 else 2)) + 3
    gen = torch.Generator(device="cuda").manual_seed(K + K_o)
    X = torch.randn((M, K), generator=gen, device="cuda").to(dtype)
    perm = torch.cat([p.sort().values for p in torch.randperm(K, generator=gen, device="cuda").split([K_o, K - K_o])]).int() if K_o else None
    Xq, s_x = q.quant_act(X, perm, K_o)
    static = q.quant_act_static(X, perm, K_o, 0.03)
    kp = q.packed_k(K, K_o)
    for rows in (slice(0, M // 2), slice(M // 2, M)):
        a, s = q.quant_act(X[rows], perm, K_o)
        assert torch.equal(a[:, :kp], Xq[rows, :kp]) and torch.equal(s, s_x[rows])
        assert torch.equal(q.quant_act_static(X[rows], perm, K_o, 0.03)[:, :kp], static[rows, :kp])
