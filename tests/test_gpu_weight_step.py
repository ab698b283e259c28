"""The offline weight step where its kernels change shape: channel counts on both sides of every register and
workgroup size, rows longer than the register kernels take, unaligned rows, norms and error sums whose parallel value
does not settle the ordered one, scales outside the exact quotient's range and rows of equal magnitudes.  Every output
against the oracle, bit for bit."""
import numpy as np
import pytest
import torch

import oracle
import workloads as wl

pytestmark = pytest.mark.gpu

q = pytest.importorskip("paper_2605_21072_amd")
from gpu_util import assert_weight_equal, dev, gpu_quantize_weight, weight_to_numpy  # noqa: E402


def check(W, **kw):
    o = oracle.quantize_weight(W, **kw)
    for bits in (8, 4):
        ref = o if bits == 8 else oracle.quantize_weight(W, bits=4, **kw)
        w = gpu_quantize_weight(W, bits=bits, **kw)
        got = dict(Wq=w.logical_Wq().cpu().numpy(), s_normal=w.s_normal.cpu().numpy(), s_outlier=w.s_outlier.cpu().numpy(),
                   perm=w.perm.cpu().numpy(), K_o=w.K_o, v=w.v.cpu().numpy())
        assert_weight_equal(got, ref)
        n_o, kp = w.n_off, w.kp
        c = w.codes().cpu().numpy()
        assert np.all(c[:, w.K_o:n_o] == 0) and np.all(c[:, n_o + w.K - w.K_o:kp] == 0)      # pads
    return o


@pytest.mark.parametrize("K", [1, 3, 255, 1536, 1537, 2560, 2561, 5120, 5121, 9216, 9217, 16384, 16385, 18400, 18432, 18433, 20001])
def test_channel_counts_at_the_kernels_edges(K):
    L = wl.small_random_case(5000 + K, 1, 21, K, min(K // 50, 40))
    check(L["W"])


@pytest.mark.parametrize("K,N", [(1536, 9001), (300, 70), (2048, 4500), (8960, 130)])
def test_clip_and_absmax_rows_over_several_rounds(K, N):
    L = wl.small_random_case(5100 + K, 1, N, K, 20)
    check(L["W"])
    check(L["W"][:200], clip_search=True)


@pytest.mark.parametrize("K", [513, 1280, 2049, 5121, 10241, 16384])
def test_clip_search_at_the_kernels_edges(K):
    L = wl.small_random_case(5200 + K, 1, 9, K, 12)
    check(L["W"], clip_search=True)


def test_rows_that_are_not_16_byte_aligned():
    L = wl.small_random_case(5300, 1, 37, 1001, 9)
    o = oracle.quantize_weight(L["W"])
    big = torch.zeros((37, 1003), device="cuda")
    big[:, 1:1002] = dev(L["W"])
    assert_weight_equal(weight_to_numpy(q.quantize_weight(big[:, 1:1002])), o)


def test_norm_half_way_between_two_floats():
    """1 + 2^-23 + 2^-48 = (1 + 2^-24)^2: the norm lies exactly between two floats, so no interval around the parallel sum
    settles it and the ordered sum decides; neighbours one bit to either side in other columns."""
    rows = np.zeros((700, 96), np.float32)
    rng = np.random.default_rng(1)
    for k in range(96):
        parts = [1.0, 2.0 ** -12, 2.0 ** -12, 2.0 ** -24] + ([2.0 ** -26] * (k % 5))
        rows[rng.choice(700, len(parts), replace=False), k] = parts
    check(rows)


def test_a_column_with_a_nan_has_a_nan_norm_and_leaves_the_others_alone():
    L = wl.small_random_case(5350, 1, 700, 1536, 9)
    v = oracle.quantize_weight(L["W"])["v"]
    W = L["W"].copy()
    cols = [0, 63, 64, 700, 1535]
    W[np.arange(5) * 99, cols] = np.nan
    for clip in (False, True):
        got = q.quantize_weight(dev(W), clip_search=clip).v.cpu().numpy()
        assert np.all(np.isnan(got[cols]))
        rest = np.setdiff1d(np.arange(1536), cols)
        assert np.array_equal(got[rest].view(np.uint32), v[rest].view(np.uint32))


@pytest.mark.parametrize("K", [1536, 8960, 12000])
@pytest.mark.parametrize("scale", [1e-38, 1e-34, 3e-31, 1e31, 1e35])
def test_scales_outside_the_exact_quotients_range(scale, K):
    L = wl.small_random_case(5400, 1, 40, K, 9)
    W = (L["W"].astype(np.float64) * scale).astype(np.float32)
    W[3] = L["W"][3]                                                     # one ordinary row among them
    check(W)
    check(W, clip_search=True)
    check(W, forced_mask=(np.arange(K) % 13 == 0).astype(np.uint8), clip_search=True)


@pytest.mark.parametrize("K", [700, 8960])
def test_clip_search_on_rows_of_equal_magnitudes(K):
    rng = np.random.default_rng(K)
    W = (rng.choice([-1.0, 1.0], (6, K)) * 0.25).astype(np.float32)
    W[1, ::3] *= np.float32(0.5)                                        # two magnitudes, hundreds of each
    W[2, 5] = 3.0
    W[3] = 0.0
    W[4, :K // 2] = 0.0
    check(W, clip_search=True)
    check(W, forced_mask=(np.arange(K) % 7 == 0).astype(np.uint8), clip_search=True)


def test_ties_among_the_fillers_take_the_smaller_indices():
    W = np.ones((5, 3000), np.float32)
    W[:, 1234] = 40.0
    o = check(W)
    assert o["K_o"] == 32 and list(o["perm"][:31]) == list(range(31))


@pytest.mark.parametrize("K", [2, 64, 65, 128, 1025, 1536, 2050, 8960, 16384])
@pytest.mark.parametrize("levels", [1, 2, 5, 40])
def test_detection_among_ties_and_infinite_norms(K, levels):
    """Norms of a few distinct values: equal norms around both medians and at the edge of the outlier block; then a few infinite ones."""
    rng = np.random.default_rng(K + levels)
    W = np.zeros((3, K), np.float32)
    W[0] = rng.choice(np.linspace(1.0, 1.5, levels), K)
    W[1, rng.choice(K, max(1, K // 40), replace=False)] = 30.0
    check(W)
    W[2, rng.choice(K, max(1, K // 60), replace=False)] = np.float32(3e38)      # the sum of squares is beyond a float's range
    W[1, W[2] > 0] = np.float32(3e38)
    check(W)


def _ulps(x, n):
    return (np.float32(x).view(np.uint32) + n).astype(np.uint32).view(np.float32)


@pytest.mark.parametrize("K", [257, 1536, 5120, 8960, 16384])
@pytest.mark.parametrize("kind", ["dead", "levels", "equal and a few near", "equal and many near", "two equal", "all"])
def test_detection_where_many_norms_are_equal(K, kind):
    """More equal norms than the sort counts through: alone in their bin, among a few neighbours within bits of them, among so many that
    the searches take over; as many as the sort still counts through, at the medians and at the edge of the outlier block.  A column with one
    nonzero weight has that weight for its norm."""
    rng = np.random.default_rng(K)
    v = rng.lognormal(0.0, 0.02, K).astype(np.float32)
    idx = rng.permutation(K)
    half = idx[:K // 2]
    if kind == "dead":
        v[half] = 0.0
    elif kind == "levels":
        v = rng.choice(np.linspace(0.5, 1.5, max(2, K // 20)).astype(np.float32), K)
    elif kind == "equal and a few near":
        v[half] = 1.0
        v[half[:12]] = _ulps(1.0, rng.integers(-6, 7, 12))
    elif kind == "equal and many near":
        v[half] = _ulps(1.0, rng.integers(-20, 21, half.size))
    elif kind == "two equal":
        v[half[::2]], v[half[1::2]] = 1.0, 2.0
        v[half[:5]], v[half[5:9]] = _ulps(1.0, np.arange(1, 6)), _ulps(2.0, -np.arange(1, 5))
    else:
        v[:] = 0.25
    for outliers in (0, 40):                      # 40: the block of 64 ends among the others
        o = v.copy()
        o[idx[-outliers:] if outliers else []] = 30.0
        W = np.zeros((3, K), np.float32)
        W[rng.integers(0, 3, K), np.arange(K)] = o
        check(W)
