"""GPU: the kernels that split fp32 values into three bf16 parts, at the sizes
where they can go wrong: strips of 128 (K <= 9) or 64 columns, patch rows of 2
or 4, maps narrower than a strip, windows that run past the end of the map,
several filters per workgroup, and values at the ends of the fp32 range.

Bars: integers exact; |O - O64| <= 1e-6 * sum|I*F| on random floats (each
product is rounded to about 2^-24 and the sums of up to 169 terms add less
than 16 roundings of 2^-24 each), and never further from the oracle than the
fp32 vector kernel by more than a tenth.
"""
import numpy as np
import pytest
import torch

import paper_2212_00404_amd as dc
from dconv_workloads import random_arrays
from gpu_util import (assert_exact, assert_within, gpu_single, oracle_multi,
                      oracle_single)

pytestmark = pytest.mark.gpu

# (Wx, Wy, K, M); rows of 4n + 1 .. 3 floats take the kernel at K = 5 and 6 too
SINGLE = [(k, k, k, 1) for k in range(10, 14)] + [
    (131, 9, 5, 1), (133, 40, 5, 7), (129, 30, 6, 3), (134, 134, 7, 2), (135, 70, 8, 5), (1024, 600, 8, 6),
    (137, 22, 9, 1), (136, 70, 9, 2), (73, 13, 10, 1), (74, 77, 11, 3), (75, 50, 12, 2),
    (77, 51, 13, 4), (301, 211, 11, 1), (1025, 33, 7, 9), (515, 600, 9, 40), (64, 1000, 10, 3),
    (41, 39, 9, 600), (2050, 67, 13, 1)]


@pytest.mark.parametrize("shape", SINGLE, ids=[str(s) for s in SINGLE])
def test_single_split_edges(shape):
    Wx, Wy, K, M = shape
    assert dc.plan_single(Wx, Wy, K, M)["kernel"] == 3
    I, F = random_arrays(1, M, Wx, Wy, K, seed=sum(shape) * 31, variant="int")
    assert_exact(gpu_single(I[0], F[:, 0]), oracle_single(I[0], F[:, 0])[0], str(shape))
    I, F = random_arrays(1, M, Wx, Wy, K, seed=sum(shape) * 37)
    O64, A64 = oracle_single(I[0], F[:, 0])
    O = gpu_single(I[0], F[:, 0])
    assert_within(O, O64, A64, str(shape), rel=1e-6)
    V = gpu_single(I[0], F[:, 0], variant="valu")
    rms = [np.sqrt(np.mean((x.astype(np.float64) - O64) ** 2)) for x in (O, V)]
    # a handful of outputs says nothing about an average
    if O64.size > 1000:
        assert rms[0] <= 1.1 * rms[1], rms


# What surrounds the tensors in the tests of reads outside them: large, and
# finite, because a non-finite sum would be taken again from the right places
# (NaN around the tensors: test_gpu_poison.py, in a build that does not).
OUTSIDE = 1e20


def framed(x, offset=0):
    """x on the GPU, `offset` floats off a 16-byte boundary, OUTSIDE before and after it."""
    buf = torch.full((x.size + 2048,), OUTSIDE, device="cuda")
    lo = 1024 + offset
    buf[lo:lo + x.size] = torch.from_numpy(x).cuda().reshape(-1)
    return buf[lo:lo + x.size].view(x.shape)


@pytest.mark.parametrize("offset", [0, 1])
@pytest.mark.parametrize("K", [5, 7, 9, 10, 13])
def test_single_split_reads_stay_in_the_tensors(K, offset):
    """What lies before and after both tensors reaches no output."""
    Wx, Wy, M = 150 - K, 37 + K, 2
    I, F = random_arrays(1, M, Wx, Wy, K, seed=K)
    O = dc.single(framed(I[0], offset), framed(F[:, 0], offset))
    O64, A64 = oracle_single(I[0], F[:, 0])
    assert_within(O.cpu().numpy(), O64, A64, "K=%d" % K, rel=1e-6)


@pytest.mark.parametrize("K", [6, 9, 11])
def test_single_split_non_finite(K):
    """Infinities, NaN and overflowing sums come out where the fp32 vector
    kernel has them, and nowhere else."""
    Wx, Wy, M = 301, 45, 2
    I, F = random_arrays(1, M, Wx, Wy, K, seed=K + 100)
    I, F = I[0], F[:, 0]
    I[3, 7], I[20, 150], I[21, 299], I[44, 0] = np.inf, -np.inf, np.nan, 3.4e38
    F[1, K - 1, 0] = 0.0
    O, V = gpu_single(I, F), gpu_single(I, F, variant="valu")
    for kind in (np.isnan, np.isposinf, np.isneginf):
        assert np.array_equal(kind(O), kind(V)), kind
    ok = np.isfinite(V)
    O64, A64 = oracle_single(np.where(np.isfinite(I), I, 0).astype(np.float32), F)
    assert (np.abs(O[ok] - O64[ok]) <= 1e-6 * A64[ok]).all()


# Factors of the input and of the filters: normal values whose low bits lie
# below the smallest bf16, denormal ones, large ones (single products above
# 2^96), each against the other operand's, and sums that are denormal.
SCALES = [(1e-30, 1), (1e-37, 1), (1, 1e-37), (1e-38, 1e20), (1e20, 1e-38), (1e-42, 1e30),
          (1e30, 1e-42), (1e-20, 1e-20), (1e30, 1), (1, 1e36)]


def scaled(x, scale):
    return (x.astype(np.float64) * scale).astype(np.float32)


@pytest.mark.parametrize("scale", SCALES, ids=str)
@pytest.mark.parametrize("K", [6, 7, 11])
def test_single_split_scales(K, scale):
    """The bar of ordinary values at both ends of the fp32 range; a denormal
    sum rounds once to a multiple of 2^-149."""
    Wx, Wy, M = 203, 50, 1
    I, F = random_arrays(1, M, Wx, Wy, K, seed=K + 7)
    I, F = scaled(I[0], scale[0]), scaled(F[:, 0], scale[1])
    O64, A64 = oracle_single(I, F)
    err = np.abs(gpu_single(I, F).astype(np.float64) - O64)
    ok = A64 < 3e38
    assert ok.any() and (err <= 1e-6 * A64 + 2.0 ** -149)[ok].all()


# (C, M, Wx, Wy, K): channel counts around the stages of 8 to 128, filters
# around the tiles of 32 and 64, tiles cut by both edges, more than one round
# of stages, an odd number of channel-tap items (K = 3, 5, 7 with 8-channel
# stages)
MULTI = [(8, 32, 20, 20, 3), (16, 33, 35, 18, 3), (17, 64, 34, 10, 3), (33, 65, 19, 37, 3),
         (31, 31, 40, 21, 5), (9, 70, 37, 22, 5), (24, 40, 40, 30, 7), (15, 33, 20, 17, 7),
         (40, 96, 50, 20, 2), (7, 5, 36, 35, 4), (20, 36, 39, 38, 6), (130, 40, 33, 9, 1),
         (1, 64, 300, 17, 3), (100, 1, 66, 70, 3), (3, 2, 4, 4, 4)]


def split_plans(C, M, Wx, Wy, K):
    return [p for p in dc.plan_multi_candidates(C, M, Wx, Wy, K) if 16 <= p["kernel"] < 99]


@pytest.mark.parametrize("layer", MULTI, ids=[str(s) for s in MULTI])
def test_multi_split_every_plan(layer):
    """Integers exact in every shape; floats within 3e-6 * sum|I*F| (sums of up
    to 1000 terms, at most 100 roundings of 2^-24 each) and no further from
    the oracle than the fp32 kernels by more than a tenth."""
    C, M, Wx, Wy, K = layer
    plans = split_plans(*layer)
    assert plans
    I, F = random_arrays(C, M, Wx, Wy, K, seed=sum(layer) * 41, variant="int")
    It, Ft = torch.from_numpy(I).cuda(), torch.from_numpy(F).cuda()
    O64 = oracle_multi(I, F)[0]
    for p in plans:
        assert_exact(dc.multi(It, Ft, plan=p).cpu().numpy(), O64, "%r %r" % (layer, p))
    I, F = random_arrays(C, M, Wx, Wy, K, seed=sum(layer) * 43)
    It, Ft = torch.from_numpy(I).cuda(), torch.from_numpy(F).cuda()
    O64, A64 = oracle_multi(I, F)
    rms = lambda O: np.sqrt(np.mean((O.astype(np.float64) - O64) ** 2))
    base = rms(dc.multi(It, Ft, variant="mfma").cpu().numpy())
    for p in plans:
        O = dc.multi(It, Ft, plan=p).cpu().numpy()
        assert_within(O, O64, A64, "%r %r" % (layer, p), rel=3e-6)
        if O64.size > 1000:
            assert rms(O) <= 1.1 * base, (p, rms(O), base)


# filters that start 4, 8 and 12 bytes off a 16-byte boundary, where the copies
# of 16 bytes start anywhere too
@pytest.mark.parametrize("offset", range(4))
@pytest.mark.parametrize("layer", [(17, 33, 21, 19, 3), (9, 34, 23, 20, 5), (70, 5, 33, 9, 1),
                                   (32, 70, 20, 13, 2), (16, 65, 19, 16, 7)])
def test_multi_split_reads_stay_in_the_tensors(layer, offset):
    """What lies before and after both tensors reaches no output."""
    C, M, Wx, Wy, K = layer
    I, F = random_arrays(C, M, Wx, Wy, K, seed=sum(layer))
    It, Ft = framed(I, (offset + 1) % 4), framed(F, offset)
    O64, A64 = oracle_multi(I, F)
    for p in split_plans(*layer):
        assert_within(dc.multi(It, Ft, plan=p).cpu().numpy(), O64, A64, str(p), rel=3e-6)


def _microseconds(call):
    call()
    best = np.inf
    for _ in range(5):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        for _ in range(4):
            call()
        b.record()
        torch.cuda.synchronize()
        best = min(best, a.elapsed_time(b) / 4 * 1e3)
    return best


def test_non_finite_values_cost_little():
    """Sums that come out non-finite are taken again in parallel: a map that is
    all NaN, or a layer with one infinity, is within 15 times the time of a
    finite one (measured 4 to 6 and 3; a sum per lane and filter, one after
    the other, took 52 and 43 times)."""
    I, F = random_arrays(1, 1, 4096, 1024, 11, seed=3)
    It, Ft = torch.from_numpy(I[0]).cuda(), torch.from_numpy(F[:, 0]).cuda()
    nan = torch.full_like(It, float("nan"))
    assert _microseconds(lambda: dc.single(nan, Ft)) < 15 * _microseconds(lambda: dc.single(It, Ft))
    layer = (512, 512, 40, 40, 3)
    I, F = random_arrays(*layer, seed=4)
    It, Ft = torch.from_numpy(I).cuda(), torch.from_numpy(F).cuda()
    p = split_plans(*layer)[3]
    t = _microseconds(lambda: dc.multi(It, Ft, plan=p))
    It[100, 20, 20] = float("inf")
    assert _microseconds(lambda: dc.multi(It, Ft, plan=p)) < 15 * t


def test_multi_split_keeps_finite_sums():
    """An infinite filter value changes no bit of the other filters' maps, nor
    an infinite pixel of the outputs that it does not reach."""
    C, M, Wx, Wy, K = 20, 40, 37, 21, 3
    I, F = random_arrays(C, M, Wx, Wy, K, seed=78)
    It, Ft = torch.from_numpy(I).cuda(), torch.from_numpy(F).cuda()
    for p in split_plans(C, M, Wx, Wy, K):
        plain = dc.multi(It, Ft, plan=p)
        Fi, Ii = Ft.clone(), It.clone()
        Fi[7, 2, 1, 1], Ii[3, 5, 9] = float("inf"), float("inf")
        O = dc.multi(It, Fi, plan=p)
        keep = [m for m in range(M) if m != 7]
        assert torch.equal(O[keep], plain[keep]) and not torch.isfinite(O[7]).all(), p
        O = dc.multi(Ii, Ft, plan=p)
        hit = torch.zeros(O.shape[1:], dtype=torch.bool, device="cuda")
        hit[3:6, 7:10] = True
        assert torch.equal(O[:, ~hit], plain[:, ~hit]) and not torch.isfinite(O[:, hit]).any(), p


def test_multi_split_non_finite():
    C, M, Wx, Wy, K = 20, 40, 37, 21, 3
    I, F = random_arrays(C, M, Wx, Wy, K, seed=77)
    I[3, 5, 9], I[19, 20, 36], I[0, 0, 0] = np.inf, np.nan, 3.4e38
    F[7, 2, 1, 1], F[39, 19, 2, 2], F[11, 3] = -np.inf, 3e38, 0.0
    It, Ft = torch.from_numpy(I).cuda(), torch.from_numpy(F).cuda()
    V = dc.multi(It, Ft, variant="valu").cpu().numpy()
    for p in split_plans(C, M, Wx, Wy, K):
        O = dc.multi(It, Ft, plan=p).cpu().numpy()
        for kind in (np.isnan, np.isposinf, np.isneginf):
            assert np.array_equal(kind(O), kind(V)), (p, kind)
        ok = np.isfinite(V)
        assert np.allclose(O[ok], V[ok], rtol=1e-4, atol=1e-3)


@pytest.mark.parametrize("scale", SCALES, ids=str)
@pytest.mark.parametrize("layer", [(20, 40, 37, 21, 3), (9, 33, 23, 20, 5), (70, 5, 33, 9, 1)])
def test_multi_split_scales(layer, scale):
    """As test_single_split_scales, in every shape."""
    I, F = random_arrays(*layer, seed=sum(layer) + 5)
    I, F = scaled(I, scale[0]), scaled(F, scale[1])
    O64, A64 = oracle_multi(I, F)
    ok = A64 < 3e38
    assert ok.any()
    It, Ft = torch.from_numpy(I).cuda(), torch.from_numpy(F).cuda()
    for p in split_plans(*layer):
        err = np.abs(dc.multi(It, Ft, plan=p).cpu().numpy().astype(np.float64) - O64)
        assert (err <= 3e-6 * A64 + 2.0 ** -149)[ok].all(), p
