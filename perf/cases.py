"""The work a user of libdconv has it do, as measurable cases.

A case is one call of the public entry points: ``single`` (one input map, M
filters) or ``multi`` (C input maps, M filters of C channels each), fp32, with
the layouts and value distributions of ``dconv_workloads.py``.  The sizes are
those of the paper's layers (maps of 7 to 1K pixels, 64 to 512 channels, 32 to
512 filters), of the 4096 x 4096 single map, and odd ones between them.  The
library has one direction (forward) and one data type (fp32).
"""
import math

import torch

import paper_2212_00404_amd as dc


def _case(name, op, C, M, Wx, Wy, K):
    return {"name": name, "op": op, "C": C, "M": M, "Wx": Wx, "Wy": Wy, "K": K}


def listed():
    return [
        # The smallest call: one small map, one small filter; launch and host
        # time are all of it.
        _case("single_64_m1_k3", "single", 1, 1, 64, 64, 3),
        # First layers on small maps with many filters (the paper's
        # single-channel layers, its smallest map).
        _case("single_28_m512_k3", "single", 1, 512, 28, 28, 3),
        # A map of odd width and height (no row starts on a 16-byte boundary),
        # a few filters: a filter bank over an image cut to an arbitrary size.
        _case("single_1021x1003_m8_k5", "single", 1, 8, 1021, 1003, 5),
        # The paper's largest single-channel layer: writes 32 output maps.
        _case("single_1024_m32_k3", "single", 1, 32, 1024, 1024, 3),
        # Whole-image filtering on a large map: a small filter (bound by
        # memory), a middle one and the largest (most arithmetic).
        _case("single_4096_m1_k3", "single", 1, 1, 4096, 4096, 3),
        _case("single_4096_m1_k7", "single", 1, 1, 4096, 4096, 7),
        _case("single_4096_m1_k11", "single", 1, 1, 4096, 4096, 11),
        # CNN layers, late in a network: many channels and a tiny map.
        _case("multi_c512_9_m512_k3", "multi", 512, 512, 9, 9, 3),
        # A 1 x 1 layer (a matrix product with few columns).
        _case("multi_c512_14_m512_k1", "multi", 512, 512, 14, 14, 1),
        # The middle of a network.
        _case("multi_c256_30_m256_k3", "multi", 256, 256, 30, 30, 3),
        # Odd everything: channels, filters and map off every tile size.
        _case("multi_c93_61x45_m131_k5", "multi", 93, 131, 61, 45, 5),
        # Early in a network: few channels, a large map; the most work.
        _case("multi_c64_512_m64_k3", "multi", 64, 64, 512, 512, 3),
    ]


def _out(case):
    return case["Wy"] - case["K"] + 1, case["Wx"] - case["K"] + 1


def work(case):
    """Each input, filter and output value moved once (4 bytes); one multiply
    and one add per term of the convolution sum."""
    C, M, K = case["C"], case["M"], case["K"]
    H, W = _out(case)
    return {"bytes": 4 * (C * case["Wx"] * case["Wy"] + M * C * K * K + M * H * W),
            "flops": 2 * C * M * K * K * H * W}


# No drawn case costs more than the listed ones: the arithmetic of the largest
# multi-channel layer, the output of the many-filter and 4096-wide maps.
_MAX_FLOPS = 2 * 64 * 64 * 9 * 510 * 510
_MAX_OUT = 32 * 1022 * 1022


def _logint(rng, lo, hi):
    return max(lo, min(hi, round(math.exp(rng.uniform(math.log(lo), math.log(hi + 0.5))))))


def draw(rng):
    while True:
        op = rng.choice(["single", "multi"])
        if op == "single":
            C, M = 1, _logint(rng, 1, 512)
            K = rng.randint(1, 11)
            Wx, Wy = _logint(rng, 28, 4096), _logint(rng, 28, 4096)
            if rng.random() < 0.5:      # half of the maps are rows of whole 16 bytes
                Wx = max(28, Wx // 4 * 4)
        else:
            C, M = _logint(rng, 32, 512), _logint(rng, 32, 512)
            K = rng.choice([1, 1, 2, 3, 3, 3, 4, 5, 5, 6, 7, 9, 11])
            Wx = max(K, _logint(rng, 7, 512))
            Wy = max(K, _logint(rng, 7, 512)) if rng.random() < 0.5 else Wx
        case = {"op": op, "C": C, "M": M, "Wx": Wx, "Wy": Wy, "K": K}
        H, W = _out(case)
        if work(case)["flops"] <= _MAX_FLOPS and M * H * W <= _MAX_OUT:
            return case


def prepare(case, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)

    def rand(*shape):
        return torch.rand(shape, generator=g, device="cuda")

    C, M, Wx, Wy, K = (case[k] for k in ("C", "M", "Wx", "Wy", "K"))
    if case["op"] == "single":
        # image and filter values uniform in [-1, 1)
        return {"op": "single", "I": rand(Wy, Wx) * 2 - 1, "F": rand(M, K, K) * 2 - 1}
    # activations after a ReLU, He-initialised weights
    F = torch.randn((M, C, K, K), generator=g, device="cuda") * math.sqrt(2.0 / (C * K * K))
    return {"op": "multi", "I": rand(C, Wy, Wx), "F": F}


def run(state):
    if state["op"] == "single":
        return dc.single(state["I"], state["F"])
    return dc.multi(state["I"], state["F"])


def exact(case, seed):
    """The convolution sum in 64 bits, one filter tap at a time."""
    st = prepare(case, seed)
    I, F = st["I"].double(), st["F"].double()
    if case["op"] == "single":
        I, F = I[None], F[:, None]
    M, C, K = F.shape[0], F.shape[1], F.shape[2]
    H, W = _out(case)
    O = torch.zeros((M, H * W), dtype=torch.float64, device="cuda")
    for r in range(K):
        for s in range(K):
            window = I[:, r:r + H, s:s + W].reshape(C, H * W)
            tap = F[:, :, r, s].contiguous()
            if C == 1:
                O.addcmul_(tap, window)
            else:
                O.add_(tap @ window)
    return O.reshape(M, H, W)


def tolerance(case):
    """fp32 products added in fp32 in any order: about four times the error the
    library showed against 64 bits over these ranges (a random walk of
    roundings, 4e-8 + 1e-8 * sqrt(terms))."""
    rel = 4 * (4e-8 + 1e-8 * math.sqrt(case["C"] * case["K"] ** 2))
    return {"rel": rel, "max": 8 * rel}
