"""fp32 inputs over fp32's whole range: values that three bf16 pieces do not hold
(below 2^-100, from 2^126 up, infinite) keep every bit, as any fp32 product would.

A power of two on v, dO, q or k moves the results by the same power, so a call is
compared with the same one in ordinary size. Both sides are fp32 sums of at most T
(O, dV, dQ, dK) or d terms: their errors are below T 2^-24 of the result's norm
each, and 2 T 2^-24 = 1.2e-5 is the bound. Results down to 2^-126 2^-24 stay
within it although they are rounded as denormals.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

import paper_2609_33591_amd as kia  # noqa: E402

T = 97
TOL = 2 * T * 2.0 ** -24
OPS = (("fwm", "nearest", "prob"), ("minmax", "lerp", "weight"), ("fwm", "softmax", "weight"))
# powers of two on q, k, v, dO
SCALES = {"v": (0, 0, -122, 0), "dO": (0, 0, 0, -122), "k": (122, -122, 0, 0),
          "q": (-122, 122, 0, 0), "dS": (0, 0, -60, -60), "large": (0, 0, 118, -110)}


def inputs(d, seed):
    g = torch.Generator().manual_seed(seed)
    return [torch.randn(2, 3, T, d, generator=g).clamp(-1.99, 1.99) for _ in range(4)]


def call(q, k, v, dO, op, causal=1):
    x = [a.cuda() for a in (q, k, v, dO)]
    args = (4, op[0], 8.0, op[1], op[2], False, causal)
    o, st = kia.forward(*x[:3], *args)
    g = kia.backward(*x[:3], o, x[3], st, *args)
    torch.cuda.synchronize()
    return dict(zip(("o", "dq", "dk", "dv"), (a.cpu().double() for a in (o, *g))))


@pytest.mark.parametrize("policy", ("auto", "wide", "split"))
@pytest.mark.parametrize("which", tuple(SCALES))
@pytest.mark.parametrize("d", (16, 32, 64, 128))
def test_powers_of_two(d, which, policy):
    a, b, c, e = SCALES[which]
    kia.kia_set_grid_policy(policy)
    try:
        for op in OPS:
            print(f"case range d{d} {which} {policy} {op}", flush=True)
            q, k, v, dO = inputs(d, 40 + d)
            ref = call(q, k, v, dO, op)
            got = call(q * 2.0 ** a, k * 2.0 ** b, v * 2.0 ** c, dO * 2.0 ** e, op)
            # scores keep their size; dS moves with v and dO
            power = {"o": c, "dv": e, "dq": c + e + b, "dk": c + e + a}
            for n, p in power.items():
                x, y = got[n], ref[n] * 2.0 ** p
                err = ((x - y).norm() / y.norm()).item()
                assert err <= TOL, (op, n, err)
    finally:
        kia.kia_set_grid_policy("auto")


@pytest.mark.parametrize("policy", ("auto", "wide"))
@pytest.mark.parametrize("which", ("v", "dO", "k"))
@pytest.mark.parametrize("d", (16, 32, 64, 128))
def test_values_below_the_smallest_piece(d, which, policy):
    """Operands that are denormal throughout, below half of bf16's smallest value: no
    piece holds any of them. They have six bits (exact at 2^-138 2^-3), results are
    sums of at most T terms rounded to fp32's smallest step: T 2^-149, and TOL of
    the result."""
    kia.kia_set_grid_policy(policy)
    try:
        for op in OPS:
            print(f"case denormal d{d} {which} {policy} {op}", flush=True)
            q, k, v, dO = ((x * 8).round() / 8 for x in inputs(d, 70 + d))
            if which == "k":  # scores of 2^-18: q 2^120, k 2^-138
                dO = dO * 2.0 ** 10
                ref = call(q * 2.0 ** -18, k, v, dO, op)
                got = call(q * 2.0 ** 120, k * 2.0 ** -138, v, dO, op)
                names = ("dq",)
            else:
                ref = call(q, k, v, dO, op)
                got = call(q, k, *((v * 2.0 ** -138, dO) if which == "v" else
                                   (v, dO * 2.0 ** -138)), op)
                names = ("o", "dq", "dk") if which == "v" else ("dv", "dq", "dk")
            for n in names:
                y = ref[n] * 2.0 ** -138
                err = (got[n] - y).abs().max().item()
                assert y.abs().max().item() > 3 * T * 2.0 ** -149
                assert err <= T * 2.0 ** -149 + TOL * y.abs().max().item(), (op, n, err)
    finally:
        kia.kia_set_grid_policy("auto")


@pytest.mark.parametrize("d", (16, 64, 128))
def test_one_tiny_row_of_dO(d):
    """A row of dO far below the others keeps its own row of dQ to fp32 rounding."""
    for op in OPS:
        print(f"case tiny row d{d} {op}", flush=True)
        q, k, v, dO = inputs(d, 80 + d)
        ref = call(q, k, v, dO, op)
        dO[:, :, 60] *= 2.0 ** -115
        got = call(q, k, v, dO, op)
        y = ref["dq"][:, :, 60] * 2.0 ** -115
        assert ((got["dq"][:, :, 60] - y).norm() / y.norm()).item() <= TOL, op


@pytest.mark.parametrize("d", (16, 64, 128))
def test_one_value_that_rounds_to_infinity_in_bf16(d):
    """A finite v above bf16's largest value takes part as what it is."""
    print(f"case near the largest d{d}", flush=True)
    q, k, v, dO = inputs(d, 50 + d)
    v[:, :, 40, 5] = 3.4e38 * 2.0 ** -115
    op = ("minmax", "lerp", "weight")
    ref, got = call(q, k, v, dO, op), call(q, k, v * 2.0 ** 115, dO * 2.0 ** -115, op)
    for n, p in (("o", 115), ("dv", -115), ("dq", 0), ("dk", 0)):
        y = ref[n] * 2.0 ** p
        assert ((got[n] - y).norm() / y.norm()).item() <= TOL, n


@pytest.mark.parametrize("value", (float("inf"), float("nan")))
@pytest.mark.parametrize("d", (16, 64, 128))
def test_non_finite_values_stay_in_their_column(d, value):
    """An infinite or NaN element of v reaches its own column of O, one of dO its
    own column of dV, and no other."""
    print(f"case non-finite d{d} {value}", flush=True)
    for op in OPS:
        q, k, v, dO = inputs(d, 60 + d)
        ref = call(q, k, v, dO, op)
        v2, dO2 = v.clone(), dO.clone()
        v2[:, :, 33, 6] = value
        dO2[:, :, 50, 9] = value
        o = call(q, k, v2, dO, op)["o"]
        dv = call(q, k, v, dO2, op)["dv"]
        others = [c for c in range(d) if c != 6]
        assert np.isfinite(o[..., others].numpy()).all(), op
        assert ((o - ref["o"])[..., others].norm() / ref["o"].norm()).item() <= TOL, op
        assert not np.isfinite(o[:, :, 33, 6].numpy()).any(), op
        others = [c for c in range(d) if c != 9]
        assert np.isfinite(dv[..., others].numpy()).all(), op
        assert ((dv - ref["dv"])[..., others].norm() / ref["dv"].norm()).item() <= TOL, op
        assert not np.isfinite(dv[:, :, 0, 9].numpy()).any(), op
