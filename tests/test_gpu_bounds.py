"""Weights stay between the ends of their interval, and pairs that take no part
(masked keys, the FWM tail) add nothing whatever their values."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

import paper_2609_33591_amd as kia  # noqa: E402
from paper_2609_33591_amd.inputs import given_score_inputs  # noqa: E402


@pytest.mark.parametrize("d", (16, 64))
def test_lerp_weights_are_never_negative(d):
    """Scores far from zero for their span (5e5, span 24): the fast position of
    an extremum errs by up to 0.006, more than e^-h = e^-6 of the step above it.
    v is the identity, so O is the probabilities."""
    print(f"case weight bounds d{d}", flush=True)
    T, rng = d, np.random.default_rng(d)
    S = (500000.0 + rng.integers(0, 48, size=(T, 1)) + 24 * rng.random((T, T))).astype(np.float32)
    lo = rng.integers(0, T, size=T)
    S[np.arange(T), lo] = S.min(1) - 1
    S[np.arange(T), (lo + 1) % T] = S[np.arange(T), lo] + np.float32(24.5)
    q, k = given_score_inputs(S, d)
    v = torch.eye(d)[None, None, :T].contiguous()
    for calib in ("minmax", "fwm"):
        o, _ = kia.forward(q.cuda(), k.cuda(), v.cuda(), 4, calib, 25.0, "lerp", "weight", False, 0)
        torch.cuda.synchronize()
        p = o[0, 0].cpu().numpy()
        assert (p >= 0).all() and (p[np.arange(T), lo] < 1e-9).all(), calib


@pytest.mark.parametrize("op", (("fwm", "nearest", "prob"), ("fwm", "lerp", "weight"),
                                ("minmax", "lerp", "weight"), ("resolved", "nearest", "prob"),
                                ("fwm", "softmax", "weight")))
@pytest.mark.parametrize("dtype", (torch.float32, torch.bfloat16))
@pytest.mark.parametrize("d", (16, 64, 128))
def test_pairs_without_part_add_nothing(d, dtype, op):
    """A key that no earlier query sees (causal) and, under FWM, one in the tail of
    every later query's window: dO.v overflows for them, and no gradient is
    touched. Everything else has the size it has without them."""
    if dtype == torch.bfloat16 and op[1] == "softmax":
        pytest.skip("fp32 inputs only")
    print(f"case no part d{d} {dtype} {op}", flush=True)
    T, j = 40, 20
    g = torch.Generator().manual_seed(d)
    q, k, v, dO = (torch.randn(1, 2, T, d, generator=g) for _ in range(4))
    if op[0] == "fwm" and op[1] != "softmax":
        q[..., j:, 0] = 8.0 * d ** 0.5   # key j lies 16 below the others' scores
        k[..., j, 0] = -2.0
    else:
        dO[..., j:, :] = 0.0             # key j's own queries have no gradient
    big = v.clone()
    big[..., j, :] = 2.0 ** 100
    dO[..., :j, :] *= 2.0 ** 40          # g = 2^140 d for queries before j
    if op[0] == "fwm" and op[1] != "softmax":
        dO[..., j:, :] *= 2.0 ** 40
    out = []
    for val in (v, big):
        x = [a.to(dtype).cuda() for a in (q, k, val, dO)]
        args = (4, op[0], 8.0, op[1], op[2], "detach", 1)
        o, st = kia.forward(*x[:3], *args)
        gr = kia.backward(*x[:3], o, x[3], st, *args)
        torch.cuda.synchronize()
        out.append([t.float().cpu() for t in gr])
    rows = torch.arange(T) != j
    for a, b, n in zip(out[0], out[1], ("dq", "dk", "dv")):
        # key j's own row sees itself: only the queries before it are compared
        sel = slice(0, j) if n == "dq" else rows
        assert torch.isfinite(b[..., sel, :]).all(), n
        err = (a - b)[..., sel, :].norm() / a[..., sel, :].norm()
        assert err < 1e-5, (n, err)
