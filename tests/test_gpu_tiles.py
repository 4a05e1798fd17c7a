"""The tiled kernels at the edges of their tiles, against the fp64 oracle.

The forward works on 32-key x 32-query tiles in workgroups of 128 ("wide") or 32
queries here (64: see the launch shapes' own test), the backward on 128-key blocks whose query range may be split and on
64-key chunks for dQ; T takes the values on both sides of each. Dyadic q and k
make every score exact, so that codes, extrema and tie counts are compared bit
for bit; the rest keeps the bounds of the parity tests (fp32: 1e-4 for O, 1e-3
for the gradients; bf16 operands: 2e-2), which the error of an fp32 product as
six bf16 ones, at most 2^-24 a term, lies well below.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

import paper_2609_33591_amd as kia  # noqa: E402
from paper_2609_33591_amd.inputs import make_inputs  # noqa: E402
import test_gpu_bf16 as B16  # noqa: E402
import test_gpu_parity as P  # noqa: E402

EDGES = (1, 31, 32, 33, 63, 64, 65, 127, 128, 129, 257)
VARIANTS = (("minmax", "lerp", "weight"), ("resolved", "nearest", "prob"),
            ("fwm", "nearest", "weight"))


@pytest.mark.parametrize("policy", ("auto", "wide", "split"))
@pytest.mark.parametrize("d", (16, 32, 64, 128))
@pytest.mark.parametrize("dtype", ("f32", "bf16"))
def test_tile_edges(oracle_mod, dtype, d, policy):
    kia.kia_set_grid_policy(policy)
    try:
        for i, T in enumerate(EDGES):
            calib, recon, ste = VARIANTS[i % 3]
            causal = 0 if i % 4 == 3 else 1
            tag = f"{dtype} {policy} T{T} d{d} {calib} {recon} {ste} causal{causal}"
            P.flush("case " + tag)
            x = make_inputs(1, 2, T, d, seed=700 + i, dyadic=True)
            sl = [(0, 0), (0, 1)]
            args = (5, calib, 8.0, recon, ste, False, causal)
            if dtype == "bf16":
                xb, x = B16.bf16_inputs(*x)
                g = B16.run_gpu16(*xb, *args)
                r = P.run_oracle(oracle_mod, *x, *args)
                B16.compare16(g, r, oracle_mod, calib, sl, tag=tag)
            else:
                g = P.run_gpu(*x, *args)
                r = P.run_oracle(oracle_mod, *x, *args)
                P.compare(g, r, oracle_mod, calib, sl, tag=tag)
    finally:
        kia.kia_set_grid_policy("auto")


@pytest.mark.parametrize("d", (16, 32, 64, 128))
def test_tiny_query_rows(d):
    """Query rows whose elements lie near fp32's smallest normal value keep the
    scores' full precision: q 2^-n against k 2^n gives the same products, and so
    the same result, bit for bit, as the rows as they were (every factor a power
    of two; MinMax, so that nothing but the scores sees q and k). q has full
    24-bit significands: as three bf16 pieces, whose last one would lie below
    bf16's smallest value, it would lose bits (checked here)."""
    P.flush(f"case tiny rows d{d}")
    q, k, v, _ = make_inputs(1, 1, 97, d, seed=31)
    q, k = (torch.where(x.abs() < 2.0 ** -5, torch.full_like(x, 2.0 ** -5), x) for x in (q, k))
    args = (4, "minmax", 8.0, "lerp", "weight", False, 1)
    ref, _ = kia.forward(q.cuda(), k.cuda(), v.cuda(), *args)
    for n in (110, 120):  # the smallest elements: 2^-115, 2^-125
        x = q * 2.0 ** -n
        assert torch.equal(x * 2.0 ** n, q)
        left = x.double()
        for _ in range(3):
            left = left - left.to(torch.bfloat16).double()
        assert (left != 0).any()
        o, _ = kia.forward(x.cuda(), (k * 2.0 ** n).cuda(), v.cuda(), *args)
        torch.cuda.synchronize()
        assert np.array_equal(o.cpu().numpy(), ref.cpu().numpy()), n


@pytest.mark.parametrize("d", (16, 64))
def test_tiny_element_beside_large_scores(d):
    """One element of 2^-115 in rows of ordinary size, against keys of 2^70:
    it is below half a unit of every score, so the result is the one without
    it, and finite."""
    P.flush(f"case tiny element d{d}")
    q, k, v, _ = make_inputs(1, 1, 97, d, seed=32, dyadic=True)
    k = k * 2.0 ** 70
    args = (4, "fwm", 8.0, "lerp", "weight", False, 1)
    q[..., 3] = 0.0
    ref, _ = kia.forward(q.cuda(), k.cuda(), v.cuda(), *args)
    q[..., 3] = 2.0 ** -115
    o, _ = kia.forward(q.cuda(), k.cuda(), v.cuda(), *args)
    torch.cuda.synchronize()
    assert np.isfinite(ref.cpu().numpy()).all()
    assert np.array_equal(o.cpu().numpy(), ref.cpu().numpy())
