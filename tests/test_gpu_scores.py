"""fp32 scores, bit for bit: the sum of q.k in one fixed order of fused
multiply-adds, d/2 steps of the terms s and d/2 + s, from zero.

An index decision jumps where a score's rounding does, so the order is part of
the operator's result (for N(0,1) inputs at T = 1024, d = 64 a sum of the same
products in another order puts about 1e-6 of the keys on another level, which
moves O by 1e-4 to 1e-3). The model is exact: 80-bit arithmetic holds the
product and the sum before the one rounding to fp32.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

import paper_2609_33591_amd as kia  # noqa: E402


def chain(q, k):
    """[T, T] scores of one slice's q, k [T, d] (float32) by the fixed order."""
    def fma(a, b, c):
        return (a[:, None].astype(np.longdouble) * b[None, :] + c).astype(np.float32)
    T, d = q.shape
    acc = np.zeros((T, T), np.float32)
    for s in range(d // 2):
        for e in (s, d // 2 + s):
            acc = fma(q[:, e], k[:, e], acc)
    return acc * np.float32(1.0 / np.sqrt(d))


def draws(d, T, kind):
    """q, k [1, 2, T, d] with full 24-bit significands. tiny_q: elements below
    fp32's normal range in all rows, tiny_k the same of the keys; mixed: query
    rows that hold both a tiny element and one of 2^50, against keys of 2^70."""
    g = torch.Generator().manual_seed(d + T)
    q, k = (torch.randn(1, 2, T, d, generator=g) for _ in range(2))
    if kind == "tiny_q":
        return q * 2.0 ** -124, k * 2.0 ** 120
    if kind == "tiny_k":
        return q * 2.0 ** 120, k * 2.0 ** -124
    if kind == "mixed":
        q[..., 1] *= 2.0 ** 50
        q[..., 3] = q[..., 3] * 2.0 ** -120
        return q, k * 2.0 ** 70
    return q, k


@pytest.mark.parametrize("kind", ("plain", "tiny_q", "tiny_k", "mixed"))
@pytest.mark.parametrize("d", (16, 32, 64, 128))
def test_scores_bit_for_bit(d, kind):
    T = 97
    print(f"case scores d{d} {kind}", flush=True)
    q, k = draws(d, T, kind)
    s = torch.zeros(1, 2, T, T, device="cuda")
    kia.kia_debug_scores(q.cuda(), k.cuda(), s, 0)
    torch.cuda.synchronize()
    for h in range(2):
        want = chain(q[0, h].numpy(), k[0, h].numpy())
        assert np.isfinite(want).all()
        assert np.array_equal(s[0, h].cpu().numpy(), want), (d, kind, h)


# launch shapes: one row group with eight and four key parts, two row groups
# with two halves, 128 rows; T on both sides of their tiles
@pytest.mark.parametrize("B,H,T,causal", ((1, 2, 300, 1), (2, 64, 40, 0), (10, 30, 97, 1),
                                          (12, 50, 130, 1)))
@pytest.mark.parametrize("d", (16, 32, 64, 128))
def test_forward_takes_the_same_scores(d, B, H, T, causal):
    """The forward's row extrema are those of the exported scores, and a
    tiny-q call's output is that of the call it was scaled from (every factor a
    power of two, normal elements only: min |q| 2^-110 > 2^-126)."""
    print(f"case forward scores d{d} B{B} H{H} T{T}", flush=True)
    g = torch.Generator().manual_seed(T)
    q, k, v = (torch.randn(B, H, T, d, generator=g).cuda() for _ in range(3))
    q = torch.where(q.abs() < 2.0 ** -12, torch.full_like(q, 2.0 ** -12), q)
    k = torch.where(k.abs() < 2.0 ** -12, torch.full_like(k, 2.0 ** -12), k)
    args = (4, "minmax", 8.0, "lerp", "weight", False, causal)
    o, st = kia.forward(q, k, v, *args)
    s = torch.zeros(B, H, T, T, device="cuda")
    kia.kia_debug_scores(q, k, s, causal)
    torch.cuda.synchronize()
    valid = torch.ones(T, T, dtype=torch.bool, device="cuda")
    if causal:
        valid = valid.tril()
    for f, want in (("M", s.masked_fill(~valid, -torch.inf).amax(-1)),
                    ("m", s.masked_fill(~valid, torch.inf).amin(-1))):
        assert torch.equal(kia.stats_field(st, B, H, T, d, f), want), f
    for a, b in ((-110, 110), (110, -110)):
        x, _ = kia.forward(q * 2.0 ** a, k * 2.0 ** b, v, *args)
        torch.cuda.synchronize()
        assert torch.equal(x, o), (a, b)
