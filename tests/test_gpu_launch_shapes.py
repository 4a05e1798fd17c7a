"""Every launch shape of the forward, by the grid sizes at which the default
policy takes it, forward and backward against the fp64 oracle.

Blocks are 128 rows of one (b, h). Up to 128 blocks take one row group with eight
key parts (fp32, d <= 64, T > 128) or four, 150 to 700 one row group with four or
two with two, by type and d, 1100 the largest shape; each T leaves the last key
tile of a part ragged in another way. Dyadic q and k: codes, extrema and tie counts
bit for bit, the rest at the bounds of the parity tests.
"""
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

import paper_2609_33591_amd as kia  # noqa: E402
from paper_2609_33591_amd.inputs import make_inputs  # noqa: E402
import test_gpu_bf16 as B16  # noqa: E402
import test_gpu_parity as P  # noqa: E402

GRIDS = ((1, 12, 300), (2, 10, 97), (3, 50, 127), (10, 20, 65), (20, 20, 97), (20, 35, 33), (22, 50, 100))
OPS = (("fwm", "nearest", "prob"), ("minmax", "lerp", "weight"), ("minmax", "nearest", "weight"))


@pytest.mark.parametrize("op", OPS, ids=lambda o: "-".join(o))
@pytest.mark.parametrize("B,H,T", GRIDS)
@pytest.mark.parametrize("d", (16, 32, 64, 128))
@pytest.mark.parametrize("dtype", ("f32", "bf16"))
def test_launch_shapes(oracle_mod, dtype, d, B, H, T, op):
    calib, recon, ste = op
    causal = 0 if T == 65 else 1
    tag = f"{dtype} B{B} H{H} T{T} d{d} {calib} {recon} {ste} causal{causal}"
    P.flush("case " + tag)
    x = make_inputs(B, H, T, d, seed=1000 + T, dyadic=True)
    args = (5, calib, 8.0, recon, ste, False, causal)
    # the first and the last slice
    keep = (0, B * H - 1)
    if dtype == "bf16":
        xb, x = B16.bf16_inputs(*x)
        g = B16.run_gpu16(*xb, *args, keep=keep)
    else:
        g = P.run_gpu(*x, *args, keep=keep)
    n = {k: v if k.startswith("codes") else v.reshape(1, -1, *v.shape[2:])[:, list(keep)]
         for k, v in g.items()}
    few = [t.reshape(1, -1, *t.shape[2:])[:, list(keep)].contiguous() for t in x]
    r = P.run_oracle(oracle_mod, *few, *args)
    (B16.compare16 if dtype == "bf16" else P.compare)(n, r, oracle_mod, calib, [(0, 0), (0, 1)],
                                                      tag=tag)


@pytest.mark.parametrize("recon", ("nearest", "lerp"))
@pytest.mark.parametrize("B,H,T", GRIDS)
@pytest.mark.parametrize("d", (16, 32, 64, 128))
@pytest.mark.parametrize("dtype", (torch.float32, torch.bfloat16))
def test_forward_bits_at_every_launch_shape(dtype, d, B, H, T, recon):
    """The forward is bitwise independent of the surrogate and of the gradient mode
    (the forward-only mode among them), and so is its launch shape."""
    P.flush(f"case forward bits {dtype} B{B} H{H} T{T} d{d} {recon}")
    q, k, v, _ = (t.to(dtype).cuda() for t in make_inputs(B, H, T, d, seed=1100 + T))
    for calib in ("fwm", "minmax"):
        ref = kia.forward(q, k, v, 4, calib, 8.0, recon, "prob", False, 1)[0]
        for ste, mode in (("weight", False), ("prob", "none"), ("weight", "none")):
            o = kia.forward(q, k, v, 4, calib, 8.0, recon, ste, mode, 1)[0]
            assert torch.equal(o, ref), (calib, ste, mode)


@pytest.mark.parametrize("T", (1024, 1001))
@pytest.mark.parametrize("d", (16, 128))
@pytest.mark.parametrize("dtype", (torch.float32, torch.bfloat16))
def test_dv_repeats_from_one_block_per_cu(dtype, d, T):
    """From one 128-key block per CU up, dV is bitwise the same on every call, and
    that of the unsplit launch up to the order of its sums (two fp32 sums of T
    terms at most: 2 T 2^-24 of the norm)."""
    B, H = 2, 16  # 256 blocks
    P.flush(f"case dv repeats {dtype} d{d} T{T}")
    assert B * H * ((T + 127) // 128) >= \
        torch.cuda.get_device_properties(0).multi_processor_count
    q, k, v, dO = (t.to(dtype).cuda() for t in make_inputs(B, H, T, d, seed=77))
    args = (4, "fwm", 8.0, "lerp", "weight", False, 1)
    o, st = kia.forward(q, k, v, *args)
    ref = kia.backward(q, k, v, o, dO, st, *args)
    for _ in range(4):
        assert torch.equal(kia.backward(q, k, v, o, dO, st, *args)[2], ref[2])
    kia.kia_set_grid_policy("wide")
    try:
        wide = kia.backward(q, k, v, o, dO, st, *args)
    finally:
        kia.kia_set_grid_policy("auto")
    for a, b, n in zip(ref, wide, ("dq", "dk", "dv")):
        assert (a - b).norm() <= 2 * T * 2.0 ** -24 * b.norm(), n
