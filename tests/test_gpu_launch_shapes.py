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
