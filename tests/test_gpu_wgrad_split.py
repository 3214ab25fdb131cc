"""Weight gradient of F(2^3, 3^3) with both transforms inside the product:
every output against the fp64 oracle at the sizes where its steps of 16 tiles,
its row blocks and its tile ranges change.  Bar: 1e-4 of the summed magnitudes,
as for every weight gradient (the products round less often than the fp32 ones:
6 times for 16 tiles)."""
import numpy as np
import pytest

from gpu_util import log, require_gpu
from oracle.metric import normalised_error
from oracle.wgrad import direct_wgrad

pytestmark = pytest.mark.gpu

# (name, batch, C, K, X): pad 1, the last extent a multiple of 4
LAYERS = [
    ("eight_tiles", 1, 1, 1, (4, 4, 4)),                # one step, half masked
    ("rows_shorter_than_a_step", 2, 5, 7, (3, 5, 4)),   # 2-tile rows: every pair ends a row
    ("rows_of_6_tiles", 1, 16, 64, (5, 7, 12)),         # rows end inside a step, cropped first axes
    ("rows_of_16_tiles", 1, 64, 65, (4, 4, 32)),        # rows end with the steps; a second row block
    ("rows_of_18_tiles", 2, 66, 128, (3, 4, 36)),       # rows longer than a step, two channel blocks
    ("ragged_blocks", 1, 130, 200, (4, 6, 8)),          # three channel blocks, 128 + 72 kernels
    ("uneven_ranges", 3, 20, 96, (9, 17, 20)),
]
# too short a contraction, a leading axis of one position, or a chain of steps
# longer than V and D take: the fp32 products
FP32 = [
    ("four_steps_of_two_blocks", 4, 96, 96, (2, 8, 8)),
    ("one_row_of_two_tiles", 1, 1, 1, (1, 1, 4)),
    ("two_tiles", 1, 1, 1, (2, 2, 4)),
    ("six_tiles", 1, 3, 2, (2, 2, 12)),
    ("one_plane", 1, 1, 1, (1, 6, 8)),
    ("one_row_a_plane", 2, 1, 1, (6, 1, 8)),
]


@pytest.mark.parametrize("layer", LAYERS + FP32, ids=lambda v: v[0])
def test_full_output(layer):
    torch = require_gpu()
    from paper_1611_06565_amd.wino import Plan
    name, batch, C, K, X = layer
    rng = np.random.default_rng(8)
    plan = Plan(3, 2, 3, C, K, [batch, *X], pad=1)
    assert plan.desc["wgrad_split"] == (layer in LAYERS), plan.desc
    x = rng.standard_normal(plan.input_shape, dtype=np.float32)
    dy = rng.standard_normal(plan.output_shape, dtype=np.float32)
    n = int(np.prod(plan.weight_shape))
    buf = torch.full((n + 2048,), 12345.5, device="cuda")
    dw = buf[1024:1024 + n].view(plan.weight_shape)
    plan.weight_gradient(torch.from_numpy(x).cuda(), torch.from_numpy(dy).cuda(), dw=dw)
    torch.cuda.synchronize()
    assert bool((buf[:1024] == 12345.5).all()) and bool((buf[1024 + n:] == 12345.5).all())
    ref, den = direct_wgrad(x, dy, 3, 1)
    err = normalised_error(dw.cpu().numpy(), ref, den)
    log(f"[gpu] wgrad split {name}: max err {err['max']:.3e} at {err['argmax']}")
    assert err["nonfinite"] == 0 and err["max"] <= 1e-4, err


def test_leading_pads():
    """The rule asks for pad 1 on the last axis only."""
    torch = require_gpu()
    from paper_1611_06565_amd.wino import Plan
    rng = np.random.default_rng(3)
    plan = Plan(3, 2, 3, 9, 10, [2, 6, 5, 8], pad=[0, 2, 1])
    assert plan.desc["wgrad_split"] == 1, plan.desc
    x = rng.standard_normal(plan.input_shape, dtype=np.float32)
    dy = rng.standard_normal(plan.output_shape, dtype=np.float32)
    dw = plan.weight_gradient(torch.from_numpy(x).cuda(), torch.from_numpy(dy).cuda()).cpu().numpy()
    xp = np.pad(x, ((0, 0), (0, 0), (0, 0), (2, 2), (1, 1)))
    ref, den = direct_wgrad(xp, dy, 3, 0)
    assert normalised_error(dw, ref, den)["max"] <= 1e-4


@pytest.mark.parametrize("X", [(1, 1, 4), (1, 2, 4), (2, 1, 4), (2, 2, 4), (2, 2, 8), (2, 2, 12), (4, 4, 4),
                               (2, 2, 16), (5, 4, 4), (4, 6, 8), (1, 8, 8), (8, 1, 8)], ids=str)
def test_error_no_larger_than_fp32_products(X):
    """Against fp64, whichever kernel the plan takes, the error is that of the
    fp32 products (which the same points in another order run) or less.  Their
    transforms sum in another order there, which moves the 2-norm over the
    48 x 48 x 27 values by up to 7% on these layers: the assertion leaves 10%.
    On two tiles the split products are 16 to 25% off."""
    torch = require_gpu()
    from paper_1611_06565_amd.wino import Plan
    C = K = 48
    for dist in ("normal", "relu"):
        rng = np.random.default_rng(12)
        x = rng.standard_normal((1, C, *X), dtype=np.float32)
        x = np.maximum(x, 0) if dist == "relu" else x
        dy = rng.standard_normal((1, K, *X), dtype=np.float32)
        ref, _ = direct_wgrad(x, dy, 3, 1)
        err = []
        for points in (None, (0, -1, 1)):
            plan = Plan(3, 2, 3, C, K, [1, *X], pad=1, points=points)
            assert points is None or plan.desc["wgrad_split"] == 0
            dw = plan.weight_gradient(torch.from_numpy(x).cuda(), torch.from_numpy(dy).cuda()).cpu().numpy()
            err.append(np.linalg.norm(dw - ref) / np.linalg.norm(ref))
        log(f"[gpu] wgrad {X} {dist}: {err[0]:.3e} against {err[1]:.3e}")
        assert err[0] <= 1.1 * err[1], (X, dist, err)
