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

# (name, batch, C, K, X): pad 1, the last extent a multiple of 4.  Extents of
# at least 2: with an extent of 1 a tap outside it sums nothing, its denominator
# is the metric's floor (1e-3 of the mean), and the 2^-24 rounding of products
# that cancel there is 6e-5 of that floor times the transforms' growth, past the
# bar (1 x 1 x 4: 2.3e-4 here, 0.8e-4 in fp32, at an absolute error of 1.9e-7 in both).
LAYERS = [
    ("two_tiles", 1, 1, 1, (2, 2, 4)),                  # one step, mostly masked
    ("rows_shorter_than_a_step", 2, 5, 7, (3, 5, 4)),   # 2-tile rows: every pair ends a row
    ("rows_of_6_tiles", 1, 16, 64, (5, 7, 12)),         # rows end inside a step, cropped first axes
    ("rows_of_16_tiles", 1, 64, 65, (4, 4, 32)),        # rows end with the steps; a second row block
    ("rows_of_18_tiles", 2, 66, 128, (3, 4, 36)),       # rows longer than a step, two channel blocks
    ("ragged_blocks", 1, 130, 200, (4, 6, 8)),          # three channel blocks, 128 + 72 kernels
    ("uneven_ranges", 3, 20, 96, (9, 17, 20)),
]


@pytest.mark.parametrize("layer", LAYERS, ids=lambda v: v[0])
def test_full_output(layer):
    torch = require_gpu()
    from paper_1611_06565_amd.wino import Plan
    name, batch, C, K, X = layer
    rng = np.random.default_rng(8)
    plan = Plan(3, 2, 3, C, K, [batch, *X], pad=1)
    assert plan.desc["wgrad_split"] == 1, plan.desc
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
