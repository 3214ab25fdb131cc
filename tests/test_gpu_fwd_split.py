"""F(2^3, 3^3) forward in one kernel (bf16-split products, V formed in LDS):
every output against the fp64 direct correlation at the sizes where its blocks,
steps and row loads change, and the layers just outside its rule beside them.

The bar is the library's for m = 2 (1e-5 of the summed magnitudes): the split
leaves out terms below 2^-22 of a product and otherwise rounds in fp32."""
import numpy as np
import pytest

from gpu_util import check_full, run_layer
from workloads import LayerSpec, draw_layer

pytestmark = pytest.mark.gpu


def layer(name, batch, C, K, X, pad=1, **kw):
    return LayerSpec(name, N=3, m=2, r=3, batch=batch, C=C, K=K, X=X, pad=pad, x_dist="normal", w_dist="he", **kw)


INSIDE = [
    layer("three_tiles_a_kernel", 1, 16, 1, (2, 16, 40)),          # 160 tiles (192 padded) for 64 kernels, one stage
    layer("odd_first_axes", 2, 32, 70, (7, 11, 36), relu=True),   # cropped tiles, ragged kernel block
    layer("ragged_tile_block", 3, 48, 64, (5, 7, 12), leaky=0.2),  # T past a whole block, three stages
    layer("rows_of_66_tiles", 1, 32, 130, (8, 6, 132)),           # rows longer than a wave's 32 tiles
    layer("two_blocks_of_kernels", 1, 16, 128, (8, 6, 132)),      # the last with 16 channels
    layer("rows_of_32_tiles", 2, 64, 128, (4, 8, 64)),            # rows end where the wave's tiles do
    layer("rows_of_2_tiles", 5, 16, 3, (9, 13, 4)),               # every pair of tiles is a row
    layer("whole_blocks", 8, 32, 64, (16, 56, 56)),               # full rounds, nothing in parts
    layer("tail_after_rounds", 15, 16, 64, (8, 48, 48)),          # full rounds, then blocks in parts
]
OUTSIDE = [
    layer("row_not_of_4", 2, 32, 64, (7, 11, 34)),
    layer("channels_not_of_16", 1, 24, 64, (8, 12, 32)),
    layer("no_padding", 2, 32, 64, (10, 12, 36), pad=0),
    layer("three_blocks_of_kernels", 1, 16, 130, (8, 6, 132)),    # too few channels for them
    layer("few_tiles_a_kernel", 1, 16, 400, (2, 4, 8)),
    layer("one_pair_of_tiles", 1, 16, 1, (1, 1, 4)),
]


@pytest.mark.parametrize("split", [True, False], ids=["parts", "whole"])
@pytest.mark.parametrize("spec", INSIDE + OUTSIDE, ids=lambda s: s.name)
def test_full_output(spec, split):
    x, w = draw_layer(spec, seed=41)
    b = (np.random.default_rng(2).standard_normal(spec.K) * 0.3).astype(np.float32)
    y, plan = run_layer(spec, x, w, bias=b, guard=1024, split=split)
    assert plan.desc["forward_split"] == (spec in INSIDE), plan.desc
    check_full(spec, y, x, w, bias=b)


def test_pads_of_the_leading_axes():
    """The rule asks for pad 1 on the last axis only."""
    import torch

    from oracle.direct import direct_blas
    from oracle.metric import normalised_error
    from paper_1611_06565_amd.wino import Plan
    spec = layer("pads_0_2_1", 2, 32, 64, (6, 9, 32))
    x, w = draw_layer(spec, seed=5)
    plan = Plan(3, 2, 3, 32, 64, [2, 6, 9, 32], pad=[0, 2, 1])
    assert plan.desc["forward_split"] == 1
    y = plan.forward(torch.from_numpy(x).cuda(), plan.transform_filter(torch.from_numpy(w).cuda())).cpu().numpy()
    xp = np.pad(x, ((0, 0), (0, 0), (0, 0), (2, 2), (1, 1)))
    ref, den = direct_blas(xp, w, 0)
    assert normalised_error(y, ref, den)["max"] <= 1e-5


def test_error_no_larger_than_two_stages():
    """Against fp64 the split products are at least as close as the fp32 ones."""
    import torch

    from oracle.direct import direct_blas
    from paper_1611_06565_amd.wino import Plan
    for C, dist in ((16, "normal"), (64, "relu_normal"), (256, "uniform")):
        spec = layer("err", 2, C, 64, (6, 8, 32)).with_(x_dist=dist)
        x, w = draw_layer(spec, seed=9)
        ref, _ = direct_blas(x, w, 1)
        err = []
        for fuse in (True, False):
            plan = Plan(3, 2, 3, C, 64, [2, 6, 8, 32], pad=1, fuse=fuse)
            assert plan.desc["forward_split"] == fuse
            y = plan.forward(torch.from_numpy(x).cuda(), plan.transform_filter(torch.from_numpy(w).cuda()))
            err.append(np.linalg.norm(y.cpu().numpy() - ref) / np.linalg.norm(ref))
        print(C, dist, err)
        assert err[0] <= err[1], (C, dist, err)


def _forward(dims, C, K, pad, x, w):
    import torch

    from paper_1611_06565_amd.wino import Plan
    plan = Plan(3, 2, 3, C, K, dims, pad=pad, split=False)
    assert plan.desc["forward_split"] == 1
    y = plan.forward(torch.from_numpy(np.ascontiguousarray(x)).cuda(), plan.transform_filter(torch.from_numpy(w).cuda()))
    return y.cpu().numpy()


def test_bitwise_invariants():
    """What needs no oracle value: a shift by one tile along an unpadded axis, a
    sample alone, and a doubled input give the same bits (whole blocks)."""
    C, K = 32, 70
    pad = [0, 0, 1]
    spec = layer("inv", 2, C, K, (10, 13, 36))
    x, w = draw_layer(spec, seed=43)
    y = _forward([2, 10, 13, 36], C, K, pad, x, w)
    assert np.array_equal(_forward([2, 8, 13, 36], C, K, pad, x[:, :, 2:], w), y[:, :, 2:])
    assert np.array_equal(_forward([2, 10, 11, 36], C, K, pad, x[:, :, :, 2:], w), y[:, :, :, 2:])
    for b in range(2):
        assert np.array_equal(_forward([1, 10, 13, 36], C, K, pad, x[b:b + 1], w)[0], y[b])
    assert np.array_equal(_forward([2, 10, 13, 36], C, K, pad, 2 * x, w), 2 * y)


def test_integer_inputs_bitwise_exact():
    """Integers in [-2, 2]: every split, product and sum is exact."""
    from oracle.direct import direct_blas
    rng = np.random.default_rng(3)
    x = rng.integers(-2, 3, size=(2, 32, 7, 12, 36)).astype(np.float32)
    w = rng.integers(-2, 3, size=(70, 32, 3, 3, 3)).astype(np.float32)
    ref, _ = direct_blas(x, w, 1)
    assert np.array_equal(_forward([2, 7, 12, 36], 32, 70, 1, x, w), ref.astype(np.float32))


@pytest.mark.parametrize("xs,ws", [(2.0 ** -110, 1.0), (1.0, 2.0 ** -102), (2.0 ** -60, 2.0 ** -60), (2.0 ** 60, 2.0 ** 50)])
def test_magnitudes(xs, ws):
    """The three parts of a value hold all its bits while the last is a normal
    bf16 number (values from about 2^-112 up: U's are 2^-5 to 2^-9 of this w's
    scale), and the products' small terms are not flushed: the relative error is that of values around 1 (2-norms over
    131,072 outputs: 5% leaves them their spread)."""
    from oracle.direct import direct_blas
    rng = np.random.default_rng(2)
    x = rng.standard_normal((4, 32, 8, 8, 16), dtype=np.float32)
    w = (0.05 * rng.standard_normal((32, 32, 3, 3, 3))).astype(np.float32)
    err = []
    for a, b in ((1.0, 1.0), (xs, ws)):
        sx, sw = x * np.float32(a), w * np.float32(b)
        ref, _ = direct_blas(sx, sw, 1)
        err.append(np.linalg.norm(_forward([4, 8, 8, 16], 32, 32, 1, sx, sw) - ref) / np.linalg.norm(ref))
    assert err[1] <= 1.05 * err[0], err
