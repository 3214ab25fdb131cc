"""F(4^2, 3^2) product on the bf16 matrix cores (split fp32 operands): every
output against the fp64 direct correlation at the edges of its blocks, channel
stages, tail parts and row stores."""
import numpy as np
import pytest

from gpu_util import check_full, run_layer
from workloads import LayerSpec, draw_layer

pytestmark = pytest.mark.gpu


def layer(name, batch, C, K, X, pad=1, **kw):
    return LayerSpec(name, N=2, m=4, r=3, batch=batch, C=C, K=K, X=X, pad=pad, x_dist="normal", w_dist="he", **kw)


SPECS = [
    layer("one_output", 1, 1, 1, (1, 1)),                         # one tile, one stage
    layer("rows_of_whole_units", 1, 16, 32, (8, 12), relu=True),  # 16-byte stores
    layer("ragged_rows", 2, 17, 33, (9, 11), leaky=0.1),          # cropped stores, two stages, a second kernel block
    layer("half_a_block", 1, 32, 40, (16, 32)),                   # 32 tiles: the block's second half is padding
    layer("past_a_block", 3, 48, 96, (20, 18)),                   # three stages, tiles past one block
    layer("many_parts", 1, 272, 32, (12, 12)),                    # 17 stages in up to 16 uneven parts
    layer("parts_of_stages", 16, 128, 64, (32, 32)),              # 16 tail blocks of 8 stages in parts
    layer("few_stages_whole", 24, 32, 32, (30, 31)),              # 24 blocks kept whole
    layer("passes_instead", 16, 96, 48, (32, 29)),                # 32 blocks of 6 stages: the fp32 passes
    layer("no_padding", 2, 64, 64, (30, 27), pad=0),
]


# layers whose blocks the fp32 passes spread further (not with WINO_NO_SPLIT)
PASSES = ("one_output", "rows_of_whole_units", "ragged_rows", "half_a_block", "passes_instead")


@pytest.mark.parametrize("split", [True, False], ids=["parts", "whole"])
@pytest.mark.parametrize("spec", SPECS, ids=lambda s: s.name)
def test_full_output(spec, split):
    x, w = draw_layer(spec, seed=17)
    b = (np.random.default_rng(4).standard_normal(spec.K) * 0.3).astype(np.float32)
    y, plan = run_layer(spec, x, w, bias=b, guard=1024, split=split)
    assert plan.desc["gemm_split"] == (0 if split and spec.name in PASSES else 1), plan.desc
    check_full(spec, y, x, w, bias=b)
