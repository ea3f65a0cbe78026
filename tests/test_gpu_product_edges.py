"""GPU parity of the bf16 products where their tiles and slabs end: reduction lengths around one slab (64), row counts
around one MFMA fragment (16), one wavefront (128) and one tile (256), and widths around one tile.

The bound is that of every bf16 product (operands rounded to 8 bits, fp32 accumulation, one rounding of the result)."""
import numpy as np
import pytest

from oracle import moe_oracle as O
from tests.util import assert_close, q, to_dev, to_np, torch_dtype

pytestmark = pytest.mark.gpu

# (T, d, f): E = 2 experts, k = 1; about half the rows each, except T = 1 (one expert has none)
SIZES = [(1, 8, 8), (31, 56, 64), (33, 64, 72), (130, 72, 128), (258, 128, 136), (509, 136, 56), (515, 264, 248),
         (1030, 192, 320)]


@pytest.mark.parametrize("gather", [True, False])
@pytest.mark.parametrize("T,d,f", SIZES)
def test_products_at_tile_and_slab_edges(T, d, f, gather):
    import torch
    from paper_2508_02317_amd.layer import MoELayer
    r = np.random.default_rng(T * 7 + d)
    X, dY = q(r.standard_normal((T, d)), "bf16"), q(r.standard_normal((T, d)), "bf16")
    Wg, Wu = (q(r.standard_normal((2, f, d)) * 0.05, "bf16") for _ in range(2))
    Wd = q(r.standard_normal((2, d, f)) * 0.05, "bf16")
    logits = r.standard_normal((T, 2)).astype(np.float32)
    fwd = O.moe_layer_fwd(X, logits, Wg, Wu, Wd, 1)
    bwd = O.moe_layer_bwd(fwd, dY, logits, Wg, Wu, Wd)
    layer = MoELayer(T, d, 2, 1, f, torch_dtype("bf16"), to_dev(Wg, "bf16"), to_dev(Wu, "bf16"), to_dev(Wd, "bf16"), gather=gather)
    z = to_dev(logits)
    layer.forward(to_dev(X, "bf16"), logits=z)
    layer.backward(to_dev(dY, "bf16"), logits=z)
    torch.cuda.synchronize()
    for name, got, ref in (("Y", layer.y, fwd["Y"]), ("dX", layer.dx, bwd["dX"]), ("dWg", layer.dw_gate, bwd["dWg"]),
                           ("dWu", layer.dw_up, bwd["dWu"]), ("dWd", layer.dw_down, bwd["dWd"])):
        assert_close(to_np(got), ref, "bf16", name)
