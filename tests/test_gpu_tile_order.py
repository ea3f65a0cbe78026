"""The order of a row product's tiles: an expert of up to four row tiles (256 rows each) has those of the same columns together,
a larger one has its row tiles one after the other.  Experts at that line and around it, none and few rows between them, with one, two and
three column tiles per product, against the oracle."""
import numpy as np
import pytest

from oracle import moe_oracle as O
from tests.util import assert_close, q, to_dev, to_np, torch_dtype

pytestmark = pytest.mark.gpu

# rows of each expert: 4 tiles exactly, 5 (one row in the last), none, 1, 4 with a partial one, 6, 2, 3
ROWS = [1024, 1025, 0, 1, 1000, 1400, 300, 700]


@pytest.mark.parametrize("gather", [True, False])
@pytest.mark.parametrize("d,f", [(264, 136), (520, 264), (64, 392)])
def test_experts_around_the_group_size(d, f, gather):
    import torch
    from paper_2508_02317_amd.layer import MoELayer
    E, T = len(ROWS), sum(ROWS)
    r = np.random.default_rng(d * 7 + f)
    X, dY = q(r.standard_normal((T, d)), "bf16"), q(r.standard_normal((T, d)), "bf16")
    Wg, Wu = (q(r.standard_normal((E, f, d)) * 0.05, "bf16") for _ in range(2))
    Wd = q(r.standard_normal((E, d, f)) * 0.05, "bf16")
    idx = r.permutation(np.repeat(np.arange(E, dtype=np.int32), ROWS))[:, None]
    w = r.uniform(0.2, 1.0, (T, 1)).astype(np.float32)
    fwd = O.moe_layer_fwd(X, None, Wg, Wu, Wd, 1, routing=(idx, w))
    bwd = O.moe_layer_bwd(fwd, dY, None, Wg, Wu, Wd)
    layer = MoELayer(T, d, E, 1, f, torch_dtype("bf16"), to_dev(Wg, "bf16"), to_dev(Wu, "bf16"), to_dev(Wd, "bf16"), prerouted=True,
                     gather=gather)
    layer.forward(to_dev(X, "bf16"), topk_idx=to_dev(idx), topk_w=to_dev(w))
    layer.backward(to_dev(dY, "bf16"))
    torch.cuda.synchronize()
    for name, got, ref in (("Y", layer.y, fwd["Y"]), ("dX", layer.dx, bwd["dX"]), ("dWg", layer.dw_gate, bwd["dWg"]),
                           ("dWu", layer.dw_up, bwd["dWu"]), ("dWd", layer.dw_down, bwd["dWd"]), ("dw", layer.dw, bwd["dw"])):
        assert_close(to_np(got), ref, "bf16", name)
