"""The order of a row product's tiles: an expert of up to four row tiles has those of the same columns together, a larger one has its row
tiles one after the other.  Experts at that line and around it, none and few rows between them, against the oracle: on the tile of 256 rows
with one to four column tiles per product, on the tile of 128 rows (few rows per expert on average), and in the 8-bit forward."""
import numpy as np
import pytest

from oracle import moe_oracle as O
from tests.util import assert_close, q, to_dev, to_np, torch_dtype

pytestmark = pytest.mark.gpu

# rows of each expert: 4 tiles exactly, 5 (one row in the last), none, 1, 4 with a partial one, 6, 2, 3
ROWS = [1024, 1025, 0, 1, 1000, 1400, 300, 700]
# the same line for tiles of 128 rows, which are taken up to an average of 128 rows per expert where d is small: 4 tiles, 5, none, 1, 4, 2, 1, 1 ...
FEW_ROWS = [512, 513, 0, 1, 500, 129, 128, 127, 20, 0, 0, 5, 7, 3, 2, 0]


def _experts_around_the_group_size(rows, d, f, gather):
    import torch
    from paper_2508_02317_amd.layer import MoELayer
    E, T = len(rows), sum(rows)
    r = np.random.default_rng(d * 7 + f)
    X, dY = q(r.standard_normal((T, d)), "bf16"), q(r.standard_normal((T, d)), "bf16")
    Wg, Wu = (q(r.standard_normal((E, f, d)) * 0.05, "bf16") for _ in range(2))
    Wd = q(r.standard_normal((E, d, f)) * 0.05, "bf16")
    idx = r.permutation(np.repeat(np.arange(E, dtype=np.int32), rows))[:, None]
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


@pytest.mark.parametrize("gather", [True, False])
@pytest.mark.parametrize("d,f", [(264, 136), (520, 264), (64, 392)])
def test_experts_around_the_group_size(d, f, gather):
    _experts_around_the_group_size(ROWS, d, f, gather)


@pytest.mark.parametrize("gather", [True, False])
@pytest.mark.parametrize("d,f", [(264, 136), (520, 392)])
def test_experts_around_the_group_size_on_the_tile_of_128_rows(d, f, gather):
    assert sum(FEW_ROWS) <= 128 * len(FEW_ROWS) and len(FEW_ROWS) * -(-d // 256) < 256      # the rule for that tile
    _experts_around_the_group_size(FEW_ROWS, d, f, gather)


@pytest.mark.parametrize("gather", [True, False])
@pytest.mark.parametrize("d,f", [(256, 128), (512, 384), (384, 256)])
def test_8_bit_experts_around_the_group_size(d, f, gather):
    """Against the oracle, and with the outputs inside larger buffers: in the last tile of the last expert, as in others, half of the waves
    have no rows; they go through the first strip of the epilogue and must store nothing, neither into the rows of the next expert nor
    behind the outputs."""
    import torch
    from paper_2508_02317_amd import libmoe as L
    from paper_2508_02317_amd.inputs import CONFIGS, make_inputs, scaled
    from tests.test_gpu_mx8 import _compare_forward
    rows = ROWS + [300]
    E, T = len(rows), sum(rows)
    cfg = scaled(CONFIGS["a3b_8k"], T=T, d=d, E=E, k=1, f=f, seed=d + f)
    inp = make_inputs(cfg)
    idx = np.random.default_rng(d + f).permutation(np.repeat(np.arange(E, dtype=np.int32), rows))[:, None]
    _, offsets = O.counts_offsets(idx, E)
    offsets, pair_of_row = offsets.astype(np.int32), O.permute_maps(idx, offsets)[1].astype(np.int32)
    print("8-bit d=%d f=%d gather=%s" % (d, f, gather), flush=True)
    ref = _compare_forward(cfg, inp, offsets, pair_of_row, gather)
    dev = lambda name: to_dev(inp[name], "bf16")
    x = dev("X") if gather else dev("X")[to_dev(pair_of_row).long()].contiguous()
    weights = [t for name in ("Wg", "Wu", "Wd") for t in L.moe_mx8_quantise(dev(name))]
    guard = [torch.full((n + 65536,), 77, dtype=dt, device="cuda") for n, dt in ((T * f, torch.uint8), (T * f // 128, torch.int32), (T * d, torch.bfloat16))]
    out = tuple(b[:b.numel() - 65536].view(shape) for b, shape in zip(guard, ((T, f), (f // 128, T), (T, d))))
    L.moe_grouped_gemm_swiglu_fwd_mx8(*L.moe_mx8_quantise(x), *weights, to_dev(offsets), pair_of_row=to_dev(pair_of_row) if gather else None, k=1, out=out)
    torch.cuda.synchronize()
    for got, want, b in zip(out, ref, guard):
        assert np.array_equal(to_np(got), want)
        assert bool((b[-65536:] == 77).all())
