"""GPU parity where experts have no rows: their weight gradients are zeros that workgroups store 128 KiB at a time, those without a
tile while the others multiply (when they are at least half of the 256), or whoever is done, by a counter.  What can go wrong: a
piece left out or stored over a neighbour (the last piece of an expert, the piece that holds both weights of [dW_gate; dW_up]), the
counter of an earlier call, no expert with rows at all.  Result buffers hold NaN before each call."""
import numpy as np
import pytest

from oracle import moe_oracle as O
from tests.util import assert_close, q, to_dev, to_np, torch_dtype

pytestmark = pytest.mark.gpu


# experts with rows: two of 32 (a tile or two each, the rest of the chip idle; results of less than a piece), one of 9 (several pieces
# each), 12 of 40 (180 tiles of dW_down, 300 of [dW_gate; dW_up]), all but the first and all but the last, and 3 with split rows
CASES = {"two_of_32": (40, 136, 32, 264, [3, 7]), "one_of_9": (70, 1032, 9, 520, [4]), "twelve_of_40": (900, 1032, 40, 520, list(range(1, 37, 3))),
         "not_the_first": (300, 264, 8, 136, list(range(1, 8))), "not_the_last": (300, 264, 8, 136, list(range(7))),
         "split_rows": (9000, 264, 16, 520, [0, 5, 15])}


@pytest.mark.parametrize("gather,save_gu", [(True, True), (False, False)])
@pytest.mark.parametrize("name", CASES)
def test_weight_gradients_of_experts_without_rows(name, gather, save_gu):
    import torch
    from paper_2508_02317_amd.layer import MoELayer
    T, d, E, f, used = CASES[name]
    r = np.random.default_rng(T + d + E)
    logits = np.full((T, E), -50.0, np.float32)
    logits[:, used] = r.standard_normal((T, len(used))).astype(np.float32)
    X, dY = q(r.standard_normal((T, d)), "bf16"), q(r.standard_normal((T, d)), "bf16")
    Wg, Wu = (q(r.standard_normal((E, f, d)) * 0.05, "bf16") for _ in range(2))
    Wd = q(r.standard_normal((E, d, f)) * 0.05, "bf16")
    fwd = O.moe_layer_fwd(X, logits, Wg, Wu, Wd, 1)
    bwd = O.moe_layer_bwd(fwd, dY, logits, Wg, Wu, Wd)
    layer = MoELayer(T, d, E, 1, f, torch_dtype("bf16"), to_dev(Wg, "bf16"), to_dev(Wu, "bf16"), to_dev(Wd, "bf16"), gather=gather, save_gu=save_gu)
    empty = [e for e in range(E) if e not in used]
    for _ in range(2):
        for t in (layer.dw_gate, layer.dw_up, layer.dw_down):
            t.fill_(float("nan"))
        layer.forward(to_dev(X, "bf16"), logits=to_dev(logits))
        layer.backward(to_dev(dY, "bf16"), logits=to_dev(logits))
        torch.cuda.synchronize()
        for what, got, ref in (("dWg", layer.dw_gate, bwd["dWg"]), ("dWu", layer.dw_up, bwd["dWu"]), ("dWd", layer.dw_down, bwd["dWd"])):
            assert_close(to_np(got), ref, "bf16", what)
            assert not to_np(got)[empty].any(), what
    assert_close(to_np(layer.dx), bwd["dX"], "bf16", "dX")


@pytest.mark.parametrize("E,d,f", [(1, 8, 8), (5, 1032, 264), (300, 136, 72)])
def test_weight_gradients_without_any_rows(E, d, f):
    import torch
    from paper_2508_02317_amd import libmoe as L
    z = lambda *s: torch.zeros(s, dtype=torch.bfloat16, device="cuda")
    offsets = torch.zeros(E + 1, dtype=torch.int32, device="cuda")
    out = (z(0, d), *(torch.full(s, float("nan"), dtype=torch.bfloat16, device="cuda") for s in ((E, f, d), (E, f, d), (E, d, f))))
    L.moe_grouped_gemm_swiglu_bwd(z(0, d), z(0, d), z(0, f), z(0, f), z(0, f), z(E, f, d), z(E, f, d), z(E, d, f), offsets, out=out)
    torch.cuda.synchronize()
    for t in out[1:]:
        assert not to_np(t).any()
