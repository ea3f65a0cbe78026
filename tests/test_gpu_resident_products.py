"""GPU parity where a workgroup of the products takes several tiles in a row: the loads of the next tile run behind the slabs of
the current one, so what can go wrong lies where one tile hands over to the next -- reductions of less than a slab, of one, two and
three slabs (64 indices; 128 for 8-bit operands), with a partial last one, between tiles of full, few and no rows; more than 256
tiles (one workgroup per CU) of 256 x 256 or 512 of 128 x 128.  Each test names the products for which its sizes reach that and counts
their tiles.

Bounds: those of every bf16 product and every router product (operands rounded to 8 bits, fp32 accumulation, one rounding)."""
import numpy as np
import pytest

from oracle import moe_oracle as O
from paper_2508_02317_amd.inputs import quantise
from tests.test_gpu_mx8 import _case, _compare_forward
from tests.util import assert_close, q, to_dev, to_np, torch_dtype

pytestmark = pytest.mark.gpu


def _tiles(counts, d, f, bm=256):
    """tiles of each product of bm x bm (gate/up: half gate, half up columns), given the rows of each expert; the weight gradients' are
    always 256 x 256, one set per chunk of at most 2048 rows (T <= 65536) of an expert"""
    up = lambda a, b: -(-a // b)
    rows, items = sum(up(int(c), bm) for c in counts), sum(up(int(c), 2048) for c in counts)
    return {"gate_up": rows * up(f, bm // 2), "down": rows * up(d, bm), "dact": rows * up(f, bm), "dx": rows * up(d, bm),
            "dw_down": items * up(d, 256) * up(f, 256), "dw_gate_up": items * up(2 * f, 256) * up(d, 256)}


def _assert_several_tiles(counts, d, f, products, bm=256):
    n = _tiles(counts, d, f, bm)
    for name in products:
        assert n[name] > (512 if bm == 128 and not name.startswith("dw") else 256), (name, n[name])


def _layer_against_oracle(T, d, E, k, f, logits, gather, save_gu, several=(), bm=256):
    import torch
    from paper_2508_02317_amd.layer import MoELayer
    r = np.random.default_rng(T + d + f)
    X, dY = q(r.standard_normal((T, d)), "bf16"), q(r.standard_normal((T, d)), "bf16")
    Wg, Wu = (q(r.standard_normal((E, f, d)) * 0.05, "bf16") for _ in range(2))
    Wd = q(r.standard_normal((E, d, f)) * 0.05, "bf16")
    fwd = O.moe_layer_fwd(X, logits, Wg, Wu, Wd, k)
    _assert_several_tiles(np.bincount(fwd["topk_idx"].reshape(-1), minlength=E), d, f, several, bm)
    bwd = O.moe_layer_bwd(fwd, dY, logits, Wg, Wu, Wd)
    layer = MoELayer(T, d, E, k, f, torch_dtype("bf16"), to_dev(Wg, "bf16"), to_dev(Wu, "bf16"), to_dev(Wd, "bf16"), gather=gather, save_gu=save_gu)
    z = to_dev(logits)
    for _ in range(2):                                   # the second call finds what the first left in the workspace
        layer.forward(to_dev(X, "bf16"), logits=z)
        layer.backward(to_dev(dY, "bf16"), logits=z)
    torch.cuda.synchronize()
    for name, got, ref in (("Y", layer.y, fwd["Y"]), ("dX", layer.dx, bwd["dX"]), ("dWg", layer.dw_gate, bwd["dWg"]),
                           ("dWu", layer.dw_up, bwd["dWu"]), ("dWd", layer.dw_down, bwd["dWd"])):
        assert_close(to_np(got), ref, "bf16", name)


def _uneven_logits(T, E, seed):
    """every fifth expert without rows, every seventh with a few, the others alike"""
    z = np.random.default_rng(seed).standard_normal((T, E)).astype(np.float32)
    z[:, ::5] -= 30.0
    z[:, 3::7] -= 3.0
    return z


# (d, f) are reduction lengths of one product and widths of another: 40 and 56 less than a slab, 64 one, 72 and 120 a slab and a
# part, 128 two, 136 two and a part, 200 three and a part; f = 1032 has more than 16 partial sums of a combine weight per row.
@pytest.mark.parametrize("gather,save_gu", [(True, True), (True, False), (False, True)])
@pytest.mark.parametrize("T,E,d,f", [(16000, 64, 40, 520), (16000, 64, 520, 56), (15000, 60, 64, 392), (12000, 40, 392, 120), (16000, 64, 72, 264),
                                     (12000, 40, 136, 128), (9000, 24, 200, 1032),        # 256 x 256 tiles
                                     (5000, 128, 40, 520), (5000, 128, 520, 72), (9000, 128, 128, 392)])   # 128 x 128 tiles
def test_short_reductions(T, E, d, f, gather, save_gu):
    """(Most of these sizes give some of the products several tiles, the tests below all of them.)"""
    _layer_against_oracle(T, d, E, 1, f, _uneven_logits(T, E, T + E), gather, save_gu)


# every reduction length with more than 256 tiles of 256 x 256: d for gate/up and dA, f for down and (two segments) dX
@pytest.mark.parametrize("gather,save_gu", [(True, True), (False, False)])
@pytest.mark.parametrize("K", [40, 64, 72, 128, 136, 200])
def test_many_large_tiles_per_workgroup(K, gather, save_gu):
    T, E, wide = 11200, 40, 2312
    z = _uneven_logits(T, E, K)
    _layer_against_oracle(T, K, E, 1, wide, z, gather, save_gu, ("gate_up", "dact", "dw_down", "dw_gate_up"))
    _layer_against_oracle(T, wide, E, 1, K, z, gather, save_gu, ("down", "dx", "dw_down", "dw_gate_up"))


# more than 512 tiles of 128 x 128: few rows per expert, and for dX few experts as well (its tile is the small one only then)
@pytest.mark.parametrize("gather,save_gu", [(True, True), (False, False)])
@pytest.mark.parametrize("T,E,d,f,several", [(3800, 64, 40, 2312, ("gate_up", "dact")), (3800, 64, 136, 2312, ("gate_up", "dact")),
                                             (3800, 64, 2312, 40, ("down",)), (3800, 64, 2312, 136, ("down",)),
                                             (12700, 100, 512, 40, ("down", "dx")), (12700, 100, 512, 136, ("down", "dx"))])
def test_many_small_tiles_per_workgroup(T, E, d, f, several, gather, save_gu):
    _layer_against_oracle(T, d, E, 1, f, _uneven_logits(T, E, T + f), gather, save_gu, several, bm=128)


@pytest.mark.parametrize("gather", [True, False])
@pytest.mark.parametrize("T,k", [(14000, 1), (9000, 2)])
def test_weight_gradients_of_experts_of_many_chunks(T, k, gather):
    """Two thirds of the rows on one expert: its chunks of 2048 rows meet in the fp32 partial tiles (more than four, and a rest)."""
    z = np.random.default_rng(T).standard_normal((T, 6)).astype(np.float32)
    z[:, 2] += 3.0
    z[:, 4] -= 30.0
    _layer_against_oracle(T, 136, 6, k, 264, z, gather, True)


@pytest.mark.parametrize("gather", [True, False])
def test_partial_tiles_followed_by_other_tiles(gather):
    """The same with more tiles than workgroups: a workgroup stores a partial tile in one round and goes on to a tile of another chunk."""
    z = np.random.default_rng(3).standard_normal((14000, 6)).astype(np.float32)
    z[:, 2] += 3.0
    z[:, 4] -= 30.0
    _layer_against_oracle(14000, 1288, 6, 1, 1032, z, gather, True, ("dw_down", "dw_gate_up"))


@pytest.mark.parametrize("T", [2047, 2048, 2049])
def test_gate_up_stores_at_the_line_of_many_rows(T):
    """256 rows per expert on average decide how gate, up and activation are stored (E = 8)."""
    _layer_against_oracle(T, 72, 8, 1, 264, _uneven_logits(T, 8, T), True, True)


# 512 tiles of 128 x 128 decide the tile of dX; chunks of 256 rows up to T = 16384 and more than eight of them in dW.  T = 16384, d = 1288:
# 384 large tiles of dX (reductions of one slab, two and one, two) and of dW; T = 33000: 516 tiles of the logits (512 run at once)
@pytest.mark.parametrize("accumulate", [True, False])
@pytest.mark.parametrize("T,d,E", [(256, 136, 8), (257, 1032, 64), (8192, 1024, 16), (8193, 1024, 16), (16500, 264, 128),
                                   (16384, 1288, 8), (16384, 1288, 72), (16384, 1288, 128), (33000, 72, 128)])
def test_router_backward_where_tiles_and_chunks_change(T, d, E, accumulate):
    from paper_2508_02317_amd import libmoe as L
    r = np.random.default_rng(T + d)
    X, Wr = q(r.standard_normal((T, d)), "bf16"), q(r.standard_normal((E, d)) * 0.05, "bf16")
    dz = r.standard_normal((T, E)).astype(np.float32)
    rdX, rdW = O.router_bwd(quantise(dz, "bf16"), X, Wr)
    base = q(r.standard_normal((T, d)), "bf16") if accumulate else np.zeros((T, d), np.float32)
    dx, dw = L.moe_router_bwd(to_dev(dz), to_dev(X, "bf16"), to_dev(Wr, "bf16"), dx=to_dev(base, "bf16") if accumulate else None)
    assert_close(to_np(dx), base.astype(np.float64) + rdX, "bf16", "dx")
    assert_close(to_np(dw), rdW, "bf16", "dw")
    assert_close(to_np(L.moe_router_logits(to_dev(X, "bf16"), to_dev(Wr, "bf16"))), O.router_logits(X, Wr), "bf16", "logits", tol=1e-5)


# one, two and three slabs of 128 indices, more than 256 tiles of the first product (d) and of the second (f), experts of few rows; and
# activation codes of more than 32 MiB, which are stored another way
@pytest.mark.parametrize("T,d,E,f,product", [(5200, 128, 64, 768, "gate_up"), (5200, 256, 64, 768, "gate_up"), (5200, 384, 64, 768, "gate_up"),
                                             (5200, 1280, 64, 128, "down"), (5200, 1280, 64, 256, "down"), (5200, 1280, 64, 384, "down"),
                                             (16400, 128, 32, 2048, "gate_up")])
def test_8_bit_products_of_many_tiles_per_workgroup(T, d, E, f, product):
    cfg, inp, offsets, pair_of_row = _case(T, d, E, 1, f, T + d)
    _assert_several_tiles(np.diff(offsets), d, f, (product,))
    a = _compare_forward(cfg, inp, offsets, pair_of_row, gather=False)
    b = _compare_forward(cfg, inp, offsets, pair_of_row, gather=True)
    for x, y in zip(a, b):
        assert np.array_equal(x, y)
