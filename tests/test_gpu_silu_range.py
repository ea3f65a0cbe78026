"""SwiGLU and its derivative over every finite bf16 pre-activation, through the expert products.

One row, one reduction index, one expert: G[j] = w_gate[j, 0], U = 1 and dA = 1 exactly, so that act[j] = silu(G[j]),
dw_up[j, 0] = silu(G[j]) and dw_gate[j, 0] = silu'(G[j]), each rounded to bf16 once.

The bound: one rounding to a significand of 8 bits (2^-8 relative) and the fp32 evaluation before it, whose relative error is at most
|G| 2^-23 from the exponential's argument (1e-5 at |G| = 88.7, beyond which exp(-G) is not a finite float) plus a few 2^-24;
together below 2^-8 (1 + 2^-5).  Two exceptions.  Near its zero at G = -1.278 the two terms of the derivative cancel: 2^-22
absolute on |G + 1.278| < 0.1.  Below -88.7 fp32 has the sigmoid as zero, where |silu| and |silu'| are below 2.6e-37; and
results in the subnormal range have an absolute rounding, far below that."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

REL = 2.0 ** -8 * (1 + 2.0 ** -5)


def _finite_bf16():
    bits = np.arange(1 << 16, dtype=np.uint32) << 16
    v = bits.view(np.float32)
    return v[np.isfinite(v) & ((np.abs(v) >= 2.0 ** -120) | (v == 0.0))]


def _close(got, ref, g, derivative):
    got = got.astype(np.float64)
    tol = REL * np.abs(ref) + np.where(g < -88.7, 2.6e-37, 2.0 ** -126)
    if derivative:
        tol = tol + np.where(np.abs(g + 1.278) < 0.1, 2.0 ** -22, 0.0)
    bad = ~(np.abs(got - ref) <= tol)
    assert not bad.any(), [(float(a), float(b), float(c)) for a, b, c in zip(g[bad][:5], got[bad][:5], ref[bad][:5])]


def _silu(g):
    g = g.astype(np.float64)
    e = np.exp(-np.abs(g))
    s = np.where(g >= 0, 1.0 / (1.0 + e), e / (1.0 + e))
    c = np.where(g >= 0, e / (1.0 + e), 1.0 / (1.0 + e))      # 1 - s
    return g * s, s * (1.0 + g * c)


def _column(g):
    import torch
    w = torch.zeros((1, g.size, 8), dtype=torch.bfloat16, device="cuda")
    w[0, :, 0] = torch.from_numpy(g.copy()).cuda().to(torch.bfloat16)
    return w


# (lowest, highest pre-activation).  Large ones: silu'(G) is 1, also where 1 + G is G in fp32.  Very negative ones: silu(G) is a
# normal number although the sigmoid is a subnormal one, and 0, not G times a smallest number, where exp(-G) is not finite.
@pytest.mark.parametrize("gather", [True, False])
@pytest.mark.parametrize("lo,hi", [(2.0, np.inf), (-16.0, 2.0), (-np.inf, -16.0)])
def test_silu_and_its_derivative(lo, hi, gather):
    import torch
    from paper_2508_02317_amd import libmoe as L
    g = _finite_bf16()
    g = g[(g >= lo) & (g <= hi)]
    g = np.concatenate([g, np.full(-g.size % 8, 2.0, dtype=np.float32)])   # widths are multiples of 8
    f = g.size
    wg, wu = _column(g), _column(np.ones(f, dtype=np.float32))
    wd = torch.zeros((1, 8, f), dtype=torch.bfloat16, device="cuda")
    wd[0, 0] = 1.0
    x = torch.zeros((1, 8), dtype=torch.bfloat16, device="cuda")
    x[0, 0] = 1.0
    offsets = torch.tensor([0, 1], dtype=torch.int32, device="cuda")
    if gather:
        pair, w = torch.zeros(1, dtype=torch.int32, device="cuda"), torch.ones((1, 1), device="cuda")
        act, _, G, U = L.moe_grouped_gemm_swiglu_fwd_gather(x, 1, pair, wg, wu, wd, offsets)
        _, dwg, dwu, _, _ = L.moe_grouped_gemm_swiglu_bwd_gather(x, x, w, pair, G, U, wg, wu, wd, offsets)
    else:
        act, _, G, U = L.moe_grouped_gemm_swiglu_fwd(x, wg, wu, wd, offsets)
        _, dwg, dwu, _ = L.moe_grouped_gemm_swiglu_bwd(x, x, G, U, act, wg, wu, wd, offsets)
    torch.cuda.synchronize()
    assert np.array_equal(G.float().cpu().numpy()[0], g)
    silu, d = _silu(g)
    _close(act.float().cpu().numpy()[0], silu, g, False)
    _close(dwu[0, :, 0].float().cpu().numpy(), silu, g, False)
    _close(dwg[0, :, 0].float().cpu().numpy(), d, g, True)
