"""GPU parity at rows of millions of columns: a strip's 32-bit offsets (range-checked stores) hold only so many rows of such a width.
Rows of 8.5 MB in every result that has one column per d, per f, and in the fp32 partial tiles of weight gradients (2056 rows on one
expert are two chunks).  The reference is the same arithmetic in fp32 on the GPU: the oracle's fp64 copies would not fit the time."""
import pytest

from tests.util import TOL

pytestmark = pytest.mark.gpu


def _close(got, ref, what):
    """max|got - ref| <= tolerance * max|ref|, a few columns at a time"""
    step = max(1, (1 << 27) // got.shape[0])
    err = max(float((got[:, c:c + step].float() - ref[:, c:c + step]).abs().max()) for c in range(0, got.shape[1], step))
    assert err <= TOL["bf16"] * float(ref.abs().max()), (what, err)


@pytest.mark.parametrize("P,d,f", [(264, 4260104, 264), (264, 264, 4260104), (2056, 2200008, 136)])
def test_rows_of_millions_of_columns(P, d, f):
    import torch
    from paper_2508_02317_amd import libmoe as L
    gen = torch.Generator(device="cuda").manual_seed(P + d)

    def normal(rows, cols, std):
        out = torch.empty((rows, cols), dtype=torch.bfloat16, device="cuda")
        for r in range(0, rows, 32):
            out[r:r + 32] = torch.randn((min(32, rows - r), cols), generator=gen, device="cuda") * std
        return out

    x, dy = normal(P, d, 1.0), normal(P, d, 1.0)
    wg, wu, wd = normal(f, d, d ** -0.5), normal(f, d, d ** -0.5), normal(d, f, d ** -0.5)
    offsets = torch.tensor([0, P], dtype=torch.int32, device="cuda")
    act, yp, g, u = L.moe_grouped_gemm_swiglu_fwd(x, wg[None], wu[None], wd[None], offsets)
    dxp, dwg, dwu, dwd = L.moe_grouped_gemm_swiglu_bwd(dy, x, g, u, act, wg[None], wu[None], wd[None], offsets)
    torch.cuda.synchronize()

    def product(a, b):                                   # a b^T in fp32
        return a.float() @ b.float().t()
    # every stage from the rounded results of the one before, as the library takes them
    G, U = product(x, wg), product(x, wu)
    _close(g, G, "g"); _close(u, U, "u")
    G, U = g.float(), u.float()
    _close(act, torch.nn.functional.silu(G) * U, "act")
    _close(yp, product(act, wd), "yp")
    del yp
    dA = dy.float() @ wd.float()
    s = torch.sigmoid(G)
    dG, dU = dA * U * (s + G * s * (1 - s)), dA * G * s
    del dA, s, G, U
    _close(dwd[0], product(dy.t(), act.t()), "dw_down")
    del dwd
    _close(dwg[0], product(dG.t(), x.t()), "dw_gate")
    _close(dwu[0], product(dU.t(), x.t()), "dw_up")
    del dwg, dwu
    dX = dG @ wg.float()
    dX += dU @ wu.float()
    _close(dxp, dX, "dxp")
