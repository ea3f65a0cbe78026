"""What the kernels promise the compiler about the alignment of memory that a caller hands over: tensors and workspaces start at a
multiple of 16 bytes (include/moe.h) and no more, so no access of global or constant memory may claim more (CPU only: hipcc
cross-compiles without a GPU).  An access that claims more works only while the instruction chosen for it needs less.  On the GPU: a
workspace at 16 bytes past a multiple of 32 gives bit for bit what an aligned one gives."""
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2508_02317_amd", "csrc")
PROMISED = 16


def accesses(ir):
    """-> (instruction, alignment) of the loads and stores of LLVM IR that may go to global (1) or constant (4) memory."""
    for line in ir.split("\n"):
        m = re.match(r"\s*(?:%\S+ = )?(?:load|store) .*?ptr(?: addrspace\((\d)\))? [^,]+, align (\d+)", line)
        if m and m[1] in (None, "0", "1", "4"):
            yield line.strip(), int(m[2])


def test_the_scan_sees_a_promise():
    ir = "\n".join(["  %1 = load <8 x i32>, ptr addrspace(4) %0, align 32, !tbaa !5", "  store <4 x i32> %1, ptr addrspace(1) %0, align 16",
                    "  %2 = load <8 x i32>, ptr addrspace(3) %0, align 64", "  %3 = load i32, ptr %0, align 4"])
    assert [a for _, a in accesses(ir)] == [32, 16, 4]


@pytest.mark.parametrize("source", ["gemm_bf16.hip", "gemm_f32.hip", "permute.hip", "route.hip"])
def test_no_access_claims_more_than_the_contract(source, tmp_path):
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("hipcc not available")
    from paper_2508_02317_amd.build import HIPCC_FLAGS
    out = str(tmp_path / "kernels.ll")
    res = subprocess.run([hipcc, *[f for f in HIPCC_FLAGS if f != "-fPIC"], "--cuda-device-only", "-emit-llvm", "-S", os.path.join(CSRC, source),
                          "-o", out], capture_output=True, text=True)
    assert res.returncode == 0, res.stderr[-2000:]
    found = list(accesses(open(out).read()))
    assert len(found) > 50
    over = [(line, a) for line, a in found if a > PROMISED]
    assert not over, "%d accesses, the first: %s" % (len(over), over[0][0])


def _at_16(ws):
    """A workspace of the same size that starts 16 bytes past a multiple of 32."""
    import torch
    whole = torch.empty(ws.numel() + 48, dtype=torch.uint8, device="cuda")
    first = (16 - whole.data_ptr()) % 32
    out = whole[first:first + ws.numel()]
    assert out.data_ptr() % 32 == 16 and out.numel() == ws.numel()
    return out


# rows per expert that take the 256-row tiles and the 128-row tiles, and full precision
@pytest.mark.gpu
@pytest.mark.parametrize("T,E,dtype", [(1100, 8, "bf16"), (300, 16, "bf16"), (150, 8, "f32")])
@pytest.mark.parametrize("gather", [True, False])
def test_steps_on_a_workspace_at_16_bytes(T, E, dtype, gather):
    import torch
    from paper_2508_02317_amd.layer import MoELayer
    from tests.util import torch_dtype
    print("T=%d E=%d %s gather=%s" % (T, E, dtype, gather), flush=True)
    d, f, k, dt = 264, 136, 2, torch_dtype(dtype)
    gen = torch.Generator(device="cuda").manual_seed(T)
    mk = lambda *s: (torch.randn(s, generator=gen, device="cuda") * 0.1).to(dt)
    layer = MoELayer(T, d, E, k, f, dt, mk(E, f, d), mk(E, f, d), mk(E, d, f), save_gu=False, gather=gather, w_router=mk(E, d))
    x, dy = mk(T, d), mk(T, d)
    aligned, results = layer.ws, []
    for ws in (aligned, _at_16(aligned)):
        layer.ws = ws
        layer.forward(x)
        layer.backward(dy)
        results.append([t.clone() for t in (layer.y, layer.dx, layer.dw_gate, layer.dw_up, layer.dw_down, layer.dw, layer.dw_router)])
    torch.cuda.synchronize()
    for a, b in zip(*results):
        assert torch.equal(a, b) and bool(a.float().abs().max() > 0)


@pytest.mark.gpu
def test_the_8_bit_forward_on_a_workspace_at_16_bytes():
    import torch
    from paper_2508_02317_amd import libmoe as L
    T, E, d, f = 1100, 4, 256, 128
    gen = torch.Generator(device="cuda").manual_seed(1)
    quantised = lambda *s: L.moe_mx8_quantise(torch.randn(s, generator=gen, device="cuda").bfloat16())
    x, weights = quantised(T, d), [t for q in (quantised(E, f, d), quantised(E, f, d), quantised(E, d, f)) for t in q]
    offsets = torch.tensor([0, 300, 300, 813, T], dtype=torch.int32, device="cuda")
    ws = torch.empty(L.lib.moe_grouped_gemm_swiglu_fwd_mx8_workspace_bytes(T, d, f, E), dtype=torch.uint8, device="cuda")
    results = [L.moe_grouped_gemm_swiglu_fwd_mx8(*x, *weights, offsets, ws=w) for w in (ws, _at_16(ws))]
    torch.cuda.synchronize()
    for a, b in zip(*results):
        assert torch.equal(a, b)
