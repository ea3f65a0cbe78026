"""The grouped-GEMM kernels read their MFMA operands from LDS with assembly statements (so that the compiler does
not order them behind every outstanding direct global->LDS load).  Such a read delivers asynchronously; the kernels
name the destination registers as operands of the wait that follows, so the compiler must keep them untouched until
then.  This test compiles the kernels to assembly and checks exactly that, instruction by instruction: between an
assembly LDS read and the wait for the LDS counter that retires it, nothing reads, copies, spills or overwrites its destination
registers -- line by line, and along every path through a kernel's branches, the back edges of its loops among them: a slab leaves
with the reads of the next one in flight (CPU only: hipcc cross-compiles without a GPU)."""
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2508_02317_amd", "csrc")


def _regs(text):
    regs = [int(x) for x in re.findall(r"\bv(\d+)\b", text)]
    for a, b in re.findall(r"v\[(\d+):(\d+)\]", text):
        regs += list(range(int(a), int(b) + 1))
    return regs


def scan_kernel(lines):
    """-> list of (line number, instruction, what) for every touch of a pending destination.
    LDS reads of a wave complete in order: a wait for the counter to drop to N retires all but the last N reads."""
    pending, bad, in_asm, order = {}, [], False, []          # order: destination register lists of the reads in flight
    vm_order = []                                            # the same for vector-memory instructions (most have no tracked destination)
    for i, line in enumerate(lines):
        if "#ASMSTART" in line:
            in_asm = True
            continue
        if "#ASMEND" in line:
            in_asm = False
            continue
        st = line.strip()
        m = in_asm and re.match(r"ds_read_b(?:64_tr_b16|128) v\[(\d+):(\d+)\]", st)
        if m:
            dst = list(range(int(m.group(1)), int(m.group(2)) + 1))
            for r in dst:
                if r in pending:
                    bad.append((i, st, "overwrites a pending destination"))
                pending[r] = i
            order.append(dst)
            continue
        # a scale word requested by an assembly statement: pending until a wait for the vector-memory counter retires it
        # (vector-memory instructions complete in order; every one of them counts)
        m = in_asm and re.match(r"global_load_dword v(\d+),", st)
        if m:
            r = int(m.group(1))
            if r in pending:
                bad.append((i, st, "overwrites a pending destination"))
            pending[r] = i
            vm_order.append([r])
            continue
        if re.match(r"(global|scratch|buffer|flat)_(load|store|atomic)", st):
            if any(r in pending for r in _regs(st)):
                bad.append((i, st, "touches a pending destination"))
            vm_order.append([])
            continue
        w = st.startswith("s_waitcnt") and re.search(r"vmcnt\((\d+)\)", st)
        if w:
            keep = int(w.group(1))
            while len(vm_order) > keep:
                for r in vm_order.pop(0):
                    pending.pop(r, None)
        w = st.startswith("s_waitcnt") and re.search(r"lgkmcnt\((\d+)\)", st)
        if w:
            keep = int(w.group(1))
            while len(order) > keep:
                for r in order.pop(0):
                    pending.pop(r, None)
            continue
        if re.match(r"s_branch\b", st) or st.startswith("s_endpgm"):
            pending, order, vm_order = {}, [], []      # what follows is reached from elsewhere
            continue
        if not st or st[0] in ";." or st.startswith("s_") or st.endswith(":"):
            continue
        if any(r in pending for r in _regs(st)):
            bad.append((i, st, "touches a pending destination"))
    return bad


def _blocks(lines):
    """-> list of (instructions, indices of the blocks that may follow); an instruction is (line number, in assembly statement, text)"""
    blocks, labels, cur, in_asm = [], {}, [], False
    for i, line in enumerate(lines):
        m = re.match(r"(\.LBB\w+):", line)
        if m:
            if cur:
                blocks.append((cur, ["next"]))
                cur = []
            labels[m.group(1)] = len(blocks)
            continue
        if "#ASMSTART" in line or "#ASMEND" in line:
            in_asm = "#ASMSTART" in line
            continue
        st = line.split(";")[0].strip()
        if not st or st[0] == "." or st.endswith(":"):
            continue
        cur.append((i, in_asm, st))
        m = re.match(r"s_(c?)branch\w*\s+(\.LBB\w+)", st)
        if m or st.startswith("s_endpgm"):
            blocks.append((cur, (["next"] if m.group(1) else []) + [m.group(2)] if m else []))
            cur = []
    if cur:
        blocks.append((cur, []))
    return [(ins, [k + 1 if n == "next" else labels[n] for n in follow]) for k, (ins, follow) in enumerate(blocks)]


def _through(ins, lds, vm, bad):
    """One block.  lds, vm: register -> how many younger reads (vector-memory instructions) there are at least, for what is in flight."""
    lds, vm = dict(lds), dict(vm)
    for i, in_asm, st in ins:
        m = in_asm and re.match(r"(ds_read_b(?:64_tr_b16|128) v\[(\d+):(\d+)\]|global_load_dword v(\d+)),", st)
        if m:
            dst = range(int(m.group(2)), int(m.group(3)) + 1) if m.group(2) else [int(m.group(4))]
            if any(r in lds or r in vm for r in dst):
                bad.add((i, st, "overwrites a pending destination"))
            flight = lds if m.group(2) else vm
            for r in flight:
                flight[r] = min(flight[r] + 1, 63)
            flight.update((r, 0) for r in dst)
            continue
        if st.startswith("s_waitcnt"):
            w = re.search(r"vmcnt\((\d+)\)", st)
            vm = {r: n for r, n in vm.items() if n < int(w.group(1))} if w else vm
            w = re.search(r"lgkmcnt\((\d+)\)", st)
            lds = {r: n for r, n in lds.items() if n < int(w.group(1))} if w else lds
            continue
        if st.startswith("s_"):
            continue
        if (lds or vm) and any(r in lds or r in vm for r in _regs(st)):
            bad.add((i, st, "touches a pending destination"))
        if re.match(r"(global|scratch|buffer|flat)_(load|store|atomic)", st):
            vm = {r: min(n + 1, 63) for r, n in vm.items()}
    return lds, vm


def scan_paths(lines):
    """The same as scan_kernel along every path: what is in flight at a block's entry is whatever any block before it leaves.
    One kind of path is left out: a wave with reads in flight does not go round the wait that ends a tile (that branch is for waves
    without rows, which issue no reads)."""
    blocks, bad = _blocks(lines), set()
    entry, todo = {0: ({}, {})}, [0]
    while todo:
        b = todo.pop()
        out = _through(blocks[b][0], *entry[b], bad)
        for t in blocks[b][1]:
            if t >= len(blocks):
                continue
            other = [n for n in blocks[b][1] if n != t]
            if out[0] and other and other[0] < len(blocks):
                ins, follow = blocks[other[0]]
                if ins and ins[0][1] and ins[0][2].startswith("s_waitcnt lgkmcnt(0)") and follow == [t]:
                    continue
            old = entry.get(t, ({}, {}))
            new = tuple({r: min(n.get(r, 63), o.get(r, 63)) for r in {**n, **o}} for n, o in zip(out, old))
            if t not in entry or new != old:
                entry[t] = new
                todo.append(t)
    return sorted(bad)


def test_paths_see_a_hazard_over_a_back_edge():
    read = ["\t;;#ASMSTART", "\tds_read_b128 v[10:13], v1 offset:64", "\t;;#ASMEND"]
    wait = ["\t;;#ASMSTART", "\ts_waitcnt lgkmcnt(0)", "\t;;#ASMEND"]
    loop = lambda top: [".LBB0_1:", *top, *wait, "\tv_mov_b32_e32 v5, v10", *read, "\ts_cbranch_scc1 .LBB0_1", *wait, "\ts_endpgm"]
    assert scan_paths(read + loop([])) == []
    late = read + loop(["\tv_add_u32_e32 v11, v2, v3"])                    # in flight from the round before
    assert len(scan_paths(late)) == 1
    kernel = loop(["\tv_add_u32_e32 v11, v2, v3"])
    assert len(scan_paths(kernel)) == 1 and scan_kernel(kernel) == []       # line by line nothing is pending there yet
    # a block reached over an unconditional branch, and a counted wait that leaves one read in flight
    away = [*read, "\t;;#ASMSTART", "\tds_read_b128 v[14:17], v1", "\t;;#ASMEND", "\t;;#ASMSTART", "\ts_waitcnt lgkmcnt(1)", "\t;;#ASMEND", "\ts_branch .LBB0_3",
            ".LBB0_2:", "\ts_endpgm", ".LBB0_3:", "\tv_mov_b32_e32 v5, v10", "\tv_mov_b32_e32 v6, v14", "\ts_branch .LBB0_2"]
    assert [st for _, st, _ in scan_paths(away)] == ["v_mov_b32_e32 v6, v14"]


def test_scanner_sees_a_planted_hazard():
    good = ["\t;;#ASMSTART", "\tds_read_b128 v[10:13], v1 offset:64", "\t;;#ASMEND", "\tv_add_u32_e32 v2, v3, v4",
            "\ts_waitcnt lgkmcnt(0)", "\tv_mov_b32_e32 v5, v10"]
    assert scan_kernel(good) == []
    copied = good[:3] + ["\tv_mov_b32_e32 v20, v11"] + good[3:]
    assert len(scan_kernel(copied)) == 1
    spilled = good[:3] + ["\tscratch_store_dwordx4 off, v[10:13], off offset:16"] + good[3:]
    assert len(scan_kernel(spilled)) == 1
    clobbered = good[:3] + ["\t;;#ASMSTART", "\tds_read_b64_tr_b16 v[12:13], v1", "\t;;#ASMEND"] + good[3:]
    assert len(scan_kernel(clobbered)) == 2
    # partial waits: two reads in flight, a wait for all but one retires the first only
    two = ["\t;;#ASMSTART", "\tds_read_b128 v[10:13], v1", "\t;;#ASMEND", "\t;;#ASMSTART", "\tds_read_b128 v[14:17], v1 offset:16", "\t;;#ASMEND",
           "\t;;#ASMSTART", "\ts_waitcnt lgkmcnt(1)", "\t;;#ASMEND"]
    assert scan_kernel(two + ["\tv_mov_b32_e32 v5, v10"]) == []
    assert len(scan_kernel(two + ["\tv_mov_b32_e32 v5, v14"])) == 1
    # a requested word followed by two younger loads: a wait for all but two retires it, a wait for all but three does not
    word = ["\t;;#ASMSTART", "\tglobal_load_dword v7, v1, s[2:3]", "\t;;#ASMEND", "\tglobal_load_lds_dwordx4 v[2:3], off",
            "\tglobal_load_lds_dwordx4 v[4:5], off"]
    assert scan_kernel(word + ["\ts_waitcnt vmcnt(2)", "\tv_lshrrev_b32_e32 v8, v9, v7"]) == []
    assert len(scan_kernel(word + ["\ts_waitcnt vmcnt(3)", "\tv_lshrrev_b32_e32 v8, v9, v7"])) == 1


@pytest.fixture(scope="module")
def assembly(tmp_path_factory):
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("hipcc not available")
    from paper_2508_02317_amd.build import HIPCC_FLAGS
    out = str(tmp_path_factory.mktemp("asm") / "gemm_bf16.s")
    flags = [f for f in HIPCC_FLAGS if f != "-fPIC"]
    res = subprocess.run([hipcc, *flags, "--cuda-device-only", "-S", os.path.join(CSRC, "gemm_bf16.hip"), "-o", out],
                         capture_output=True, text=True)
    assert res.returncode == 0, res.stderr[-2000:]
    return open(out).read()


def _is_product(name):
    return any(k in name for k in ("row_grouped_kernel", "wgrad_kernel", "mx8_row_kernel"))


def _products(assembly):
    return [n for n in re.findall(r"\.amdhsa_kernel (\S+)", assembly) if _is_product(n)]


def test_no_instruction_touches_a_pending_lds_read(assembly):
    kernels = re.split(r"\n(?=_ZN3moe[^\n]*:\s*;\s*@)", assembly)
    checked = 0
    for k in kernels:
        name = k.split(":")[0]
        if not _is_product(name):
            continue
        lines = k.split("\n")
        n_reads = sum(1 for l in lines if re.match(r"\s*ds_read_b(?:64_tr_b16|128) ", l))
        assert n_reads > 0, name
        for bad in (scan_kernel(lines), scan_paths(lines[1:])):
            assert not bad, "%s: %s" % (name, bad[:5])
        checked += 1
    assert checked == len(_products(assembly)) >= 34


def test_products_keep_nothing_in_scratch_memory(assembly):
    """Accumulators, fragments and addresses fill the register file; a value that does not fit is reloaded for every tile or slab,
    behind a wait for all outstanding loads, which drains the rings."""
    checked = 0
    for k in re.split(r"\n  - ", assembly[assembly.index("amdhsa.kernels"):]):
        name = re.search(r"\.name:\s*(\S+)", k)
        if name is None or not _is_product(name[1]):
            continue
        for field in ("private_segment_fixed_size", "vgpr_spill_count"):
            assert int(re.search(r"\.%s:\s*(\d+)" % field, k)[1]) == 0, (field, name[1])
        checked += 1
    assert checked == len(_products(assembly))


def test_much_8_bit_activation_is_stored_through_the_l2(assembly):
    """A wave stores 32 bytes of a line of activation codes: with non-temporal stores each piece is a write to memory of its own.  The
    variants for many codes must not have them (the last template argument), the others do."""
    kernels = [k for k in re.split(r"\n(?=_ZN3moe[^\n]*:\s*;\s*@)", assembly) if re.match(r"\S*mx8_row_kernelILi0E", k)]
    assert len(kernels) == 4
    for k in kernels:
        stores = re.findall(r"buffer_store_dwordx4 [^\n]*", k)
        through_l2 = re.match(r"\S*mx8_row_kernelILi0E\S*Lb1EEEvNS", k) is not None
        assert stores and all((re.search(r"\bnt\b", st) is None) == through_l2 for st in stores), k.split(":")[0]
