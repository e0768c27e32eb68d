"""What the compiled device code of the library must hold whatever its inputs: read off the code objects
that were built from this tree's sources (their disassembly), on the CPU."""
from __future__ import annotations

import os
import re
import shutil
import subprocess

import pytest

from paper_2412_17560_amd import binding

LLVM = "/opt/rocm/llvm/bin"
pytestmark = pytest.mark.skipif(not os.path.exists(os.path.join(LLVM, "llvm-objdump")), reason="no llvm-objdump here")


@pytest.fixture(scope="module")
def code_objects(tmp_path_factory):
    """The gfx950 code objects in the built library, as files."""
    binding._lib()                                     # (builds it if nothing is built)
    d = tmp_path_factory.mktemp("code")
    shutil.copy(binding.library_path(), d / "lib.so")
    subprocess.run([f"{LLVM}/llvm-objdump", "--offloading", "lib.so"], cwd=d, check=True, capture_output=True)
    files = [d / f for f in os.listdir(d) if f.endswith("gfx950")]
    if not files:
        pytest.skip("a library without device code")
    return files


def _kernels(code_object, part_of_name):
    """(name, [(address, mnemonic, operands, comment)]) of every kernel whose name has the part."""
    text = subprocess.run([f"{LLVM}/llvm-objdump", "-d", "--no-show-raw-insn", str(code_object)], check=True,
                          capture_output=True, text=True).stdout
    for body in re.split(r"\n(?=[0-9a-f]+ <)", text):
        head = re.match(r"[0-9a-f]+ <(\S+)>:", body)
        if head and part_of_name in head[1]:
            lines = re.findall(r"^\s+(\S+)[ \t]*(.*?)\s*// ([0-9A-F]+):(.*)$", body, re.M)
            yield head[1], [(int(a, 16), op, args, rest) for op, args, a, rest in lines]


def _loads_into_lds_with_reads_outstanding(code):
    """Addresses of the loads from global memory into LDS that some path reaches with reads of LDS still under way:
    (LDS reads possibly outstanding, scalar loads possibly outstanding) carried along every path to a fixed
    point.  LDS operations return in order, so a wait for n leaves at most n of them -- unless scalar
    loads, which share the counter and return out of order, are outstanding too: then only a wait for 0 counts."""
    place = {a: i for i, (a, *_) in enumerate(code)}
    seen, todo, found = {}, [(0, (0, 0))], set()
    while todo:
        i, state = todo.pop()
        while i < len(code):
            if i in seen:
                merged = tuple(map(max, seen[i], state))
                if merged == seen[i]:
                    break
                state = merged
            seen[i] = state
            reads, scalar = state
            address, op, args, rest = code[i]
            if op.startswith("ds_read"):
                reads = min(reads + 1, 64)
            elif op.startswith(("s_load", "s_buffer_load")):
                scalar = 1
            elif op == "s_waitcnt" and (n := re.search(r"lgkmcnt\((\d+)\)", args)):
                if int(n[1]) == 0:
                    reads = scalar = 0
                elif not scalar:
                    reads = min(reads, int(n[1]))
            elif "load_lds" in op and reads:
                found.add(address)
            state = (reads, scalar)
            if op == "s_endpgm":
                break
            if op == "s_branch" or op.startswith("s_cbranch"):
                target = re.search(r"<[^>]*?(?:\+0x([0-9a-f]+))?>", rest)
                to = place[code[0][0] + int(target[1] or "0", 16)]
                if op != "s_branch":
                    todo.append((i + 1, state))
                i = to
            else:
                i += 1
    return found


def test_the_check_itself_sees_a_missing_wait():
    def at(*ops):
        return [(4 * i, op, args, rest) for i, (op, args, rest) in enumerate(ops)]
    read, load, end = ("ds_read_b96", "v[0:2], v3", ""), ("global_load_lds_dwordx4", "v[4:5], off", ""), ("s_endpgm", "", "")
    assert _loads_into_lds_with_reads_outstanding(at(read, load, end)) == {4}
    assert not _loads_into_lds_with_reads_outstanding(at(read, ("s_waitcnt", "lgkmcnt(0)", ""), load, end))
    assert _loads_into_lds_with_reads_outstanding(at(read, read, ("s_waitcnt", "lgkmcnt(1)", ""), load, end)) == {12}
    # round a loop: the load at its top follows the read at its end
    assert _loads_into_lds_with_reads_outstanding(at(load, read, ("s_cbranch_scc1", "", " <k>"), end)) == {0}


def test_panel_kernels_wait_for_their_lds_reads_before_staging_over_them(code_objects):
    """The panel kernels (of one matrix and of several: gqsa_panel_kernel, gqsa_panel_multi_kernel) stage a unit's records by
    loads from global memory straight into LDS, over the records of the panels, quad or unit before.  In no
    compiled form may such a load be reached while reads of those are outstanding."""
    checked, found = set(), {}
    for f in code_objects:
        for name, code in _kernels(f, "gqsa_panel_"):
            assert any("load_lds" in c[1] for c in code), name
            checked.add(re.search(r"gqsa_panel\w*?kernelI\w*?ELNS0_4RowsE\d", name)[0])
            if late := _loads_into_lds_with_reads_outstanding(code):
                found[name] = len(late)
    assert len(checked) == 90 and sum("multi" in name for name in checked) == 40
    assert not found


def _wait_states(op, args):
    return int(args, 0) + 1 if op == "s_nop" else 1


def _hand_issued_loads(code):
    """(address, wait states that its own statement puts ahead of it) of every load into LDS that is issued under lanes switched by hand:
    s_mov_b64 save, exec; s_mov_b64 exec, lanes; s_nop n; the load.  (The compiler switches lanes with s_and_saveexec_b64.)"""
    for i, (address, op, args, _) in enumerate(code):
        if "load_lds" not in op:
            continue
        first = i
        while code[first - 1][1] == "s_nop" or (code[first - 1][1] == "s_mov_b64" and "exec" in code[first - 1][2]):
            first -= 1
        if any(c[1] == "s_mov_b64" and c[2].startswith("exec") for c in code[first:i]):
            yield address, sum(_wait_states(c[1], c[2]) for c in code[first:i])


def test_hand_issued_copies_bring_the_wait_states_of_their_address(code_objects):
    """A vector-memory instruction may read scalar registers that a vector instruction (v_readlane) wrote only five wait states
    later.  The compiler does not look inside a statement of assembly, so what it happens to put ahead of one says nothing
    about the next build: the statement has to bring all five."""
    def at(*ops):
        return [(4 * i, op, args, "") for i, (op, args) in enumerate(ops)]
    short = [("v_readlane_b32", "s4, v1, 0"), ("s_mov_b64", "s[8:9], exec"), ("s_mov_b64", "exec, s[10:11]"), ("global_load_lds_dwordx4", "v2, s[4:5]")]
    assert list(_hand_issued_loads(at(*short))) == [(12, 2)]
    assert list(_hand_issued_loads(at(*short[:3], ("s_nop", "2"), short[3]))) == [(16, 5)]
    assert not list(_hand_issued_loads(at(("s_and_saveexec_b64", "s[8:9], vcc"), short[3])))
    loads, late = 0, {}
    for f in code_objects:
        for name, code in _kernels(f, "gqsa_panel_"):
            found = list(_hand_issued_loads(code))
            loads += len(found)
            if any(states < 5 for _, states in found):
                late[name] = min(states for _, states in found)
    assert loads > 0
    assert not late


def test_sums_of_8_bit_codes_lie_apart_where_that_is_faster(code_objects):
    """A kernel for 4 or 8 rows reads four rows' sums of a slot at once (16 bytes) unless every row keeps its own (4 bytes each): with
    8-bit codes in the format's own tiles 8 rows do, and 4 rows of K > 8192, unpruned of K > 4096: 4096x11008 took 20.4 us, not 18.8."""
    apart = set()
    for f in code_objects:
        for name, code in _kernels(f, "gqsa_gemv_kernel"):
            form = re.search(r"FmtILi(\d+)ELi(\d+)ELi(\d+)ELb(\d)EEELi(\d+)ELi(\d+)E", name)
            bits, chunks, blocks, spread, slots, rows = map(int, form.groups())
            if rows >= 4 and chunks >= 1 and any(c[1].startswith(("ds_read_b32", "ds_read2")) for c in code):
                apart.add((bits, chunks, blocks, spread, slots, rows))
    assert apart == ({(8, 1, 0, spread, slots, 8) for spread in (0, 1) for slots in (256, 512)}
                     | {(8, 1, 0, spread, slots, 4) for spread in (0, 1) for slots in (768, 1024)} | {(8, 1, 0, 1, 512, 4)})


def test_form_for_one_panel_is_compiled_for_one(code_objects):
    """The form that turns the activations takes one matrix of one panel a workgroup (its code is the 1 of the last parameter): 16 columns' products with
    4-bit codes, 8 with 8-bit ones -- twice where the zeros are any -- and none for panels that never come."""
    checked = 0
    for f in code_objects:
        for name, code in _kernels(f, "gqsa_panel_kernel"):
            form = re.search(r"kernelILi(\d)ELi\dELb(\d)ELi16ELi1ELNS0_4RowsE1", name)
            if form:
                checked += 1
                products = {"4": 16, "8": 8}[form[1]] * (1 if form[2] == "1" else 2)
                assert sum(op.startswith("v_mfma") for _, op, *_ in code) == products, name
    assert checked == 14


def _spills_among_products(code):
    """Addresses of the accesses to private memory between a kernel's first and last matrix product."""
    products = [i for i, (_, op, *_) in enumerate(code) if op.startswith("v_mfma")]
    return [a for a, op, *_ in code[products[0]:products[-1]] if op.startswith("scratch_")] if products else []


def test_panel_kernels_keep_their_sums_in_registers(code_objects):
    """A panel kernel that runs out of registers loads, awaits and stores a spilled sum at every column of the panel it belongs to: three sums
    of the eighth panel in a joint launch of 9 to 16 rows took 2 x 16384x4096 W4 from 26 to 32 us, 39 registers of another form cost 3 to 17 %,
    a header word per panel 2 to 3 %.  None may lie in memory between the first product and the last."""
    def at(*ops):
        return [(4 * i, op, "", "") for i, op in enumerate(ops)]
    assert _spills_among_products(at("scratch_store_dword", "v_mfma_f32", "scratch_load_dword", "v_mfma_f32", "scratch_load_dword")) == [8]
    spilled = {}
    for f in code_objects:
        for name, code in _kernels(f, "gqsa_panel_"):
            if found := _spills_among_products(code):
                spilled[name] = len(found)
    assert not spilled


@pytest.mark.parametrize("kernel,at_least,most", [("gqsa_gemv_kernel", 200, 16), ("gqsa_panel_", 90, 8)])
def test_kernels_keep_their_registers(code_objects, kernel, at_least, most):
    """A GEMV kernel that runs out of registers waits for its own spills between the loads of x and those of the tile:
    with 24 of them 8 rows of 4096x8192 W8 took longer in one launch than in two of 4 rows.  Four words a lane at most.
    The panel kernels: two words, ahead of the first product and behind the last (see above)."""
    checked, spilled = 0, {}
    for f in code_objects:
        notes = subprocess.run([f"{LLVM}/llvm-readelf", "--notes", str(f)], check=True, capture_output=True, text=True).stdout
        for name, size in re.findall(r"\.name: +(\S+)\n.*?\.private_segment_fixed_size: +(\d+)", notes, re.S):
            if kernel in name:
                checked += 1
                if int(size) > most:
                    spilled[name] = int(size)
    assert checked >= at_least
    assert not spilled
