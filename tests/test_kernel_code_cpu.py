"""Branches of the built tile kernels (dstream.h, dslab.h, dplanar.h, and group.h, which holds bodies of all three), read from their machine code.  Their operand reads from LDS
complete behind the compiler's back, and the compiler copies registers where paths join: a copy of a register whose read is in flight
copies stale data.  So the streaming kernels with row-major B, the slab and the planar kernels may not branch at all between such a
read and its wait, and the other streaming kernels not more often than the loop over the stages needs."""
import os
import re
import subprocess

import pytest

import paper_2210_12415_amd as alt

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"


FAMILIES = ("dstream_kernel", "dslab_kernel", "dplanar_kernel", "group_kernel")


def tile_kernels(folder):
    """family -> template arguments -> [(address, operation, operands)] of every kernel of these families in the library."""
    lib = os.path.join(os.path.dirname(alt.__file__), "libalt.so")
    os.symlink(lib, os.path.join(folder, "lib.so"))
    subprocess.run([OBJDUMP, "--offloading", "lib.so"], cwd=folder, check=True, capture_output=True)
    out = {k: {} for k in FAMILIES}
    for f in sorted(os.listdir(folder)):
        path = os.path.join(folder, f)
        if "gfx950" not in f or not any(k.encode() in open(path, "rb").read() for k in FAMILIES):
            continue
        text = subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", "--demangle", path], check=True, capture_output=True, text=True).stdout
        code = None
        for line in text.splitlines():
            head = re.match(r"^[0-9a-f]+ <(.*)>:$", line)
            if head:
                name = re.search(r"(%s)<(.*)>\(" % "|".join(FAMILIES), head.group(1))
                code = out[name.group(1)].setdefault(name.group(2), []) if name else None
            elif code is not None:
                m = re.match(r"^\s+(\S+)\s*(.*?)\s*//\s*([0-9A-F]+)", line)
                if m:
                    code.append((int(m.group(3), 16), m.group(1), m.group(2)))
    return out


def branches_with_reads_in_flight(code, writes_end=True, most=None):
    """Indices of the branches of the main loop that some path reaches with operand reads in flight.  (It ends with the last matrix
    instruction; in the streaming kernels, which write nothing to LDS themselves before, also with the write that opens the epilogue: the
    compiler keeps the waits of its own reads there.)  most: filled with the instructions reached and the reads in flight there."""
    at = {a: i for i, (a, _, _) in enumerate(code)}
    end = max(i for i, (_, op, _) in enumerate(code) if "mfma" in op)
    most = {} if most is None else most
    todo, found = [(0, 0)], set()
    while todo:
        i, reads = todo.pop()
        if most.get(i, -1) >= reads:
            continue
        most[i] = reads
        address, op, text = code[i]
        if op == "s_endpgm" or (writes_end and op.startswith("ds_write")) or i > end:
            continue
        if op.startswith("ds_read"):
            reads += 1
        elif op == "s_waitcnt" and "lgkmcnt" in text:
            reads = min(reads, int(re.search(r"lgkmcnt\((\d+)\)", text).group(1)))
        elif op == "s_branch" or op.startswith("s_cbranch"):
            if reads:
                found.add(i)
            off = int(text.split()[0])
            todo.append((at[address + 4 + 4 * (off - 65536 if off >= 32768 else off)], reads))
            if op == "s_branch":
                continue
        todo.append((i + 1, reads))
    return found


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    if not os.path.exists(OBJDUMP):
        pytest.skip("no disassembler")
    found = tile_kernels(str(tmp_path_factory.mktemp("code")))
    assert len(found["dstream_kernel"]) > 40
    return found


def test_row_major_b_kernels_do_not_branch_with_reads_in_flight(kernels):
    row_major = {n: c for n, c in kernels["dstream_kernel"].items() if n.split(", ")[7] == "true"}
    assert {n.split(", ")[8] for n in row_major} == {"0", "4"}
    for name, code in row_major.items():
        assert not branches_with_reads_in_flight(code), name


def test_kernels_over_filter_taps_branch_for_the_stages_alone(kernels):
    taps = {n: c for n, c in kernels["dstream_kernel"].items() if n.split(", ")[8] != "0"}
    assert len(taps) >= 20
    for name, code in taps.items():
        # the loop over whole rounds, and each step of the last one is entered or left out
        assert len(branches_with_reads_in_flight(code)) <= 2 * int(name.split(", ")[5]) + 1, name


@pytest.mark.parametrize("family,count", [("dslab_kernel", 42), ("dplanar_kernel", 14)])
def test_slab_and_planar_kernels_do_not_branch_with_reads_in_flight(kernels, family, count):
    assert len(kernels[family]) >= count
    for name, code in kernels[family].items():
        most = {}
        assert not branches_with_reads_in_flight(code, writes_end=False, most=most), name
        assert max(i for i, (_, op, _) in enumerate(code) if "mfma" in op) in most and max(most.values()) >= 2, name    # the loop was walked, with reads in flight


def bodies(code):
    """(first, last) instruction of each body of a kernel that holds several, up to its last matrix instruction: what lies between that and the next
    body's first one is its epilogue, which stores."""
    last, stored, begin, out = None, False, 0, []
    for i, (_, op, _) in enumerate(code):
        if "mfma" in op:
            if stored and last is not None:
                out.append((begin, last))
                begin = last + 1
            last, stored = i, False
        elif op.startswith(("buffer_store", "global_store")):
            stored = True
    return out + [(begin, last)]


@pytest.mark.parametrize("family,most_branches", [("F32", [2 * 3 + 1] * 3 + [2 * 4 + 1] * 3), ("Slab", [0] * 7 + [2 * 3 + 1] * 2), ("Planar", [0] * 8)])
def test_kernels_of_several_bodies_branch_for_the_stages_alone(kernels, family, most_branches):
    """The same for every body of a kernel that holds several: a streaming body branches for its stages (3 or 4), the others not at all.  (Those of the
    slab kernel are told by their products: nine taps.  In an epilogue the compiler keeps the waits of its own reads.)"""
    name, code = next((n, c) for n, c in kernels["group_kernel"].items() if n.endswith("::" + family))
    matters = [i for i, (_, op, _) in enumerate(code) if "mfma" in op or op.startswith(("buffer_store", "global_store"))]
    most, branches = {}, []
    for i in branches_with_reads_in_flight(code, writes_end=False, most=most):
        ahead = next(j for j in matters if j >= i)
        if "mfma" in code[ahead][1]:
            branches.append(i)
    found = bodies(code)
    assert len(found) == len(most_branches), (name, found)
    counts = []
    for first, last in found:
        assert last in most and max(most.get(i, 0) for i in range(first, last)) >= 2, name      # the body was walked, with reads in flight
        counts.append(sum(first <= i <= last for i in branches))
        products = sum("mfma" in code[i][1] for i in range(first, last + 1))
        if family == "Slab" and products % 9 == 0:
            assert counts[-1] == 0, (name, first, last)
    assert all(c <= m for c, m in zip(sorted(counts), most_branches)), (name, counts)
